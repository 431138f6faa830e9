// Sizes shared by the workspace carving and the backward kernels' launchers.
#pragma once
#include <stddef.h>
#define SPK_NORM_BWD_BLOCKS 256   // partial rows of the gain-gradient reduction
#define SPK_MSE_PARTS 1024        // partial sums of the loss reduction
#define SPK_STATIC_MAX_D 4096      // widest row spk_rmsnorm_bwd_static's built-in partial-row array holds
#define SPK_SPIN_MAX_US 20000        // longest delay one spin kernel may take (debug delay mode)
constexpr int kDecodeMaxLen = 32768;      // longest key/value cache
// Decode attention splits the positions while (sequences x key/value heads x splits) stays within this
// many work-groups, two per CU; each leaves one row of partial results per query head.
constexpr int kDecodeSplitGroups = 512;
inline size_t decode_scratch_floats(int n_q_heads, int n_kv_heads, int head_dim) {
    return (size_t)(n_q_heads / n_kv_heads) * kDecodeSplitGroups * (head_dim + 2);
}
