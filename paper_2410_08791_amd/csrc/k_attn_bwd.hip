// Attention backward, two deterministic kernels (no atomics):
//   dq kernel    -- a work-group owns 128 queries of one head and walks the key
//                   tiles, like the forward;
//   dk/dv kernel -- a work-group owns 128 keys of one kv head and walks the
//                   query tiles of every query head that shares it.
// Both recompute P = exp(s - lse) from the forward's log-sum-exp and form
// dS = P * (dP - delta), delta = rowsum(dO * O).
//
// MFMA layouts follow the forward kernel.  In the dq kernel scores are formed
// transposed (S^T = K Q^T, dP^T = V dO^T): a lane holds one query, and dS^T in
// bf16 is already the B operand of dQ^T = K^T dS^T.  In the dk/dv kernel scores
// are formed straight (S = Q K^T, dP = dO V^T): a lane holds one key, and P, dS
// in bf16 are the B operands of dV^T = dO^T P and dK^T = Q^T dS.  The A operands
// K^T, dO^T, Q^T are read out of the same token-row LDS tiles the score products use,
// through the transposing LDS read: no transposed copies exist in memory.
//
// Tiles go from memory straight into LDS (global_load_lds_dwordx4), one tile ahead into the
// other of two stages, one barrier per tile.  What bounds the kernels is the chain score MFMAs ->
// exp -> bf16 -> second MFMAs of a wave, so two waves per SIMD are kept in every kernel: the dk/dv
// kernel at head_dim 128 (dK^T and dV^T of 32 keys are 128 registers) gets there with K in LDS and
// V in registers, eight waves sharing 128 keys as 4 key groups x 2 query halves, the halves' sums
// added through LDS at the end.  Before (register staging, two barriers per tile, one wave per
// SIMD at head_dim 128), dq and dk/dv together with rowsum(dO * O), us: 8 x 2048, 32 heads of 128, causal
// 2062 -> 1388; 8 x 1024, 16 heads of 128 399 -> 280; 4 x 1024, 64 query and 8 key heads of 128 748 -> 463;
// 5 x 777, 32 and 8 heads of 64 231 -> 121; 32 x 257, 16 heads of 80, bidirectional 160 -> 145.
#include "sp_gemm.h"

namespace {

// A 64-row token tile in LDS: rows of ROWB bytes (head_dim 80: 192, the padding is never loaded), the 16-byte
// chunk c of row r at position c ^ swz(r).  swz serves both readers: the 16 rows of a straight 16-byte read
// fall on all banks, and the four consecutive rows of a transposing read in different 64-byte blocks.  It has
// period 16 in r, and r + 8 flips exactly bit 1 (the hi half of a transposed fragment: address ^ 32).
template <int HD>
struct TokTile {
    static constexpr int ROWB = HD == 80 ? 192 : HD * 2, CPR = HD / 8;
    static constexpr int NKS = HD / 16, NMT = (HD + 31) / 32;
    static constexpr int ROWS = 64, BYTES = ROWS * ROWB;
    __device__ static int swz(int r) {
        return HD == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : HD == 64 ? (((r >> 1) & 1) << 2) | ((r >> 2) & 3) : (r >> 2) & 3;
    }
    // lane part of the straight fragment of k-step ks: row l32, head-dimension elements 16 ks + 8 half ..
    __device__ static int row_pos(int ks, int l32, int half) { return l32 * ROWB + (((2 * ks + half) ^ swz(l32)) << 4); }
    __device__ static bf16x8_t row_frag(const unsigned char* p) { return *reinterpret_cast<const bf16x8_t*>(p); }
    // Transposed MFMA operand: the lane ends up with head-dimension row (lane & 31) of the 32-row block mt and
    // the eight tokens 4*half + {0..3} and 8 + 4*half + {0..3} of a 16-token step -- the token order in which
    // the score tiles hold their bf16 operands.  ds_read_b64_tr_b16 works on groups of 16 lanes: lane s
    // supplies the address of four values of one token row, lane i receives element i%4 of the blocks
    // supplied by lanes i/4, i/4+4, i/4+8, i/4+12.
    __device__ static int tr_pos(int mt, int lane) {
        const int s16 = lane & 15, row = 4 * (lane >> 5) + (s16 >> 2);
        const int chunk = mt * 4 + 2 * ((lane >> 4) & 1) + ((s16 & 3) >> 1);
        return row * ROWB + ((chunk ^ swz(row)) << 4) + (s16 & 1) * 8;
    }
    __device__ static bf16x8_t tr_frag(const unsigned char* step, int pos) {
        const s16x4_t lo = sp_tr_read((lds_s16x4_ptr)(step + pos));
        const s16x4_t hi = sp_tr_read((lds_s16x4_ptr)(step + (pos ^ 32) + 8 * ROWB));
        return __builtin_bit_cast(bf16x8_t, s16x8_t{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
    }
};

// Loads of one stage: two token tiles (X, then Y) of the same rows, NW waves.  Instruction i of a wave lands at
// byte (wave * NI + i) * 1024 + lane * 16 of the stage.
template <int HD, int NW>
struct StageLoad {
    typedef TokTile<HD> T;
    static constexpr int STAGE = 2 * T::BYTES, NI = STAGE / 1024 / NW;
    static_assert(STAGE % (1024 * NW) == 0 && T::BYTES % 1024 == 0, "whole load instructions per wave and tile");
    int row[NI], col[NI];
    bool on[NI], y[NI];
    __device__ __forceinline__ void init(int wave, int lane) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int blk = wave * NI + i;
            y[i] = blk >= T::BYTES / 1024;                      // wave-uniform
            const int rel = blk * 1024 + lane * 16 - (y[i] ? T::BYTES : 0);
            row[i] = rel / T::ROWB;
            const int c = ((rel % T::ROWB) >> 4) ^ T::swz(row[i]);
            on[i] = c < T::CPR;
            col[i] = on[i] ? c * 8 : 0;
        }
    }
    // rows r0 .. of X and Y, clamped to lastx / lasty
    __device__ __forceinline__ void issue(unsigned char* stage, int wave, const bf16_t* X, int ldx, const bf16_t* Y, int ldy,
                                          int r0, int lastx, int lasty) const {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const ptrdiff_t r = min(r0 + row[i], y[i] ? lasty : lastx);
            const bf16_t* src = (y[i] ? Y + r * ldy : X + r * ldx) + col[i];
            if (on[i]) __builtin_amdgcn_global_load_lds(src, (lds_void_ptr)(stage + (wave * NI + i) * 1024), 16, 0, 0);
        }
#endif
    }
};

__device__ __forceinline__ void stage_ready() {
    // this wave's loads have landed and its LDS accesses are complete; after the barrier every wave's
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(sp_waitcnt(0, 0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// LDS read with an alias scope (restrict), for the reason given at sp_tr_read
__device__ __forceinline__ float4 lds_f4(const float* __restrict__ p) { return *reinterpret_cast<const float4*>(p); }

__device__ __forceinline__ f32x16_t zero16() {
    f32x16_t z;
#pragma unroll
    for (int e = 0; e < 16; ++e) z[e] = 0.f;
    return z;
}

// ------------------------------------------------------------------------- dq
// A work-group owns 128 queries of one head (a wave 32 of them, one query per lane as the B
// operand) and walks 64-key tiles: S^T = K Q^T and dP^T = V dO^T read the tiles straight,
// dQ^T += K^T dS^T reads K through the transposing LDS read.
template <int HD>
__global__ __launch_bounds__(256, 2) void attn_bwd_dq_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dO,
                                                          const float* __restrict__ lse, const float* __restrict__ delta,
                                                          bf16_t* __restrict__ dqkv, int S, int Hq, int Hkv, int ld_qkv,
                                                          int causal, float scale, float scale_log2e) {
    typedef TokTile<HD> T;
    typedef StageLoad<HD, 4> Load;
    constexpr int KB = T::ROWS;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    // work-group ids are dealt round-robin to the 8 XCDs: remapped so that an XCD works through a
    // contiguous range of (batch, head, query block) and a head's keys and values are fetched
    // through one L2
    const int job = xcd_remap(blockIdx.x + (int)gridDim.x * (blockIdx.y + (int)gridDim.y * blockIdx.z),
                              (int)(gridDim.x * gridDim.y * gridDim.z));
    const int bx = job % (int)gridDim.x, h = (job / (int)gridDim.x) % (int)gridDim.y, b = job / (int)(gridDim.x * gridDim.y);
    const int qb = causal ? gridDim.x - 1 - bx : bx;
    const int kvh = h / (Hq / Hkv);
    const int q0 = qb * 128, wq0 = q0 + wave * 32, qi = wq0 + l32;
    const size_t tok0 = (size_t)b * S;
    const int qr = min(qi, S - 1);
    const bf16_t* kbase = qkv + tok0 * ld_qkv + (size_t)Hq * HD + (size_t)kvh * HD;
    const bf16_t* vbase = kbase + (size_t)Hkv * HD;
    const int k_end = causal ? min(S, q0 + 128) : S;
    const int ntiles = (k_end + KB - 1) / KB;
    Load ld;
    ld.init(wave, lane);
    ld.issue(smem, wave, kbase, ld_qkv, vbase, ld_qkv, 0, S - 1, S - 1);

    bf16x8_t qf[T::NKS], dof[T::NKS];
    {
        const bf16_t* qp = qkv + (tok0 + qr) * ld_qkv + h * HD + half * 8;
        const bf16_t* dp = dO + (tok0 + qr) * (size_t)(Hq * HD) + h * HD + half * 8;
#pragma unroll
        for (int ks = 0; ks < T::NKS; ++ks) {
            qf[ks] = *reinterpret_cast<const bf16x8_t*>(qp + ks * 16);
            dof[ks] = *reinterpret_cast<const bf16x8_t*>(dp + ks * 16);
        }
    }
    const float lse_q = lse[((size_t)b * Hq + h) * S + qr] * 1.4426950408889634f;
    const float delta_q = delta[((size_t)b * Hq + h) * S + qr];
    int kpos[T::NKS], tpos[T::NMT];
#pragma unroll
    for (int ks = 0; ks < T::NKS; ++ks) kpos[ks] = T::row_pos(ks, l32, half);
#pragma unroll
    for (int mt = 0; mt < T::NMT; ++mt) tpos[mt] = T::tr_pos(mt, lane);

    f32x16_t acc[T::NMT];
#pragma unroll
    for (int t = 0; t < T::NMT; ++t) acc[t] = zero16();

    stage_ready();
    for (int tile = 0; tile < ntiles; ++tile) {
        const int key0 = tile * KB;
        if (tile + 1 < ntiles) ld.issue(smem + ((tile + 1) & 1) * Load::STAGE, wave, kbase, ld_qkv, vbase, ld_qkv, key0 + KB, S - 1, S - 1);
        const unsigned char* sK = smem + (tile & 1) * Load::STAGE;
        const unsigned char* sV = sK + T::BYTES;
        // wave-uniform skips: no key of the tile visible, no query of this wave exists
        if (!((causal && key0 > wq0 + 31) || wq0 >= S)) {
            const bool need_mask = (causal && key0 + KB - 1 > wq0) || key0 + KB > S;
            bf16x8_t dsf[2][2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                f32x16_t s = zero16(), dp = zero16();
#pragma unroll
                for (int ks = 0; ks < T::NKS; ++ks) {
                    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(T::row_frag(sK + t * 32 * T::ROWB + kpos[ks]), qf[ks], s, 0, 0, 0);
                    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(T::row_frag(sV + t * 32 * T::ROWB + kpos[ks]), dof[ks], dp, 0, 0, 0);
                }
                if (need_mask) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int key = key0 + t * 32 + (e >> 2) * 8 + half * 4 + (e & 3);
                        if (key >= S || (causal && key > qi)) s[e] = -INFINITY;
                    }
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(s[e], scale_log2e, -lse_q));
                    dsf[t][e >> 3][e & 7] = (__bf16)(p * (dp[e] - delta_q));
                }
            }
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int mt = 0; mt < T::NMT; ++mt)
                        acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            T::tr_frag(sK + (t * 32 + 16 * j) * T::ROWB, tpos[mt]), dsf[t][j], acc[mt], 0, 0, 0);
        }
        if (tile + 1 < ntiles) stage_ready();
    }
    if (qi < S) {
        bf16_t* op = dqkv + (tok0 + qi) * ld_qkv + h * HD;
#pragma unroll
        for (int mt = 0; mt < T::NMT; ++mt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int e0 = mt * 32 + g * 8 + half * 4;
                if (e0 < HD)
                    *reinterpret_cast<uint2*>(op + e0) =
                        make_uint2(pack_bf2(acc[mt][g * 4] * scale, acc[mt][g * 4 + 1] * scale),
                                   pack_bf2(acc[mt][g * 4 + 2] * scale, acc[mt][g * 4 + 3] * scale));
            }
    }
}

// ---------------------------------------------------------------------- dk, dv
// A work-group owns 128 keys of one kv head and walks 64-query tiles of every query head of the group.
// Wave w takes the 32 keys of group w & 3 (one key per lane as the B operand of S = Q K^T and dP = dO V^T)
// against the query half w >> 2 of each tile: the score products read the Q and dO tiles straight,
// dV^T += dO^T P and dK^T += Q^T dS through the transposing LDS read.
template <int HD>
struct DkvCfg {
    static constexpr bool K_IN_LDS = HD == 128;      // K fragments would not fit beside the accumulators
    static constexpr int KBYTES = K_IN_LDS ? 2 * TokTile<HD>::BYTES : 0;      // 128 key rows
    static constexpr int ROWVALS = 2 * 64 * 2 * 4;   // two stages of lse and delta of 64 queries
    static constexpr int LDS = 2 * StageLoad<HD, 8>::STAGE + KBYTES + ROWVALS;
    static_assert(4 * TokTile<HD>::NMT * 16 * 256 <= 2 * StageLoad<HD, 8>::STAGE, "one accumulator set of four waves fits the stages");
};

template <int HD>
__global__ __launch_bounds__(512) void attn_bwd_dkv_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dO,
                                                           const float* __restrict__ lse, const float* __restrict__ delta,
                                                           bf16_t* __restrict__ dqkv, int S, int Hq, int Hkv,
                                                           int ld_qkv, int causal, float scale, float scale_log2e) {
    typedef TokTile<HD> T;
    typedef StageLoad<HD, 8> Load;
    typedef DkvCfg<HD> C;
    constexpr int QT = T::ROWS;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* sKeys = smem + 2 * Load::STAGE;
    float* rowvals = reinterpret_cast<float*>(smem + 2 * Load::STAGE + C::KBYTES);   // [stage][lse | delta][64]

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5, kg = wave & 3, sub = wave >> 2;
    // the same XCD-contiguous order as in the dq kernel: the key blocks of a head share its queries
    const int job = xcd_remap(blockIdx.x + (int)gridDim.x * (blockIdx.y + (int)gridDim.y * blockIdx.z),
                              (int)(gridDim.x * gridDim.y * gridDim.z));
    const int bx = job % (int)gridDim.x, kvh = (job / (int)gridDim.x) % (int)gridDim.y, b = job / (int)(gridDim.x * gridDim.y);
    const int grp = Hq / Hkv;
    const int k0 = bx * 128, wk0 = k0 + kg * 32, kj = wk0 + l32;
    const size_t tok0 = (size_t)b * S;
    const int ld_do = Hq * HD;
    const bf16_t* kbase = qkv + tok0 * ld_qkv + (size_t)Hq * HD + (size_t)kvh * HD;
    const bf16_t* vbase = kbase + (size_t)Hkv * HD;

    // the tiles of this work-group in walking order: (query head of the group, 64-query tile)
    const int q_begin = causal ? (k0 / QT) * QT : 0;
    const int tiles_per_head = (S - q_begin + QT - 1) / QT;
    const int n_tiles = grp * tiles_per_head;            // at least one: k0 < S
    Load ld;
    ld.init(wave, lane);
    float r_lse = 0.f, r_delta = 0.f;
    auto fetch = [&](int tile) {
        const int h = kvh * grp + tile / tiles_per_head;
        const int q0 = q_begin + (tile % tiles_per_head) * QT;
        ld.issue(smem + (tile & 1) * Load::STAGE, wave, qkv + tok0 * ld_qkv + h * HD, ld_qkv, dO + tok0 * ld_do + h * HD, ld_do, q0, S - 1, S - 1);
        if (threadIdx.x < QT) {
            const size_t row = ((size_t)b * Hq + h) * S + min(q0 + (int)threadIdx.x, S - 1);
            r_lse = lse[row] * 1.4426950408889634f;
            r_delta = delta[row];
        }
    };
    auto put_rowvals = [&](int tile) {
        if (threadIdx.x < QT) {
            rowvals[(tile & 1) * 128 + threadIdx.x] = r_lse;
            rowvals[(tile & 1) * 128 + 64 + threadIdx.x] = r_delta;
        }
    };
    // the two 64-row halves of the keys have the form of a stage's two tiles (rows clamped to S - 1 in both)
    if (C::K_IN_LDS) ld.issue(sKeys, wave, kbase, ld_qkv, kbase + (ptrdiff_t)64 * ld_qkv, ld_qkv, k0, S - 1, S - 1 - 64);
    fetch(0);

    bf16x8_t kf[C::K_IN_LDS ? 1 : T::NKS], vf[T::NKS];
    {
        const size_t kr = min(kj, S - 1);
#pragma unroll
        for (int ks = 0; ks < T::NKS; ++ks) {
            if (!C::K_IN_LDS) kf[C::K_IN_LDS ? 0 : ks] = *reinterpret_cast<const bf16x8_t*>(kbase + kr * ld_qkv + half * 8 + ks * 16);
            vf[ks] = *reinterpret_cast<const bf16x8_t*>(vbase + kr * ld_qkv + half * 8 + ks * 16);
        }
    }
    int rpos[T::NKS], tpos[T::NMT];
#pragma unroll
    for (int ks = 0; ks < T::NKS; ++ks) rpos[ks] = T::row_pos(ks, l32, half);
#pragma unroll
    for (int mt = 0; mt < T::NMT; ++mt) tpos[mt] = T::tr_pos(mt, lane);
    f32x16_t dk[T::NMT], dv[T::NMT];
#pragma unroll
    for (int t = 0; t < T::NMT; ++t) { dk[t] = zero16(); dv[t] = zero16(); }

    put_rowvals(0);
    stage_ready();
    for (int tile = 0; tile < n_tiles; ++tile) {
        const bool more = tile + 1 < n_tiles;
        if (more) fetch(tile + 1);
        const unsigned char* sQ = smem + (tile & 1) * Load::STAGE + sub * 32 * T::ROWB;
        const unsigned char* sdO = sQ + T::BYTES;
        const float* lrow = rowvals + (tile & 1) * 128 + sub * 32 + half * 4;
        const int qs = q_begin + (tile % tiles_per_head) * QT + sub * 32;
        // wave-uniform skips: every query of the half precedes this wave's keys, none exists, no key exists
        if (!(qs >= S || wk0 >= S || (causal && qs + 31 < wk0))) {
            f32x16_t s = zero16(), dp = zero16();
#pragma unroll
            for (int ks = 0; ks < T::NKS; ++ks) {
                const bf16x8_t kfr = C::K_IN_LDS ? T::row_frag(sKeys + kg * 32 * T::ROWB + rpos[ks]) : kf[C::K_IN_LDS ? 0 : ks];
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(T::row_frag(sQ + rpos[ks]), kfr, s, 0, 0, 0);
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(T::row_frag(sdO + rpos[ks]), vf[ks], dp, 0, 0, 0);
            }
            if ((causal && qs < wk0 + 31) || qs + 32 > S) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int q = qs + (e >> 2) * 8 + half * 4 + (e & 3);
                    if (q >= S || (causal && kj > q)) s[e] = -INFINITY;
                }
            }
            bf16x8_t pf[2], dsf[2];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 l4 = lds_f4(lrow + g * 8);
                const float4 d4 = lds_f4(lrow + 64 + g * 8);
                const float l[4] = {l4.x, l4.y, l4.z, l4.w}, dl[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int e = g * 4 + i;
                    const float p = __builtin_amdgcn_exp2f(fmaf(s[e], scale_log2e, -l[i]));
                    pf[e >> 3][e & 7] = (__bf16)p;
                    dsf[e >> 3][e & 7] = (__bf16)(p * (dp[e] - dl[i]));
                }
            }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int mt = 0; mt < T::NMT; ++mt) {
                    dv[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(T::tr_frag(sdO + 16 * j * T::ROWB, tpos[mt]), pf[j], dv[mt], 0, 0, 0);
                    dk[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(T::tr_frag(sQ + 16 * j * T::ROWB, tpos[mt]), dsf[j], dk[mt], 0, 0, 0);
                }
        }
        if (more) put_rowvals(tile + 1);
        stage_ready();
    }
    // The query halves' sums meet in the stages: half 1 hands dK^T to half 0, then half 0 dV^T to half 1.
    float4* x = reinterpret_cast<float4*>(smem) + kg * (T::NMT * 4 * 64) + lane;
    auto give = [&](const f32x16_t* a) {
#pragma unroll
        for (int t = 0; t < T::NMT; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                x[(t * 4 + g) * 64] = make_float4(a[t][g * 4], a[t][g * 4 + 1], a[t][g * 4 + 2], a[t][g * 4 + 3]);
    };
    auto take_and_store = [&](const f32x16_t* a, int col, float f) {
        bf16_t* out = dqkv + (tok0 + min(kj, S - 1)) * ld_qkv + (size_t)(Hq + col) * HD + (size_t)kvh * HD;
#pragma unroll
        for (int t = 0; t < T::NMT; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 o = x[(t * 4 + g) * 64];
                const int e0 = t * 32 + g * 8 + half * 4;
                if (kj < S && e0 < HD)
                    *reinterpret_cast<uint2*>(out + e0) =
                        make_uint2(pack_bf2((a[t][g * 4] + o.x) * f, (a[t][g * 4 + 1] + o.y) * f),
                                   pack_bf2((a[t][g * 4 + 2] + o.z) * f, (a[t][g * 4 + 3] + o.w) * f));
            }
    };
    if (sub == 1) give(dk);
    sp_lds_barrier();
    if (sub == 0) take_and_store(dk, 0, scale);
    sp_lds_barrier();
    if (sub == 0) give(dv);
    sp_lds_barrier();
    if (sub == 1) take_and_store(dv, Hkv, 1.0f);
}

template <int HD>
hipError_t launch_bwd(hipStream_t st, const AttnBwdArgs& g, const AttnShape& a) {
    constexpr int LDS_Q = 2 * StageLoad<HD, 4>::STAGE, LDS_KV = DkvCfg<HD>::LDS;
    static LdsLimitOnce lim_q, lim_kv;
    hipError_t e = lim_q.set(reinterpret_cast<const void*>(attn_bwd_dq_kernel<HD>), LDS_Q);
    if (e == hipSuccess) e = lim_kv.set(reinterpret_cast<const void*>(attn_bwd_dkv_kernel<HD>), LDS_KV);
    if (e != hipSuccess) return e;
    const float scale = 1.0f / sqrtf((float)a.hd), sl2 = scale * 1.4426950408889634f;
    dim3 gq((a.S + 127) / 128, a.Hq, a.B);
    attn_bwd_dq_kernel<HD><<<gq, 256, LDS_Q, st>>>(g.qkv, g.dO, g.lse, g.delta, g.dqkv, a.S, a.Hq, a.Hkv, a.ld_qkv, a.causal,
                                                   scale, sl2);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    dim3 gk((a.S + 127) / 128, a.Hkv, a.B);
    attn_bwd_dkv_kernel<HD><<<gk, 512, LDS_KV, st>>>(g.qkv, g.dO, g.lse, g.delta, g.dqkv, a.S, a.Hq, a.Hkv, a.ld_qkv,
                                                     a.causal, scale, sl2);
    return hipGetLastError();
}

}  // namespace

hipError_t spk_launch_attention_bwd(hipStream_t st, const AttnBwdArgs& g, const AttnShape& a) {
    if (a.B <= 0 || a.S <= 0) return hipSuccess;
    if (a.Hkv <= 0 || a.Hq % a.Hkv || a.ld_qkv % 8 || a.B > 65535 || a.Hq > 65535) return hipErrorInvalidValue;
    if (!g.qkv || !g.dO || !g.lse || !g.delta || !g.dqkv) return hipErrorInvalidValue;
    switch (a.hd) {
        case 64: return launch_bwd<64>(st, g, a);
        case 80: return launch_bwd<80>(st, g, a);
        case 128: return launch_bwd<128>(st, g, a);
    }
    return hipErrorInvalidValue;
}
