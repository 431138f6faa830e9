// Device helpers shared by the GEMM kernels that stage their operand tiles with LDS-DMA loads.
#pragma once
#include "sp_common.h"
#include "sp_kernels.h"

struct GemmDev {
    const bf16_t* A; const bf16_t* W; void* C; const float* R; const bf16_t* bias;
    int lda, ldw, ldc, ldr;
    int M, N, K;
    int tilesM, tilesN;
};

typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4_t* lds_s16x4_ptr;

// Transposing LDS read.  The restrict parameter matters: without an alias scope on the read the compiler
// takes it for a possible reader of every LDS-DMA load in flight and waits for all of them (s_waitcnt
// vmcnt(0)) in front of it.  What a read needs is waited for by the kernels themselves.
__device__ __forceinline__ s16x4_t sp_tr_read(lds_s16x4_ptr __restrict p) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16(p); }

// LDS image of one 64-deep operand tile of ROWS rows, as LDS-DMA loads write it (16-byte pieces, a
// wave's 64 pieces land on 1 KiB contiguously, so the bank swizzle sits in which piece a lane fetches).
//   OP_KMAJOR: one 128-byte LDS row per operand row; piece p of row r holds chunk p ^ ((r >> 1) & 7).
//   OP_RMAJOR: one LDS row of 2 ROWS bytes per contraction index; its 64-byte blocks are XOR-ed with
//              k & 3 (row a multiple of 256 bytes) or (k >> 1) & 1 (an odd multiple of 128), so that
//              the four k rows of a transposing read fall into different banks.
template <int ROWS, int FORM>
struct OpTile {
    static constexpr int BYTES = ROWS * 128;
    static constexpr int RB = FORM == OP_KMAJOR ? 128 : ROWS * 2;
    static constexpr int SWZ = FORM == OP_KMAJOR ? 0 : RB % 256 == 0 ? 2 : RB % 128 == 0 ? 1 : 0;
    // what the 16-byte piece at byte `off` of the tile holds: operand row r .. and contraction index k ..
    __device__ static void piece(int off, int* r, int* k) {
        const int row = off / RB, pos = (off % RB) >> 4;
        if (FORM == OP_KMAJOR) {
            *r = row;
            *k = (pos ^ ((row >> 1) & 7)) * 8;
        } else {
            const int s = SWZ == 2 ? row & 3 : SWZ == 1 ? (row >> 1) & 1 : 0;
            *r = (pos ^ (s << 2)) * 8;
            *k = row;
        }
    }
    // lane part of the address of the fragment of the 32-row block `blk`
    __device__ static int frag_base(int blk, int lane) {
        if (FORM == OP_KMAJOR) return blk * 32 * 128 + (lane & 31) * 128;
        const int s16 = lane & 15, half = lane >> 5;
        const int s = SWZ == 2 ? s16 >> 2 : SWZ == 1 ? (s16 >> 3) & 1 : 0;
        return (8 * half + (s16 >> 2)) * RB + ((blk ^ s) << 6) + 32 * ((lane >> 4) & 1) + 8 * (s16 & 3);
    }
    // fragment of 16-deep step ks: lane l -> operand row l & 31 of the block, eight contraction indexes
    // 16 ks + 8 (l >> 5) .. in both forms.  ds_read_b64_tr_b16 works on groups of 16 lanes: lane s of a
    // group supplies the address of four values of one k row, lane i receives element i % 4 of the
    // blocks supplied by lanes i/4, i/4 + 4, i/4 + 8, i/4 + 12.
    __device__ static bf16x8_t frag(const unsigned char* tile, int base, int ks, int lane) {
        if (FORM == OP_KMAJOR) {
            const int sw = ((lane & 31) >> 1) & 7;
            return *reinterpret_cast<const bf16x8_t*>(tile + base + (((2 * ks + (lane >> 5)) ^ sw) << 4));
        }
        const unsigned char* p = tile + base + ks * 16 * RB;
        const s16x4_t lo = sp_tr_read((lds_s16x4_ptr)(p));
        const s16x4_t hi = sp_tr_read((lds_s16x4_ptr)(p + 4 * RB));
        return __builtin_bit_cast(bf16x8_t, s16x8_t{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
    }
};

// The same tile for v_mfma_f32_16x16x32: 32-deep k-steps, fragments of 16 rows, lane l -> operand row l & 15 of the
// block, eight contraction indexes 32 ks + 8 (l >> 4) ..  A row-contiguous tile has its 32-byte pieces XOR-ed with
// (k >> 3) & 1 on top: a transposing read takes 32 bytes of the k rows 8 g .. 8 g + 3 for each group g of 16 lanes, and
// two groups eight rows apart would otherwise share their banks.
template <int ROWS, int FORM>
struct OpTile16 {
    typedef OpTile<ROWS, FORM> T;
    __device__ static void piece(int off, int* r, int* k) {
        T::piece(off, r, k);
        if (FORM == OP_RMAJOR) *r ^= ((*k >> 3) & 1) << 4;
    }
    // lane part of the address of the fragment of the 16-row block `blk`; a contraction-contiguous tile: without the chunk
    __device__ static int frag_base(int blk, int lane) {
        if (FORM == OP_KMAJOR) return blk * 16 * 128 + (lane & 15) * 128;
        const int s16 = lane & 15, g = lane >> 4;
        const int s = T::SWZ == 2 ? s16 >> 2 : T::SWZ == 1 ? (s16 >> 3) & 1 : 0;
        return (8 * g + (s16 >> 2)) * T::RB + ((blk ^ (s << 1) ^ (g & 1)) << 5) + 8 * (s16 & 3);
    }
    __device__ static bf16x8_t frag(const unsigned char* tile, int base, int ks, int lane) {
        if (FORM == OP_KMAJOR) {
            const int sw = ((lane & 15) >> 1) & 7;
            return *reinterpret_cast<const bf16x8_t*>(tile + base + (((4 * ks + (lane >> 4)) ^ sw) << 4));
        }
        const unsigned char* p = tile + base + ks * 32 * T::RB;
        const s16x4_t lo = sp_tr_read((lds_s16x4_ptr)(p));
        const s16x4_t hi = sp_tr_read((lds_s16x4_ptr)(p + 4 * T::RB));
        return __builtin_bit_cast(bf16x8_t, s16x8_t{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
    }
};

// s_waitcnt immediate (gfx9 encoding: vmcnt[3:0] | expcnt << 4 | lgkmcnt << 8 | vmcnt[5:4] << 14)
constexpr int sp_waitcnt(int vm, int lgkm) { return (vm & 15) | (7 << 4) | (lgkm << 8) | ((vm >> 4) << 14); }
// Barrier over LDS traffic only: unlike __syncthreads() it does not wait for global stores.
__device__ __forceinline__ void sp_lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(sp_waitcnt(63, 0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
