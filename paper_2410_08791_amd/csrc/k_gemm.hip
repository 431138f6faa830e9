// bf16 GEMM on the gfx950 matrix cores: C[M,N] = sum_k A(m,k) W(n,k), fp32
// accumulate, used for every dense projection of a layer (QKV, O, gate/up,
// down) and for the backward contractions.
//
// Block tile BM x BN x 64.  Both operand tiles are staged in LDS with the contraction index contiguous
// (128-byte rows, 16-byte chunks XOR-swizzled so that both the 16-byte stores
// and the per-lane 16-byte fragment loads spread over all banks), more than one k-tile
// deep.  Two kernels build that LDS image: gemm_dma_kernel (global loads
// that write LDS directly; every projection, forward and backward; v_mfma_f32_16x16x32_bf16) and gemm_kernel
// (register staging: global loads for tile t+1 are issued before the MFMAs of tile t
// and stored to the other buffer afterwards, one barrier per tile; takes the outputs
// whose rows do not start on 16 bytes, which the other kernel's epilogue cannot write, and operands beyond the reach of
// its 32-bit lane offsets; 4 or 8 waves in a 2 x (waves/2)
// grid, each with its share as 32x32 tiles of v_mfma_f32_32x32x16_bf16).
//
// The MFMA is issued "transposed" (weights as the A operand, activations as B)
// so that a lane's four consecutive accumulator registers are four consecutive
// n of one row m: the epilogue then writes 8-byte (bf16) or 16-byte (fp32)
// pieces of a row instead of single elements.
//
// An operand whose contraction index is NOT contiguous in memory (the backward
// GEMMs) is staged as it lies in memory (LDS row = contraction index) and read
// with the transposing LDS load of gfx950 (ds_read_b64_tr_b16), which hands each
// lane four consecutive contraction elements of one operand row.
#include "sp_gemm.h"

namespace {

constexpr int BK = 64;
constexpr int ROW_BYTES = BK * 2;  // 128

__device__ __forceinline__ int lds_off(int row, int chunk) {
    return row * ROW_BYTES + ((chunk ^ ((row >> 1) & 7)) << 4);
}

// ---- tile loaders -----------------------------------------------------------
// K-major source: rows of 64 contiguous k. ROWS*8 16-byte chunks over 256 threads.
template <int ROWS, int NT>
struct LoaderK {
    static constexpr int ITERS = ROWS * 8 / NT;
    static constexpr int N_LOADS = ITERS, N_STORES = ITERS;   // per thread and tile
    const bf16_t* src[ITERS];
    int dst[ITERS];
    u32x4_t regs[ITERS];
    // row_of(r) maps a tile row to a (clamped) global row.
    template <class RowMap>
    __device__ __forceinline__ void init(const bf16_t* base, int ld, RowMap row_of) {
#pragma unroll
        for (int i = 0; i < ITERS; ++i) {
            const int q = threadIdx.x + i * NT;
            const int row = q >> 3, c = q & 7;
            src[i] = base + (size_t)row_of(row) * ld + c * 8;
            dst[i] = lds_off(row, c);
        }
    }
    __device__ __forceinline__ void fetch(int k0) {
#pragma unroll
        for (int i = 0; i < ITERS; ++i) regs[i] = *reinterpret_cast<const u32x4_t*>(src[i] + k0);
    }
    __device__ __forceinline__ void store(unsigned char* lds) {
#pragma unroll
        for (int i = 0; i < ITERS; ++i) *reinterpret_cast<u32x4_t*>(lds + dst[i]) = regs[i];
    }
};

// Row-major source (element (r,k) at base[k*ld + r]): the tile is copied as it lies in
// memory -- LDS row = contraction index k (64 rows), ROWS contiguous r values per row, rows
// padded by 64 bytes -- with the same coalesced 16-byte chunks as above.  The transposition
// happens in the fragment read (ds_read_b64_tr_b16, see tr_frag below).
template <int ROWS>
struct TLayout {
    static constexpr int STRIDE = ROWS * 2 + 64;   // bytes per k row
    static constexpr int BYTES = BK * STRIDE;
};

template <int ROWS, int NT>
struct LoaderR {
    static constexpr int CPR = ROWS / 8;           // 16-byte chunks per k row
    static constexpr int ITERS = BK * CPR / NT;
    static constexpr int N_LOADS = ITERS, N_STORES = ITERS;
    const bf16_t* src[ITERS];
    int dst[ITERS];
    int ld_;
    u32x4_t regs[ITERS];
    // col_of(r) maps the tile's first r of a chunk to a (clamped) global r.
    template <class ColMap>
    __device__ __forceinline__ void init(const bf16_t* base, int ld, ColMap col_of) {
        ld_ = ld;
#pragma unroll
        for (int i = 0; i < ITERS; ++i) {
            const int q = threadIdx.x + i * NT;
            const int k = q / CPR, c = q % CPR;
            src[i] = base + (size_t)k * ld + col_of(c * 8);
            dst[i] = k * TLayout<ROWS>::STRIDE + c * 16;
        }
    }
    __device__ __forceinline__ void fetch(int k0) {
#pragma unroll
        for (int i = 0; i < ITERS; ++i) regs[i] = *reinterpret_cast<const u32x4_t*>(src[i] + (size_t)k0 * ld_);
    }
    __device__ __forceinline__ void store(unsigned char* lds) {
#pragma unroll
        for (int i = 0; i < ITERS; ++i) *reinterpret_cast<u32x4_t*>(lds + dst[i]) = regs[i];
    }
};

// Fragment of a 32-row MFMA operand out of a k-row tile.  ds_read_b64_tr_b16 works on
// groups of 16 lanes: lane s of a group supplies the address of an 8-byte block (4 values of
// one k row), and lane i receives element i%4 of the blocks supplied by lanes i/4, i/4+4,
// i/4+8, i/4+12 (layout checked on the device with an index pattern).  With lane s pointing at
// k row (s>>2) and r block 4*(s&3), lane i ends up with r = 4*(i>>2) + (i&3) = i and four
// consecutive k: two reads give the eight k of a lane's operand, in the same order as the
// 16-byte read of a k-contiguous tile, so both operand forms can be mixed.
__device__ __forceinline__ bf16x8_t tr_frag(const unsigned char* p, int stride) {
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * stride));
    const s16x8_t both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8_t, both);
}

template <int ROWS, int NT, int FORM>
struct LoaderSel { typedef LoaderK<ROWS, NT> type; };
template <int ROWS, int NT>
struct LoaderSel<ROWS, NT, OP_RMAJOR> { typedef LoaderR<ROWS, NT> type; };

// Epilogue of the register-staged kernel.  acc[j][i] is the 32x32 tile (n tile j, m tile i) of
// a wave whose first row is m_base and first output column n_base; a lane holds row l32 of
// the m tile and, in register e, column j*32 + (e/4)*8 + half*4 + e%4.
template <int EPI, int TM, int TN>
__device__ __forceinline__ void gemm_epilogue(const GemmDev& p, f32x16_t (&acc)[TN][TM], int m_base, int n_base,
                                              int l32, int half) {
    constexpr bool SWIGLU = (EPI == EPI_SWIGLU_BF16);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m_base + i * 32 + l32;
        if (m >= p.M) continue;
        if (SWIGLU) {
#pragma unroll
            for (int j = 0; j < TN / 2; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int n = n_base + j * 32 + g * 8 + half * 4;
                    if (n >= p.N) continue;
                    float z[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float gv = acc[j][i][g * 4 + e], uv = acc[j + TN / 2][i][g * 4 + e];
                        z[e] = gv * __builtin_amdgcn_rcpf(1.0f + __expf(-gv)) * uv;
                    }
                    *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(p.C) + (size_t)m * p.ldc + n) =
                        make_uint2(pack_bf2(z[0], z[1]), pack_bf2(z[2], z[3]));
                }
        } else {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int n = n_base + j * 32 + g * 8 + half * 4;
                    if (n >= p.N) continue;
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc[j][i][g * 4 + e];
                    if (p.bias) {
                        const uint2 b = *reinterpret_cast<const uint2*>(p.bias + n);
                        v[0] += bf_lo(b.x); v[1] += bf_hi(b.x); v[2] += bf_lo(b.y); v[3] += bf_hi(b.y);
                    }
                    if (EPI == EPI_RESID_F32) {
                        const float4 r = *reinterpret_cast<const float4*>(p.R + (size_t)m * p.ldr + n);
                        *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.C) + (size_t)m * p.ldc + n) =
                            make_float4(r.x + v[0], r.y + v[1], r.z + v[2], r.w + v[3]);
                    } else if (EPI == EPI_F32) {
                        *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.C) + (size_t)m * p.ldc + n) =
                            make_float4(v[0], v[1], v[2], v[3]);
                    } else {
                        if (EPI == EPI_GELU_BF16) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] = gelu_erf(v[e]);
                        }
                        *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(p.C) + (size_t)m * p.ldc + n) =
                            make_uint2(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]));
                    }
                }
        }
    }
}


// ---- the kernel ---------------------------------------------------------------
template <int BM, int BN, int EPI, int AFORM, int WFORM, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void gemm_kernel(GemmDev p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int NT = WAVES * 64;
    constexpr int WNC = WAVES / 2;               // wave grid: 2 (m) x WNC (n)
    constexpr int WN = BN / WNC;                 // tile rows of W per wave column
    constexpr int TM = BM / 64, TN = WN / 32;    // 32x32 tiles per wave
    constexpr int A_BYTES = AFORM == OP_KMAJOR ? BM * ROW_BYTES : TLayout<BM>::BYTES;
    constexpr int W_BYTES = WFORM == OP_KMAJOR ? BN * ROW_BYTES : TLayout<BN>::BYTES;
    constexpr int STAGE = A_BYTES + W_BYTES;
    constexpr bool SWIGLU = (EPI == EPI_SWIGLU_BF16);
    constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;  // output columns per block
    static_assert(!SWIGLU || (TN % 2 == 0), "gate and up tiles pair up inside a wave");

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int l32 = lane & 31, half = lane >> 5;

    // XCD-aware, grouped tile order: 8 m-tiles share each n-tile back to back.
    int pid = xcd_remap(blockIdx.x, gridDim.x);
    constexpr int GM = 8;
    const int group = GM * p.tilesN;
    const int first_m = (pid / group) * GM;
    const int gm = min(p.tilesM - first_m, GM);
    const int tm = first_m + (pid % group) % gm;
    const int tn = (pid % group) / gm;
    const int m0 = tm * BM, n0 = tn * BN_OUT;

    typename LoaderSel<BM, NT, AFORM>::type la;
    typename LoaderSel<BN, NT, WFORM>::type lw;
    {
        const int M = p.M, N = p.N;
        if (AFORM == OP_KMAJOR)
            la.init(p.A, p.lda, [=](int r) { return min(m0 + r, M - 1); });
        else
            la.init(p.A, p.lda, [=](int r) { return min(m0 + r, M - 8); });
        if (SWIGLU) {
            // tile row r -> wave column wr, 32-row tile j; first half of a wave's
            // tiles are gate rows, second half the matching up rows (offset N).
            lw.init(p.W, p.ldw, [=](int r) {
                const int wr = r / WN, j = (r % WN) >> 5, rr = r & 31;
                const int isup = j >= TN / 2;
                const int col = n0 + wr * (WN / 2) + (isup ? j - TN / 2 : j) * 32 + rr;
                return min(col, N - 1) + (isup ? N : 0);
            });
        } else if (WFORM == OP_KMAJOR) {
            lw.init(p.W, p.ldw, [=](int r) { return min(n0 + r, N - 1); });
        } else {
            lw.init(p.W, p.ldw, [=](int r) { return min(n0 + r, N - 8); });
        }
    }

    f32x16_t acc[TN][TM];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][i][e] = 0.f;

    // per-lane fragment offsets: row l32 of a 32-row tile, chunk 2*ks + half
    const int sw = (l32 >> 1) & 7;
    int foff[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) foff[ks] = l32 * ROW_BYTES + (((2 * ks + half) ^ sw) << 4);
    // k-row tiles: lane -> k row 8*half + (s>>2), r block 16*((lane>>4)&1) + 4*(s&3), s = lane&15
    const int s16 = lane & 15;
    const int tro_a = (8 * half + (s16 >> 2)) * TLayout<BM>::STRIDE + (16 * ((lane >> 4) & 1) + 4 * (s16 & 3)) * 2;
    const int tro_w = (8 * half + (s16 >> 2)) * TLayout<BN>::STRIDE + (16 * ((lane >> 4) & 1) + 4 * (s16 & 3)) * 2;
    const int a_base = AFORM == OP_KMAJOR ? wm * (BM / 2) * ROW_BYTES : wm * (BM / 2) * 2 + tro_a;
    const int w_base = A_BYTES + (WFORM == OP_KMAJOR ? wn * WN * ROW_BYTES : wn * WN * 2 + tro_w);

    const int KT = p.K / BK;
    la.fetch(0);
    lw.fetch(0);
    la.store(smem);
    lw.store(smem + A_BYTES);
    __syncthreads();

    // Main loop, one barrier per 64-deep tile.  The body is branch-free (the last
    // iteration re-fetches the last tile into the idle buffer) so that it is one
    // scheduling region; fragments are double buffered in registers and the
    // scheduling hints interleave the LDS reads of step s+1 with the MFMAs of step
    // s, and the LDS stores of the next tile with the MFMAs of the last step.
    constexpr int NFRAG = TM + TN, NMFMA = TM * TN;
    typedef typename LoaderSel<BM, NT, AFORM>::type LA;
    typedef typename LoaderSel<BN, NT, WFORM>::type LW;
    constexpr int LA_LOADS = LA::N_LOADS, LW_LOADS = LW::N_LOADS, LA_STORES = LA::N_STORES, LW_STORES = LW::N_STORES;
    constexpr int M_MFMA = 0x008, M_VMEM_RD = 0x020, M_DS_RD = 0x100, M_DS_WR = 0x200;
    for (int kt = 0; kt < KT; ++kt) {
        unsigned char* cur = smem + (kt & 1) * STAGE;
        unsigned char* nxt = smem + ((kt + 1) & 1) * STAGE;
        const int knext = min(kt + 1, KT - 1) * BK;
        bf16x8_t af[2][TM], wf[2][TN];
        auto load_frags = [&](int ks, int buf) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                af[buf][i] = AFORM == OP_KMAJOR
                                 ? *reinterpret_cast<const bf16x8_t*>(cur + a_base + i * 32 * ROW_BYTES + foff[ks])
                                 : tr_frag(cur + a_base + i * 64 + ks * 16 * TLayout<BM>::STRIDE, TLayout<BM>::STRIDE);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                wf[buf][j] = WFORM == OP_KMAJOR
                                 ? *reinterpret_cast<const bf16x8_t*>(cur + w_base + j * 32 * ROW_BYTES + foff[ks])
                                 : tr_frag(cur + w_base + j * 64 + ks * 16 * TLayout<BN>::STRIDE, TLayout<BN>::STRIDE);
        };
        load_frags(0, 0);
        la.fetch(knext);
        lw.fetch(knext);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (ks < 3) {
                load_frags(ks + 1, (ks + 1) & 1);
            } else {
                la.store(nxt);
                lw.store(nxt + A_BYTES);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ks & 1][j], af[ks & 1][i], acc[j][i], 0, 0, 0);
        }
        // One pipeline description for the whole body, in issue order: the step-0
        // fragments; then per step 2 MFMAs per fragment read of the next step (the
        // tile's global loads ride along in step 0); in the last step one LDS store
        // of the next tile per MFMA.
        constexpr int AR = AFORM == OP_KMAJOR ? 1 : 2, WR = WFORM == OP_KMAJOR ? 1 : 2;   // LDS reads per fragment
        __builtin_amdgcn_sched_group_barrier(M_DS_RD, TM * AR + TN * WR, 0);
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) {
#pragma unroll
            for (int i = 0; i < NFRAG; ++i) {
                __builtin_amdgcn_sched_group_barrier(M_MFMA, NMFMA / NFRAG, 0);
                if (i < TM) __builtin_amdgcn_sched_group_barrier(M_DS_RD, AR, 0);
                else __builtin_amdgcn_sched_group_barrier(M_DS_RD, WR, 0);
                if (ks == 0) __builtin_amdgcn_sched_group_barrier(M_VMEM_RD, (LA_LOADS + LW_LOADS + NFRAG - 1) / NFRAG, 0);
            }
            if (NMFMA % NFRAG) __builtin_amdgcn_sched_group_barrier(M_MFMA, NMFMA % NFRAG, 0);
        }
#pragma unroll
        for (int i = 0; i < NMFMA; ++i) {
            __builtin_amdgcn_sched_group_barrier(M_MFMA, 1, 0);
            __builtin_amdgcn_sched_group_barrier(M_DS_WR, (LA_STORES + LW_STORES + NMFMA - 1) / NMFMA, 0);
        }
        __syncthreads();
    }

    gemm_epilogue<EPI, TM, TN>(p, acc, m0 + wm * (BM / 2), SWIGLU ? n0 + wn * (WN / 2) : n0 + wn * WN, l32, half);
}

// Epilogue through LDS (used by the LDS-DMA kernel, whose LDS is idle once the k-loop ends).
// Written straight from the accumulators a store instruction covers 32 rows x 16 or 32 bytes:
// 2 M write requests of 16 bytes per round of 256 tiles, which the L2 takes ~9 us to absorb
// (a fifth of the ViT-H first MLP projection).  Here the values (bias, GELU, SwiGLU applied)
// are first laid out in LDS as the output tile, RP rows at a time (row stride + 16 bytes: a
// wave's 32 rows spread over the banks), and then written with 16 bytes per lane, consecutive
// lanes on consecutive bytes of a row: whole 128-byte lines.  The residual is read the same way.
// acc[j][i]: 16x16 tile (n tile j, m tile i) of a wave whose first tile row is wrow0 and first output
// column inside the tile wcol0; a lane holds row lane & 15 and the four columns 4 (lane >> 4) ..
template <int EPI, int TM, int TN, int BM, int BN_OUT, int NT, int LDS_BYTES>
__device__ __forceinline__ void gemm_epilogue_staged(const GemmDev& p, f32x4_t (&acc)[TN][TM], unsigned char* smem,
                                                     int m0, int n0, int wrow0, int wcol0, int lane) {
    constexpr bool SWIGLU = (EPI == EPI_SWIGLU_BF16);
    constexpr bool F32OUT = (EPI == EPI_RESID_F32 || EPI == EPI_F32);
    constexpr int ESZ = F32OUT ? 4 : 2;
    constexpr int ROWB = BN_OUT * ESZ, STRIDE = ROWB + 16;
    constexpr int BIAS_BYTES = BN_OUT * 2;                // the tile's bias values, staged behind the passes
    constexpr int ROOM = LDS_BYTES - BIAS_BYTES;
    constexpr int RP = BM * STRIDE <= ROOM ? BM : (BM / 2) * STRIDE <= ROOM ? BM / 2 : BM / 4;
    static_assert(RP * STRIDE <= ROOM && RP % 32 == 0 && BIAS_BYTES % 16 == 0, "a pass of the output tile fits the LDS");
    const bf16_t* sbias = reinterpret_cast<const bf16_t*>(smem + ROOM);
    constexpr int TNO = SWIGLU ? TN / 2 : TN;
    constexpr int CPR = ROWB / 16, CHUNKS = RP * CPR;     // 16-byte chunks per row / per pass
    // the values of 4 consecutive columns (register group g of tile (j, i))
    const int l16 = lane & 15, quarter = lane >> 4;
    auto values = [&](int i, int j, float (&v)[4]) {
        const int nl = wcol0 + j * 16 + quarter * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (SWIGLU) {
                const float gv = acc[j][i][e], uv = acc[j + TN / 2][i][e];
                v[e] = gv * __builtin_amdgcn_rcpf(1.0f + __expf(-gv)) * uv;
            } else {
                v[e] = acc[j][i][e];
            }
        }
        if (!SWIGLU && p.bias) {
            const uint2 b = *reinterpret_cast<const uint2*>(sbias + nl);
            v[0] += bf_lo(b.x); v[1] += bf_hi(b.x); v[2] += bf_lo(b.y); v[3] += bf_hi(b.y);
        }
        if (EPI == EPI_GELU_BF16) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = gelu_erf(v[e]);
        }
    };
    __syncthreads();   // every wave is done with the operand stages, no load is in flight
    // Barriers from here on order LDS traffic only (lgkmcnt): a __syncthreads() would also wait
    // for the global stores of a pass to be acknowledged, several microseconds per pass with the
    // matrix pipes idle.
    constexpr int WAIT_LGKM0 = 15 | (7 << 4) | (0 << 8) | (3 << 14);   // vmcnt 63, expcnt 7, lgkmcnt 0
    auto lds_barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // The tile's bias values go through LDS once: fetched from global memory where they are used,
    // every one of a lane's TM x TN x 4 little loads was waited for in turn (a cache round trip each).
    if (!SWIGLU && p.bias) {
        for (int c = threadIdx.x; c < BN_OUT / 8; c += NT) {
            const int n = n0 + c * 8;
            const u32x4_t b = n < p.N ? *reinterpret_cast<const u32x4_t*>(p.bias + n) : u32x4_t{0, 0, 0, 0};   // N % 8 == 0
            *reinterpret_cast<u32x4_t*>(smem + ROOM + c * 16) = b;
        }
        lds_barrier();
    }
    // bf16 outputs: every wave computes and packs all of its values first (the activation
    // functions are the expensive part and must not be serialised by the passes below)
    uint2 pk[F32OUT ? 1 : TM][F32OUT ? 1 : TNO];
    if (!F32OUT) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TNO; ++j) {
                float v[4];
                values(i, j, v);
                pk[F32OUT ? 0 : i][F32OUT ? 0 : j] = make_uint2(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]));
            }
    }
    // A thread's residual loads of a pass are all issued before the first is used (one after the
    // other, each waited for, they cost a memory round trip per 16 bytes), the first batch before
    // the pass's LDS writes, so that its latency runs under those.
    constexpr int ITER = (CHUNKS + NT - 1) / NT;
    constexpr int SB = ITER > 6 ? (ITER + 1) / 2 : ITER;     // residual pieces in flight per thread
    auto chunk_pos = [&](int pass, int it, int* row, int* ch, int* m, int* n) {
        const int c = threadIdx.x + it * NT;
        *row = c / CPR;
        *ch = c % CPR;
        *m = m0 + pass * RP + *row;
        *n = n0 + *ch * (16 / ESZ);
        return c < CHUNKS && *m < p.M && *n < p.N;
    };
    float4 rr[EPI == EPI_RESID_F32 ? SB : 1];
    auto load_resid = [&](int pass, int it0) {
#pragma unroll
        for (int it = it0; it < it0 + SB && it < ITER; ++it) {
            int row, ch, m, n;
            const bool ok = chunk_pos(pass, it, &row, &ch, &m, &n);
            rr[it - it0] = ok ? *reinterpret_cast<const float4*>(p.R + (size_t)m * p.ldr + n) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
#pragma unroll
    for (int pass = 0; pass < BM / RP; ++pass) {
        if (EPI == EPI_RESID_F32) load_resid(pass, 0);
        if (pass) lds_barrier();     // the previous pass has been read out
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int r = wrow0 + i * 16;                 // wave-uniform
            if (r / RP != pass) continue;
            unsigned char* rowp = smem + (r - pass * RP + l16) * STRIDE;
#pragma unroll
            for (int j = 0; j < TNO; ++j) {
                const int nl = wcol0 + j * 16 + quarter * 4;
                if (F32OUT) {
                    float v[4];
                    values(i, j, v);
                    *reinterpret_cast<float4*>(rowp + nl * 4) = make_float4(v[0], v[1], v[2], v[3]);
                } else {
                    *reinterpret_cast<uint2*>(rowp + nl * 2) = pk[F32OUT ? 0 : i][F32OUT ? 0 : j];
                }
            }
        }
        lds_barrier();
#pragma unroll
        for (int it0 = 0; it0 < ITER; it0 += SB) {
            if (EPI == EPI_RESID_F32 && it0) load_resid(pass, it0);
#pragma unroll
            for (int it = it0; it < it0 + SB && it < ITER; ++it) {
                int row, ch, m, n;
                if (chunk_pos(pass, it, &row, &ch, &m, &n)) {
                    u32x4_t v = *reinterpret_cast<const u32x4_t*>(smem + row * STRIDE + ch * 16);
                    if (EPI == EPI_RESID_F32) {
                        const float4 a = __builtin_bit_cast(float4, v);
                        const float4 r = rr[it - it0];
                        v = __builtin_bit_cast(u32x4_t, make_float4(a.x + r.x, a.y + r.y, a.z + r.z, a.w + r.w));
                    }
                    *reinterpret_cast<u32x4_t*>(static_cast<unsigned char*>(p.C) + ((size_t)m * p.ldc + n) * ESZ) = v;
                }
            }
        }
    }
}

// ---- LDS-DMA kernel ----------------------------------------------------------------------------
// Global loads write LDS directly (global_load_lds_dwordx4): no staging registers and no
// ds_write instructions.  Measured on MI355X, LDS writes issued by the waves run at about
// 75 bytes/clk per CU and serialise with the fragment reads (215 bytes/clk), so a 256x256x64
// tile costs ~870 + ~900 LDS cycles against 2048 MFMA cycles; the DMA writes overlap the reads.
// A wave instruction lands 64 lanes x 16 bytes contiguously, so the XOR swizzle of the 16-byte
// pieces is applied on the global side (which piece a lane fetches, OpTile); a contraction-contiguous
// operand gets the LDS image the register-staged kernel builds, a row-contiguous one lies as in memory
// (LDS row = contraction index) and is read with the transposing LDS read.
//
// What bounds it is the power of the matrix pipes on operands that toggle (the clock falls to 1.8-2.0 GHz) and what
// keeps them from issuing.  Three things about the loop follow from that, us on random operands (before -> after all
// three; 8192^3 780 with two stages and the compiler's order on zeros, 998 on random operands):
//   8192 x 8192 x 8192 998 -> 755      2048 x 22016 x 4096 336 -> 289     4096 x 10240 x 8192 514 -> 462
//   2048 x 12288 x 4096 196 -> 162     16384 x 1280 x 5120 175 -> 164     16384 x 3840 x 1280 158 -> 141
//   dW 22016 x 4096 x 16384 2640 -> 2400   dX 16384 x 4096 x 22016 2419 -> 2149   dX 16384 x 11008 x 4096 1234 -> 1073
// * v_mfma_f32_16x16x32 instead of 32x32x16.  Both take 1024 flop per cycle and SIMD, but an instruction of the former
//   goes 32 deep, so each accumulator is read and written half as often: MFMAs alone on N(0,1) x N(0,0.02)
//   operands run at 2.05 PFLOP/s against 1.64-1.8 (on zeros both at 2.45).
// * Loads that miss the L2 take more than a k-tile's 1.0-1.4 us under load, and two stages leave a load one k-tile at
//   most.  RING5: five slots of one operand's tile, i.e. two k-tiles and ONE operand of the k-tile after; which one
//   alternates over the output's tiles like the colours of a chess board.  Every row of A (of W) is used by
//   neighbouring work-groups of both colours at the same time, so half of its users fetch it two k-tiles ahead and the
//   others, one k-tile ahead, find it in the L2.  (8192^3 with the compiler's order 986 -> 868; the 256x320
//   tile has no room for a fifth slot.)  The 128x256 tile has three whole stages: 2048 x 4096 x 11008 229 -> 183.
// * The order of MFMAs, fragment reads and loads is fixed by hand (sched_barrier after every MFMA).  With scheduling
//   hints the compiler read fragments just before their use, and it waits for ALL reads in flight
//   (s_waitcnt lgkmcnt(0)) once LDS-DMA loads are about: five such waits per k-tile, each right behind a read.
//
// The only barrier of a tile sits before its LAST part: by then a wave
// has read all its fragments of the tile (the last part's are in registers) and its loads of the
// next tile have landed, so after the barrier the next tile is
// readable and this one's slots are free.  The last part then runs with the first fragments of the
// next tile being read under its MFMAs: nothing that follows the barrier waits on memory.
// The loads of a tile are spread over three parts: issued in one burst they fill the address unit's queue and stall
// the wave's MFMAs behind them (253 -> 231 us on the gate/up shape with zero operands).
// The compiler does not order these loads against later LDS reads; the kernel waits with
// explicit vmcnt/lgkmcnt counts and uses a bare s_barrier (the fence of __syncthreads() is
// what the counts replace).
// (Four waves of 128x128 instead of eight of 128x64, a third less LDS traffic: 5-10 % slower, one wave per SIMD
// hides nothing.)

template <int BM, int BN, int EPI, int AFORM, int WFORM, int WAVES, int WM, int NST>
__global__ __launch_bounds__(WAVES * 64, WAVES == 4 ? 2 : 1) void gemm_dma_kernel(GemmDev p) {
    typedef OpTile16<BM, AFORM> TA;
    typedef OpTile16<BN, WFORM> TW;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int WNC = WAVES / WM;              // wave grid: WM (m) x WNC (n)
    constexpr int WMR = BM / WM, WN = BN / WNC;  // tile rows of A / of W per wave
    constexpr int TM = WMR / 16, TN = WN / 16;   // 16x16 tiles per wave
    static_assert(WMR % 32 == 0 && WN % 32 == 0, "whole halves of MFMA tiles per wave");
    constexpr int A_BYTES = BM * ROW_BYTES, STAGE = (BM + BN) * ROW_BYTES;
    constexpr bool SWIGLU = (EPI == EPI_SWIGLU_BF16);
    constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;
    // 1 KiB load blocks (8 tile rows each) per wave and tile, A's and W's
    constexpr int NA = BM / 8 / WAVES, NW = BN / 8 / WAVES, NI = NA + NW;
    static_assert(BM / 8 % WAVES == 0 && BN / 8 % WAVES == 0, "whole load blocks per wave");
    static_assert(!SWIGLU || (TN % 2 == 0), "gate and up tiles pair up inside a wave");
    constexpr bool RING5 = NST == 5;
    constexpr int SLOT = RING5 ? (BM > BN ? BM : BN) * ROW_BYTES : STAGE;
    constexpr int LDS_BYTES = NST * SLOT;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WM, wn = wave / WM;

    int pid = xcd_remap(blockIdx.x, gridDim.x);
    constexpr int GM = 8;
    const int group = GM * p.tilesN;
    const int first_m = (pid / group) * GM;
    const int gm = min(p.tilesM - first_m, GM);
    const int tm = first_m + (pid % group) % gm;
    const int tn = (pid % group) / gm;
    const int m0 = tm * BM, n0 = tn * BN_OUT;

    // Loads: lane l of a 1 KiB block lands at its 16 bytes l and fetches the piece that the swizzle puts there; its
    // address is a base that is uniform in the wave plus a 32-bit lane offset inside the tile's rows.  The operands of
    // a tile are fetched in the order first, second: RING5 alternates it between neighbouring tiles of the output.
    const bool w_first = RING5 && ((tm ^ tn) & 1);
    constexpr int NMAX = NA > NW ? NA : NW;
    [[maybe_unused]] constexpr int NMIN = NA < NW ? NA : NW;
    const int n_first = w_first ? NW : NA, n_second = NI - n_first;
    const bf16_t* const a_src = p.A + (AFORM == OP_KMAJOR ? (size_t)m0 * p.lda : (size_t)m0);
    // SwiGLU: the first half of a wave's W rows are gate rows, the second half the matching up rows, N further on; a
    // wave loads one half of such a group
    static_assert(!SWIGLU || NW * 8 == WN / 2, "gate or up rows per wave");
    const bool up = SWIGLU && (wave & 1);
    const bf16_t* const w_src = p.W + (WFORM == OP_KMAJOR ? (size_t)(n0 + (up ? p.N : 0)) * p.ldw : (size_t)n0);
    const size_t a_step = AFORM == OP_KMAJOR ? BK : (size_t)BK * p.lda, w_step = WFORM == OP_KMAJOR ? BK : (size_t)BK * p.ldw;
    // byte offset of the lane's piece of the wave's block i
    auto lane_offset = [&](bool is_w, int i) -> uint32_t {
        int row, k;
        if (is_w) {
            TW::piece((wave * NW + i) * 1024 + lane * 16, &row, &k);
            if (SWIGLU) row = row / WN * (WN / 2) + row % (WN / 2);
            row = min(row, p.N - n0 - (WFORM == OP_KMAJOR ? 1 : 8));
            return 2 * (WFORM == OP_KMAJOR ? (uint32_t)row * p.ldw + k : (uint32_t)k * p.ldw + row);
        }
        TA::piece((wave * NA + i) * 1024 + lane * 16, &row, &k);
        row = min(row, p.M - m0 - (AFORM == OP_KMAJOR ? 1 : 8));
        return 2 * (AFORM == OP_KMAJOR ? (uint32_t)row * p.lda + k : (uint32_t)k * p.lda + row);
    };
    uint32_t off1[NMAX], off2[NMAX];     // of the first and the second operand
#pragma unroll
    for (int i = 0; i < NMAX; ++i) {
        off1[i] = w_first ? lane_offset(true, min(i, NW - 1)) : lane_offset(false, min(i, NA - 1));
        off2[i] = w_first ? lane_offset(false, min(i, NA - 1)) : lane_offset(true, min(i, NW - 1));
    }
    const bf16_t *const src1 = w_first ? w_src : a_src, *const src2 = w_first ? a_src : w_src;
    const size_t step1 = w_first ? w_step : a_step, step2 = w_first ? a_step : w_step;
    const int KT = p.K / BK;
    // (The builtin's address-space-qualified parameters do not type-check in the host pass
    // of a template, which would silently drop the kernel's host stub: device pass only.)
#if defined(__HIP_DEVICE_COMPILE__)
#define SP_DMA(src, step, off, n, tile, lds, i)                                                                \
    if ((i) < NMIN || (i) < (n))                                                                               \
        __builtin_amdgcn_global_load_lds(reinterpret_cast<const unsigned char*>((src) + min((tile), KT - 1) * (step)) + (off)[i], \
                                         (lds_void_ptr)((lds) + (wave * (n) + (i)) * 1024), 16, 0, 0);
#else
#define SP_DMA(src, step, off, n, tile, lds, i) ((void)(src), (void)(step), (void)(off), (void)(n), (void)(lds), (void)(tile));
#endif
    // load l of a tile's first / second operand
#define SP_LOAD1(tile, lds, l) SP_DMA(src1, step1, off1, n_first, tile, lds, l)
#define SP_LOAD2(tile, lds, l) SP_DMA(src2, step2, off2, n_second, tile, lds, l)

    f32x4_t acc[TN][TM];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[j][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    int abase[TM], wbase[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) abase[i] = TA::frag_base(wm * TM + i, lane);
#pragma unroll
    for (int j = 0; j < TN; ++j) wbase[j] = TW::frag_base(wn * TN + j, lane);

    // A 32-deep k-step is worked in NP parts: all fragments of one operand (X, the one with fewer) against a part of
    // the other's (Y), so that besides a part's NX + NY fragments only the next part's are in registers.
    constexpr bool X_IS_W = TN <= TM;
    constexpr int NP = TM * TN > 32 ? 5 : 2, NPT = 2 * NP;           // parts per k-step, per tile
    constexpr int NX = X_IS_W ? TN : TM, NY = (X_IS_W ? TM : TN) / NP, NMFMA = NX * NY;
    static_assert((X_IS_W ? TM : TN) % NP == 0 && NX + NY < NMFMA, "equal parts, a read behind each MFMA but the first");
    bf16x8_t fx[2][NX], fy[2][NY];
    auto load_x = [&](const unsigned char* ta, const unsigned char* tw, int ks, int x) {
        if constexpr (X_IS_W) fx[ks][x] = TW::frag(tw, wbase[x], ks, lane); else fx[ks][x] = TA::frag(ta, abase[x], ks, lane);
    };
    auto load_y = [&](const unsigned char* ta, const unsigned char* tw, int part, int y) {
        const int ks = part / NP, i = part % NP * NY + y;
        if constexpr (X_IS_W) fy[part & 1][y] = TA::frag(ta, abase[i], ks, lane); else fy[part & 1][y] = TW::frag(tw, wbase[i], ks, lane);
    };
    // read r of those that bring the operands of part `part` (with a new k-step its X too)
    auto load_part = [&](const unsigned char* ta, const unsigned char* tw, int part, int r) {
        const int nx = part % NP == 0 ? NX : 0;
        if (r < nx) load_x(ta, tw, part / NP, r);
        else if (r < nx + NY) load_y(ta, tw, part, r - nx);
    };
    auto mfma = [&](int part, int q) {
        const int ks = part / NP, x = q % NX, y = q / NX, i = part % NP * NY + y;
        if constexpr (X_IS_W) acc[x][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx[ks][x], fy[part & 1][y], acc[x][i], 0, 0, 0);
        else acc[i][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fy[part & 1][y], fx[ks][x], acc[i][x], 0, 0, 0);
    };
    auto wg_barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // One part: its MFMAs one by one, behind them the reads of the next part's operands and loads of later tiles; the
    // order is fixed here.  The first MFMA stands before the reads because the compiler waits for all reads in flight
    // in front of it.  SP_RIDE: load l of n goes out with MFMA (2 l + 1) NMFMA / 2 n.
#define SP_PART(part, ta, tw, ISSUE)                                                                           \
    _Pragma("unroll") for (int q_ = 0; q_ < NMFMA; ++q_) {                                                     \
        if (q_) load_part(ta, tw, ((part) + 1) % NPT, q_ - 1);                                                 \
        ISSUE(q_)                                                                                              \
        mfma(part, q_);                                                                                        \
        __builtin_amdgcn_sched_barrier(0);                                                                     \
    }
#define SP_RIDE(q, l0, n, LOAD)                                                                                \
    _Pragma("unroll") for (int l_ = 0; l_ < (n); ++l_)                                                         \
        if ((2 * l_ + 1) * NMFMA / (2 * (n) + ((n) == 0)) == (q)) { [[maybe_unused]] const int i_ = (l0) + l_; LOAD(i_) }
    if constexpr (RING5) {
        auto wrap = [](int s) { return s >= 5 ? s - 5 : s; };
        auto slot = [&](int s) { return smem + s * SLOT; };
#pragma unroll
        for (int i = 0; i < NMAX; ++i) { SP_LOAD1(0, slot(0), i) }
#pragma unroll
        for (int i = 0; i < NMAX; ++i) { SP_LOAD2(0, slot(1), i) }
#pragma unroll
        for (int i = 0; i < NMAX; ++i) { SP_LOAD1(1, slot(2), i) }
#pragma unroll
        for (int i = 0; i < NMAX; ++i) { SP_LOAD2(1, slot(3), i) }
        __builtin_amdgcn_s_waitcnt(sp_waitcnt(NI, 15));                   // tile 0
        wg_barrier();
        int s0 = 0;                                                       // slot of tile kt's first operand
#pragma unroll
        for (int r = 0; r < NX + NY; ++r) load_part(slot(w_first), slot(!w_first), 0, r);
        for (int kt = 0; kt < KT; ++kt) {
            const int s1 = wrap(s0 + 1), s2 = wrap(s0 + 2), s3 = wrap(s0 + 3);
            [[maybe_unused]] const int s4 = wrap(s0 + 4);
            const unsigned char *ca = slot(w_first ? s1 : s0), *cw = slot(w_first ? s0 : s1);
            const unsigned char *na = slot(w_first ? s3 : s2), *nw = slot(w_first ? s2 : s3);
            __builtin_amdgcn_sched_barrier(0);
            // the first operand of tile kt + 2, to the slot that tile kt - 1 left with its second
            constexpr int H = (NMAX + 1) / 2;
#define SP_L1(i) SP_LOAD1(kt + 2, slot(s4), i)
#define SP_L2(i) SP_LOAD2(kt + 2, slot(s0), i)
#define SP_ISSUE(q) if (part == 0) { SP_RIDE(q, 0, H, SP_L1) } else if (part == 1) { SP_RIDE(q, H, NMAX - H, SP_L1) }
#define SP_ISSUE_LAST(q) SP_RIDE(q, 0, NMAX, SP_L2)
#pragma unroll
            for (int part = 0; part < NPT - 1; ++part) { SP_PART(part, ca, cw, SP_ISSUE) }
            // This wave's reads of tile kt are complete and its loads of tile kt + 1 have landed (only the first
            // operand of tile kt + 2 may be in flight); after the barrier that holds for every wave: the next tile is
            // readable, this one's slots may be refilled.
            if (NA == NW || !w_first) __builtin_amdgcn_s_waitcnt(sp_waitcnt(NA, 0));
            else __builtin_amdgcn_s_waitcnt(sp_waitcnt(NW, 0));
            wg_barrier();
            SP_PART(NPT - 1, na, nw, SP_ISSUE_LAST)
            s0 = s2;
#undef SP_L1
#undef SP_L2
#undef SP_ISSUE
#undef SP_ISSUE_LAST
        }
    } else {
        constexpr int LATER = (NST - 2) * NI;      // loads of later tiles that may be in flight when a tile is needed
        // of a tile's loads, those with the last part of the tile NST before it, and with each of the next LP parts
        constexpr int N_AFTER = (3 * NI + 7) / 8, LP = NP == 2 ? 2 : 3, PER = (NI - N_AFTER + LP - 1) / LP;
        static_assert(LATER + N_AFTER < 64, "fits the load counter");
#define SP_LOAD(tile, stage, i)                                                                                \
        if ((i) < NA) { SP_LOAD1(tile, smem + (stage) * STAGE, i) } else { SP_LOAD2(tile, smem + (stage) * STAGE + A_BYTES, (i) - NA) }
#pragma unroll
        for (int t = 0; t < NST - 1; ++t)
#pragma unroll
            for (int i = 0; i < NI; ++i) { SP_LOAD(t, t, i) }
#pragma unroll
        for (int i = 0; i < N_AFTER; ++i) { SP_LOAD(NST - 1, NST - 1, i) }
        __builtin_amdgcn_s_waitcnt(sp_waitcnt(LATER + N_AFTER, 15));      // this thread's loads of tile 0 have landed
        wg_barrier();
#pragma unroll
        for (int r = 0; r < NX + NY; ++r) load_part(smem, smem + A_BYTES, 0, r);
        int st = 0;                                        // stage of tile kt
        for (int kt = 0; kt < KT; ++kt) {
            const int st1 = st + 1 == NST ? 0 : st + 1;
            [[maybe_unused]] const int st_last = st == 0 ? NST - 1 : st - 1;
            const unsigned char *cur = smem + st * STAGE, *nxt = smem + st1 * STAGE;
            __builtin_amdgcn_sched_barrier(0);
            // the rest of tile kt + NST - 1's loads (its first N_AFTER went out after the last barrier)
#define SP_L(i) SP_LOAD(kt + NST - 1, st_last, i)
#define SP_LN(i) SP_LOAD(kt + NST, st, i)
#define SP_ISSUE(q)                                                                                            \
            if (part < LP) {                                                                                   \
                const int l0_ = N_AFTER + part * PER, n_ = NI - l0_ < PER ? (NI - l0_ > 0 ? NI - l0_ : 0) : PER; \
                SP_RIDE(q, l0_, n_, SP_L)                                                                      \
            }
#define SP_ISSUE_LAST(q) SP_RIDE(q, 0, N_AFTER, SP_LN)
#pragma unroll
            for (int part = 0; part < NPT - 1; ++part) { SP_PART(part, cur, cur + A_BYTES, SP_ISSUE) }
            // as above: the loads of tile kt + 1 were issued NST - 1 tiles ago
            __builtin_amdgcn_s_waitcnt(sp_waitcnt(LATER, 0));
            wg_barrier();
            SP_PART(NPT - 1, nxt, nxt + A_BYTES, SP_ISSUE_LAST)
            st = st1;
#undef SP_L
#undef SP_LN
#undef SP_LOAD
#undef SP_ISSUE
#undef SP_ISSUE_LAST
        }
    }
#undef SP_PART
#undef SP_RIDE
    __builtin_amdgcn_s_waitcnt(sp_waitcnt(0, 0));   // drain the tail's idle loads
    gemm_epilogue_staged<EPI, TM, TN, BM, BN_OUT, WAVES * 64, LDS_BYTES>(p, acc, smem, m0, n0, wm * WMR,
                                                                         SWIGLU ? wn * (WN / 2) : wn * WN, lane);
#undef SP_DMA
#undef SP_LOAD1
#undef SP_LOAD2
}

template <int BM, int BN, int EPI, int AFORM, int WFORM, int WAVES, int WM, int NST = 2>
hipError_t launch_dma(hipStream_t st, const GemmArgs& g) {
    constexpr int LDS = NST == 5 ? 5 * std::max(BM, BN) * ROW_BYTES : NST * (BM + BN) * ROW_BYTES;
    static_assert(LDS <= 160 * 1024, "the stages fit a CU's LDS");
    constexpr int BN_OUT = (EPI == EPI_SWIGLU_BF16) ? BN / 2 : BN;
    static LdsLimitOnce lds_limit;
    hipError_t e = lds_limit.set(reinterpret_cast<const void*>(gemm_dma_kernel<BM, BN, EPI, AFORM, WFORM, WAVES, WM, NST>), LDS);
    if (e != hipSuccess) return e;
    GemmDev d;
    d.A = g.A; d.W = g.W; d.C = g.C; d.R = g.R; d.bias = g.bias;
    d.lda = g.lda; d.ldw = g.ldw; d.ldc = g.ldc; d.ldr = g.ldr;
    d.M = g.M; d.N = g.N; d.K = g.K;
    d.tilesM = (g.M + BM - 1) / BM;
    d.tilesN = (g.N + BN_OUT - 1) / BN_OUT;
    gemm_dma_kernel<BM, BN, EPI, AFORM, WFORM, WAVES, WM, NST><<<d.tilesM * d.tilesN, WAVES * 64, LDS, st>>>(d);
    return hipGetLastError();
}

template <int BM, int BN, int EPI, int AFORM, int WFORM, int WAVES>
hipError_t launch_one(hipStream_t st, const GemmArgs& g) {
    constexpr int LDS = 2 * ((AFORM == OP_KMAJOR ? BM * ROW_BYTES : TLayout<BM>::BYTES) +
                             (WFORM == OP_KMAJOR ? BN * ROW_BYTES : TLayout<BN>::BYTES));
    constexpr int BN_OUT = (EPI == EPI_SWIGLU_BF16) ? BN / 2 : BN;
    static LdsLimitOnce lds_limit;   // one per instantiation
    auto kern = gemm_kernel<BM, BN, EPI, AFORM, WFORM, WAVES>;
    hipError_t e = lds_limit.set(reinterpret_cast<const void*>(kern), LDS);
    if (e != hipSuccess) return e;
    GemmDev d;
    d.A = g.A; d.W = g.W; d.C = g.C; d.R = g.R; d.bias = g.bias;
    d.lda = g.lda; d.ldw = g.ldw; d.ldc = g.ldc; d.ldr = g.ldr;
    d.M = g.M; d.N = g.N; d.K = g.K;
    d.tilesM = (g.M + BM - 1) / BM;
    d.tilesN = (g.N + BN_OUT - 1) / BN_OUT;
    const int nblocks = d.tilesM * d.tilesN;
    gemm_kernel<BM, BN, EPI, AFORM, WFORM, WAVES><<<nblocks, WAVES * 64, LDS, st>>>(d);
    return hipGetLastError();
}

// Tile ids: register-staged kernel 1 = 128x128, 2 = 128x256 (BM x BN), 3 = 256x256 (4 waves each),
// 4 = 256x256 with 8 waves; LDS-DMA kernel 5 = 256x256 and
// 6 = 128x256 with 8 waves, 7 = 128x128 with 4 waves (two work-groups per CU), 8 = 256x192 with 8
// waves in a 4 x 2 grid (not with the SwiGLU epilogue, which pairs tiles inside a wave); 9 =
// at most 64 activation rows (the small-tile kernel, k_gemm_small.hip; 11, 12, 13 force its 16, 32 and
// 64 row tiles there, 14..20 its tiles for any shape); 10 = 256x320 of the
// LDS-DMA kernel, 4 x 2 waves (not with SwiGLU): N = 1280 is four of its columns, so the ViT-H
// projections back to d_model are one round of 256 work-groups once the ragged rows are cut off.
//
// Choice (shapes only, so a stack's kernels never depend on the streaming window): the chip
// runs 256 work-groups at a time (512 of tile 7), so a launch costs
// ceil(tiles / concurrent) rounds of one tile's time; a tile's time is its area over a measured
// relative efficiency (larger tiles move fewer operand bytes per MFMA).  Take the cheapest.
// (Activation rows are contiguous in A, C and R, so a launch can be cut along M.)
// The efficiencies, like the rate that turns a cost into us in resolve_gemm and the one in plan_large's tail, were measured
// on this kernel with two stages everywhere; the tiles with a ring have gained more since than the 256x320 one.  No launch is
// slower for it, but on 37 shapes the choice is 3.2 % off the best tile now (3260 x 896 x 2944 50.8 us on 96x64 tiles, 34.5
// on 128x128; 4218 x 320 x 1152 14.5 and 11.7).
struct TileCost { int id, bm, bn, concurrent; float eff; };
constexpr TileCost kDmaTiles[] = {{5, 256, 256, 256, 1.00f}, {10, 256, 320, 256, 1.02f}, {8, 256, 192, 256, 0.85f},
                                  {6, 128, 256, 256, 0.84f}, {7, 128, 128, 512, 0.70f}};
constexpr TileCost kRegTiles[] = {{4, 256, 256, 256, 1.00f}, {1, 128, 128, 512, 0.66f}};

template <int NC>
int pick_tile(const TileCost (&cand)[NC], int M, int N, int epi, float* cost_out) {
    int best = cand[0].id;
    float best_cost = 0.f;
    for (int c = 0; c < NC; ++c) {
        const TileCost& t = cand[c];
        if ((t.id == 8 || t.id == 10) && epi == EPI_SWIGLU_BF16) continue;
        const int bn_out = (epi == EPI_SWIGLU_BF16) ? t.bn / 2 : t.bn;
        const long tiles = (long)((M + t.bm - 1) / t.bm) * ((N + bn_out - 1) / bn_out);
        // in units of "every CU busy with one tile": the two-per-CU tile fills a CU with two
        float units = (float)(tiles / t.concurrent * (t.concurrent / 256));
        const long rem = tiles % t.concurrent;
        if (rem) units += rem <= 256 ? 1.f : (float)(t.concurrent / 256);
        const float cost = units * (float)(t.bm * t.bn) / t.eff;
        if (c == 0 || cost < best_cost) { best = t.id; best_cost = cost; }   // candidate 0 takes every epilogue
    }
    if (cost_out) *cost_out = best_cost;
    return best;
}

// Operands with the row index contiguous: the estimated time in us of a tile, as fitted to some 300 shapes with the weights
// transposed and 260 with both operands (rows 64..33536, contraction 64..23808, weights not in the caches; rms of the
// LDS-DMA tiles 4-9 %, of the small ones 5-10 %): launch and prologue a, per unit (one
// work-group on every CU) b and c per 1000 of K, w per MB of output; the small tiles also ma and mw per MB of the A and W
// operands, whose first reads so many short work-groups do not hide.  A last round of the two-per-CU tiles that fills one
// half of the slots counts `half` units.  The LDS-DMA tiles and the small ones (16, 18; not with the residual epilogue)
// stand in one table, so that every pair is compared by measured time.  On 171 and 131 other shapes the choice is 0.4 and
// 0.3 % off the best tile on average, at most 15 and 6 %.  (A fit to 79 shapes was 2.0 and 0.9 % off on these, its small tiles
// up to 30 %: 704 x 640 x 4864 23.6 us on 32x32 tiles, 18.3 on 64x64.)
struct TileTime { int id, bm, bn, concurrent; float a, b, c, w, half, ma, mw; };
constexpr TileTime kTimesKR[] = {
    {5, 256, 256, 256, 0.f, 3.884f, 18.928f, 0.279f, 1.f, 0.f, 0.f}, {10, 256, 320, 256, 1.291f, 2.627f, 25.057f, 0.22f, 1.f, 0.f, 0.f},
    {8, 256, 192, 256, 0.f, 4.292f, 15.534f, 0.218f, 1.f, 0.f, 0.f}, {6, 128, 256, 256, 0.097f, 3.491f, 11.553f, 0.194f, 1.f, 0.f, 0.f},
    {7, 128, 128, 512, 2.548f, 0.666f, 6.842f, 0.137f, 1.22f, 0.f, 0.f}, {16, 32, 32, 512, 2.194f, 0.342f, 1.558f, 0.f, 1.02f, 0.499f, 0.228f},
    {18, 64, 64, 256, 1.388f, 2.138f, 2.876f, 0.214f, 1.f, 0.304f, 0.154f}};
constexpr TileTime kTimesRR[] = {
    {5, 256, 256, 256, 3.437f, 3.673f, 20.84f, 0.124f, 1.f, 0.f, 0.f}, {10, 256, 320, 256, 2.236f, 6.602f, 25.206f, 0.095f, 1.f, 0.f, 0.f},
    {8, 256, 192, 256, 2.682f, 3.774f, 16.575f, 0.108f, 1.f, 0.f, 0.f}, {6, 128, 256, 256, 2.93f, 1.453f, 12.001f, 0.151f, 1.f, 0.f, 0.f},
    {7, 128, 128, 512, 3.845f, 0.f, 7.384f, 0.129f, 1.02f, 0.f, 0.f}, {16, 32, 32, 512, 2.101f, 0.166f, 1.673f, 0.328f, 1.16f, 0.717f, 0.028f},
    {18, 64, 64, 256, 1.474f, 2.039f, 2.446f, 0.168f, 1.f, 0.589f, 0.07f}};

int quickest_tile(int epi, int a_form, int M, int N, int K, float* us) {
    const bool small_ok = epi != EPI_RESID_F32;
    const float out_mb = (float)M * (float)N * (epi == EPI_BF16 ? 2e-6f : 4e-6f);
    const float a_mb = (float)M * (float)K * 2e-6f, w_mb = (float)N * (float)K * 2e-6f;
    int best = 0;
    for (const TileTime& t : a_form == OP_KMAJOR ? kTimesKR : kTimesRR) {
        if (t.id >= 14 && !small_ok) continue;
        const long tiles = (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn), rem = tiles % t.concurrent;
        const float units = (float)(tiles / t.concurrent * (t.concurrent / 256)) + (rem == 0 ? 0.f : rem <= 256 ? t.half : (float)(t.concurrent / 256));
        const float c = t.a + units * (t.b + t.c * (float)K * 1e-3f) + t.w * out_mb + t.ma * a_mb + t.mw * w_mb;
        if (!best || c < *us) { best = t.id; *us = c; }
    }
    return best;
}

// Cuts a launch along M where the ragged rows beyond the last multiple of 256 cost less as a launch of their own
// (ViT-H: 16448 tokens = 64 tiles + 64 rows, 1300 tiles = 5.08 rounds of 256).  pick(rows, &cost) -> tile.
template <class PICK, class TAIL>
GemmPlan cut_plan(int M, PICK pick, TAIL tail_pick, float* cost) {
    float whole, c_body, c_tail;
    GemmPlan pl{pick(M, &whole), M, 0};
    const int tail = M % 256, body = M - tail;
    if (tail && body) {
        const int t_body = pick(body, &c_body), t_tail = tail_pick(tail, &c_tail);
        if (c_body + c_tail < 0.97f * whole) {
            pl = GemmPlan{t_body, body, t_tail};
            whole = c_body + c_tail;
        }
    }
    if (cost) *cost = whole;
    return pl;
}

// The large-tile plan of operands with the contraction index contiguous, from M and N alone.
GemmPlan plan_large(int epi, int M, int N, float* cost = nullptr) {
    if (M <= SPK_FEW_ROWS) return GemmPlan{9, M, 0};     // a decode step: nothing of W is re-used, stream it
    auto pick = [&](int m, float* c) { return pick_tile(kDmaTiles, m, N, epi, c); };
    auto tail = [&](int m, float* c) {
        if (m > SPK_FEW_ROWS) return pick(m, c);
        // the small-tile kernel in the units of pick_tile (a round of 256x256 tiles = 65536):
        // N x K x 2 bytes at ~4.5 TB/s against 256 tiles x 2 x 65536 K flop at ~1.3 PFLOP/s, plus a launch
        *c = 1.13f * (float)N + 6000.f;
        return 9;
    };
    return cut_plan(M, pick, tail, cost);
}

// What a launch with tile = 0 runs, for every operand form: rows [0, body_rows) on `tile`, the others on `tail_tile`
// (tile ids of launch_tile, 9 resolved).  `wide`: the rows of C start on 16 bytes.
GemmPlan resolve_gemm(int epi, bool wide, int a_form, int w_form, int M, int N, int K) {
    const bool kmajor = a_form == OP_KMAJOR && w_form == OP_KMAJOR;
    float small_us, cost;
    if (!kmajor && wide) {
        auto pick = [&](int m, float* c) { return quickest_tile(epi, a_form, m, N, K, c); };
        return cut_plan(M, pick, pick, nullptr);
    }
    const int small_id = spk_small_gemm_tile(epi, a_form, w_form, M, N, K, &small_us);
    GemmPlan pl{0, M, 0};
    if (wide) pl = plan_large(epi, M, N, &cost);
    else pl.tile = pick_tile(kRegTiles, M, N, epi, &cost);
    if (pl.tile == 9) return GemmPlan{small_id, M, 0};
    // Both estimates are fits with 10-18 % error, so the small tiles have to be cheaper by a tenth:
    // over 180 shapes of up to 2560 rows the choice was within 1 % of the better kernel on average
    // (2.1 times as fast as the large tiles alone) and in one of them slower than the large tiles, when those had two stages.
    if (small_id && small_us < 0.9f * (4.5f + cost * (float)K * 4.55e-7f)) return GemmPlan{small_id, M, 0};
    if (pl.tail_tile == 9) pl.tail_tile = spk_small_gemm_tile(epi, a_form, w_form, M - pl.body_rows, N, K, &small_us);
    return pl;
}

// Whether the lane offsets of the LDS-DMA kernel, 32-bit byte offsets from a tile's first row (contraction-contiguous) or
// first contraction index, reach every element of the largest tile.  Views whose rows lie further apart (8.4 M elements
// at 256 rows) or run backwards take the register-staged kernel, which forms 64-bit addresses.
bool lanes_reach(const GemmArgs& g) {
    auto reach = [](int form, int rows, long ld) { return ld >= 0 && (form == OP_KMAJOR ? (rows - 1) * ld + BK : (BK - 1) * ld + rows) <= 1L << 31; };
    return reach(g.a_form, std::min(g.M, 256), g.lda) && reach(g.w_form, std::min(g.N, 320), g.ldw);
}

template <int EPI, int AFORM, int WFORM>
hipError_t launch_tile(hipStream_t st, const GemmArgs& g) {
    constexpr bool KMAJOR = (AFORM == OP_KMAJOR && WFORM == OP_KMAJOR);
    constexpr int NOSWIGLU = EPI == EPI_SWIGLU_BF16 ? EPI_BF16 : EPI;   // tiles 8, 10: a wave's load blocks are no half of gate or up rows
    constexpr size_t CSZ = (EPI == EPI_RESID_F32 || EPI == EPI_F32) ? 4 : 2;
    // the LDS-DMA kernel writes C (and reads R) in 16-byte pieces of a row
    const bool dma = (g.ldc * CSZ) % 16 == 0 && lanes_reach(g);
    int tile = g.tile;
    auto small = [&](int id) { GemmArgs t = g; t.tile = id; return spk_launch_gemm_small(st, EPI, t); };
    if (tile == 9 || (tile >= 11 && tile <= 13)) {
        // few rows: the small-tile kernel with its own choice of tile, or 16, 32, 64 rows per work-group
        if (!KMAJOR || g.M > SPK_FEW_ROWS) return hipErrorInvalidValue;
        float us;
        return small(tile == 9 ? spk_small_gemm_tile(EPI, g.a_form, g.w_form, g.M, g.N, g.K, &us) : tile == 11 ? 14 : tile == 12 ? 16 : 17);
    }
    if (!tile) {
        const GemmPlan pl = resolve_gemm(EPI, dma, AFORM, WFORM, g.M, g.N, g.K);
        tile = pl.tile;
        if (pl.body_rows < g.M) {
            GemmArgs a = g, b = g;
            a.M = pl.body_rows; a.tile = pl.tile;
            b.M = g.M - pl.body_rows; b.tile = pl.tail_tile;
            b.A = AFORM == OP_KMAJOR ? g.A + (size_t)pl.body_rows * g.lda : g.A + pl.body_rows;
            b.C = static_cast<unsigned char*>(g.C) + (size_t)pl.body_rows * g.ldc * CSZ;
            if (g.R) b.R = g.R + (size_t)pl.body_rows * g.ldr;
            hipError_t e = launch_tile<EPI, AFORM, WFORM>(st, a);
            return e != hipSuccess ? e : launch_tile<EPI, AFORM, WFORM>(st, b);
        }
    }
    if (tile >= 14) return small(tile);
    if (!dma && ((tile >= 5 && tile <= 8) || tile == 10)) tile = tile == 6 ? 2 : tile == 7 ? 1 : 4;   // register-staged instead
    switch (tile) {
        case 1: return launch_one<128, 128, EPI, AFORM, WFORM, 4>(st, g);
        case 2: return launch_one<128, 256, EPI, AFORM, WFORM, 4>(st, g);
        case 3: return launch_one<256, 256, EPI, AFORM, WFORM, 4>(st, g);
        case 4: return launch_one<256, 256, EPI, AFORM, WFORM, 8>(st, g);
        case 5: return launch_dma<256, 256, EPI, AFORM, WFORM, 8, 2, 5>(st, g);
        case 6: return launch_dma<128, 256, EPI, AFORM, WFORM, 8, 2, 3>(st, g);
        case 7: return launch_dma<128, 128, EPI, AFORM, WFORM, 4, 2, 5>(st, g);
        case 8: if (EPI != EPI_SWIGLU_BF16) return launch_dma<256, 192, NOSWIGLU, AFORM, WFORM, 8, 4, 5>(st, g); break;
        case 10: if (EPI != EPI_SWIGLU_BF16) return launch_dma<256, 320, NOSWIGLU, AFORM, WFORM, 8, 4>(st, g); break;
    }
    return hipErrorInvalidValue;
}

}  // namespace

GemmPlan spk_gemm_resolve_host(int epi, bool wide, int a_form, int w_form, int M, int N, int K) {
    return resolve_gemm(epi, wide, a_form, w_form, M, N, K);
}

GemmPlan spk_gemm_plan_host(int epi, int a_form, int w_form, int M, int N) {
    if (a_form == OP_KMAJOR && w_form == OP_KMAJOR) return plan_large(epi, M, N);
    return GemmPlan{pick_tile(kRegTiles, M, N, epi, nullptr), M, 0};
}

hipError_t spk_launch_gemm(hipStream_t st, int epi, const GemmArgs& g) {
    if (g.M <= 0 || g.N <= 0) return hipSuccess;
    if (g.K <= 0 || g.K % BK || g.N % 8 || g.lda % 8 || g.ldw % 8 || !g.A || !g.W || !g.C) return hipErrorInvalidValue;
    if (((uintptr_t)g.A | (uintptr_t)g.W | (uintptr_t)g.C | (uintptr_t)g.R | (uintptr_t)g.bias) & 15) return hipErrorInvalidValue;
    if (g.ldc % 4 || (epi == EPI_RESID_F32 && (!g.R || g.ldr % 4))) return hipErrorInvalidValue;
    if (g.a_form == OP_RMAJOR && (g.M < 8 || g.M % 8)) return hipErrorInvalidValue;
    if (g.w_form == OP_RMAJOR && (g.N < 8 || g.N % 8)) return hipErrorInvalidValue;
    const int forms = g.a_form * 2 + g.w_form;
    switch (epi) {
        case EPI_BF16:
            if (forms == 0) return launch_tile<EPI_BF16, OP_KMAJOR, OP_KMAJOR>(st, g);
            if (forms == 1) return launch_tile<EPI_BF16, OP_KMAJOR, OP_RMAJOR>(st, g);
            break;
        case EPI_RESID_F32:
            if (forms == 0) return launch_tile<EPI_RESID_F32, OP_KMAJOR, OP_KMAJOR>(st, g);
            if (forms == 1) return launch_tile<EPI_RESID_F32, OP_KMAJOR, OP_RMAJOR>(st, g);
            break;
        case EPI_GELU_BF16:
            if (forms == 0 && g.bias) return launch_tile<EPI_GELU_BF16, OP_KMAJOR, OP_KMAJOR>(st, g);
            break;
        case EPI_SWIGLU_BF16:
            if (forms == 0 && !g.bias) return launch_tile<EPI_SWIGLU_BF16, OP_KMAJOR, OP_KMAJOR>(st, g);
            break;
        case EPI_F32:
            if (forms == 1) return launch_tile<EPI_F32, OP_KMAJOR, OP_RMAJOR>(st, g);
            if (forms == 3) return launch_tile<EPI_F32, OP_RMAJOR, OP_RMAJOR>(st, g);
            if (forms == 0) return launch_tile<EPI_F32, OP_KMAJOR, OP_KMAJOR>(st, g);
            break;
    }
    return hipErrorInvalidValue;
}
