// GEMM for outputs too small to fill the chip with large tiles, down to the one to 64 rows of a decode
// step or of a ragged tail: C[M,N] = epilogue(sum_k A(m,k) W(n,k)).
//
// The large-tile kernels give one 128x128 tile or more to a work-group: 257 rows of a 1280-wide
// projection are 30 work-groups on 256 CUs, each walking the whole contraction with one k-tile in
// flight.  Here a tile is 16 to 96 rows by 16 to 128 columns and the contraction is split over KG
// groups of waves INSIDE the work-group (no partial sums in memory, no second launch).  Operands come
// in 64-deep k-tiles by LDS-DMA.  Up to 96x64 a group is one wave: its stages are its own, so its loop
// has no barrier, and a stage is refilled as soon as its fragments are in registers.  At 64x128 eight
// waves share the k-tiles of a four-stage ring with one barrier each.  The groups' partial tiles meet
// in LDS and are added in group order (deterministic); the same pass applies the epilogue and writes
// whole rows.
//
// What bounds it: a CU gets 70-80 GB/s of operand tiles through LDS-DMA with ~100 KB in flight (the
// loads that miss the L2 take about 1.5 us and a wave's loads return in order), so a tile costs
// (BM + BN) x 128 bytes per k-tile at that rate, and with few rows the weights themselves at
// 4.5-5.6 TB/s of HBM.  Measured (weights not in any cache; before = the 128x128 tile, at most 64 rows
// the weight-streaming kernel this one replaced), us:
//   257 x {3840, 1280, 5120} x 1280 and 257 x 1280 x 5120   17.1 / 19.4 / 17.7 / 57.8 -> 9.8 / 5.9 / 10.6 / 14.2
//   8 x 12288 x 4096, 8 x 4096 x 4096, 8 x 11008 x 4096 SwiGLU, 8 x 4096 x 11008
//                                                            27.6 / 11.2 / 41.4 / 25.5 -> 21.1 /  8.5 / 32.1 / 21.7
//   64 x 1280 x 5120, 64 x 4096 x 11008                      16.3 / 64.5 ->  9.0 / 31.4
//   512 x 4096 x 4096, 1024 x 2048 x 2048                    62.2 / 26.7 -> 30.6 / 17.0
// (Measured and not kept: groups of four or six waves with 32x32 wave tiles for 64x64 and 96x64, equal;
// eight one-stage groups of one wave, equal.)
#include "sp_gemm.h"

namespace {

template <int BM_, int BN_, int WM_, int WN_, int KG_, int NST_>
struct SmallCfg {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KG = KG_, NST = NST_;
    static constexpr int GW = WM * WN;                 // waves per contraction group
    static constexpr int THREADS = GW * KG * 64;
    static constexpr bool ROW16 = BM == 16;            // v_mfma_f32_16x16x32: a wave's tile is 16 x 16 TN
    static constexpr int TM = ROW16 ? 1 : BM / WM / 32, TN = BN / WN / (ROW16 ? 16 : 32);
    static constexpr int STAGE = (BM + BN) * 128;
    static constexpr int NBLK = STAGE / 1024;          // 1 KiB load instructions per k-tile and group
    static constexpr int NI = (NBLK + GW - 1) / GW;    // per wave (the last may repeat a block)
    static constexpr int CSTR = BN + 4;                // floats per row of a partial tile
    static constexpr int LDS_LOOP = KG * NST * STAGE, LDS_EPI = KG * BM * CSTR * 4;     // stages; all groups' partial tiles
    static constexpr int LDS = LDS_LOOP > LDS_EPI ? LDS_LOOP : LDS_EPI;
    static_assert(!ROW16 || GW == 1);
    static_assert(NI * (NST - 1) < 63 && LDS <= 160 * 1024 && THREADS <= 1024, "fits the counters, the LDS and a work-group");
};

// NACC: accumulator sets, taken in turn by a k-tile's steps and added at the end.  Two with four contraction groups,
// at most SPK_FEW_ROWS rows and an fp32 output: the sums are then as short as with eight groups, which such launches
// always had (relative error of 64 x 8192 x 28672 3.6e-7, with one set 5.1e-7; of a bf16 output the rounding is
// 1.7e-3 either way).  Costs 0 to 0.7 us of a launch.
template <class C, int EPI, int AFORM, int WFORM, int NACC>
__global__ __launch_bounds__(C::THREADS) void gemm_small_kernel(GemmDev p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr bool SWIGLU = (EPI == EPI_SWIGLU_BF16);
    constexpr int BM = C::BM, BN = C::BN, TM = C::TM, TN = C::TN, NI = C::NI, NST = C::NST;
    constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;
    typedef OpTile<BM, AFORM> TA;
    typedef OpTile<BN, WFORM> TW;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave / C::GW, gw = wave % C::GW;
    const int wm = gw % C::WM, wn = gw / C::WM;
    const int l32 = lane & 31, half = lane >> 5;

    // the row tiles of one column block are neighbours on one XCD: its W rows are fetched once
    const int pid = xcd_remap(blockIdx.x, gridDim.x);
    const int m0 = (pid % p.tilesM) * BM, n0 = (pid / p.tilesM) * BN_OUT;

    const int KT = p.K / 64;
    // group g takes the k-tiles g, g + KG, ...: the groups of a work-group read neighbouring pieces of a row
    const int nkt = (KT - grp + C::KG - 1) / C::KG, nmax = (KT + C::KG - 1) / C::KG;
    unsigned char* stages = smem + grp * NST * C::STAGE;

    const bf16_t* src[NI];
    size_t step[NI];             // elements from one of the group's k-tiles to the next
    int dst[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int blk = min(gw + i * C::GW, C::NBLK - 1);      // wave-uniform; a repeated block rewrites the same bytes
        const int off = blk * 1024 + lane * 16;
        int r, k;
        if (blk * 1024 < TA::BYTES) {
            TA::piece(off, &r, &k);
            if (AFORM == OP_KMAJOR) src[i] = p.A + (size_t)min(m0 + r, p.M - 1) * p.lda + k;
            else src[i] = p.A + (size_t)k * p.lda + min(m0 + r, p.M - 8);
            step[i] = AFORM == OP_KMAJOR ? 64 : (size_t)64 * p.lda;
        } else {
            TW::piece(off - TA::BYTES, &r, &k);
            if (WFORM == OP_KMAJOR) {
                int row;
                if (SWIGLU) row = r < BN_OUT ? min(n0 + r, p.N - 1) : p.N + min(n0 + r - BN_OUT, p.N - 1);   // gate rows, then the matching up rows
                else row = min(n0 + r, p.N - 1);
                src[i] = p.W + (size_t)row * p.ldw + k;
            } else {
                src[i] = p.W + (size_t)k * p.ldw + min(n0 + r, p.N - 8);
            }
            step[i] = WFORM == OP_KMAJOR ? 64 : (size_t)64 * p.ldw;
        }
        src[i] += step[i] * grp;
        step[i] *= C::KG;
        dst[i] = blk * 1024;
    }
#if defined(__HIP_DEVICE_COMPILE__)
#define SP_SMALL_ISSUE(kt_)                                                                            \
    do {                                                                                               \
        unsigned char* st_ = stages + ((kt_) % NST) * C::STAGE;                                        \
        _Pragma("unroll") for (int i_ = 0; i_ < NI; ++i_) {                                            \
            __builtin_amdgcn_global_load_lds(src[i_], (lds_void_ptr)(st_ + dst[i_]), 16, 0, 0);        \
            src[i_] += step[i_];                                                                       \
        }                                                                                              \
    } while (0)
#else
#define SP_SMALL_ISSUE(kt_) ((void)src, (void)dst, (void)stages)
#endif

    constexpr int ACC = C::ROW16 ? 4 : 16;             // accumulator registers per tile: ACC / 4 groups of four columns
    typedef float acc_t __attribute__((ext_vector_type(ACC)));
    acc_t sums[NACC][TN][TM];
#pragma unroll
    for (int a = 0; a < NACC; ++a)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int e = 0; e < ACC; ++e) sums[a][j][i][e] = 0.f;
    constexpr int KS = C::ROW16 ? 2 : 4;               // MFMA steps per k-tile
    int abase[TM], wbase[TN];
    if constexpr (C::ROW16) {
        abase[0] = (lane & 15) * 128;
#pragma unroll
        for (int j = 0; j < TN; ++j) wbase[j] = TA::BYTES + (j * 16 + (lane & 15)) * 128;
    } else {
#pragma unroll
        for (int i = 0; i < TM; ++i) abase[i] = TA::frag_base(wm * TM + i, lane);
#pragma unroll
        for (int j = 0; j < TN; ++j) wbase[j] = TA::BYTES + TW::frag_base(wn * TN + j, lane);
    }
    bf16x8_t af[KS][TM], wf[KS][TN];
    auto read_frags = [&](const unsigned char* cur) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if constexpr (C::ROW16) {
                // lane l: row l & 15, contraction indexes 32 ks + 8 (l >> 4) ..
                const int c = ((4 * ks + (lane >> 4)) ^ (((lane & 15) >> 1) & 7)) << 4;
                af[ks][0] = *reinterpret_cast<const bf16x8_t*>(cur + abase[0] + c);
#pragma unroll
                for (int j = 0; j < TN; ++j) wf[ks][j] = *reinterpret_cast<const bf16x8_t*>(cur + wbase[j] + c);
            } else {
#pragma unroll
                for (int i = 0; i < TM; ++i) af[ks][i] = TA::frag(cur, abase[i], ks, lane);
#pragma unroll
                for (int j = 0; j < TN; ++j) wf[ks][j] = TW::frag(cur, wbase[j], ks, lane);
            }
        }
    };
    auto mfmas = [&]() {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    acc_t& s = sums[ks % NACC][j][i];
                    if constexpr (C::ROW16) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ks][j], af[ks][i], s, 0, 0, 0);
                    else s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ks][j], af[ks][i], s, 0, 0, 0);
                }
    };
    constexpr int NMFMA = KS * TM * TN;

    if constexpr (C::GW == 1) {
        // A wave owns the whole tile for every KG-th k-tile: its stages are its own and no barrier is
        // needed.  Once a tile's fragments are in registers its stage is refilled, so NST k-tiles are
        // in flight under the MFMAs.
#pragma unroll
        for (int s = 0; s < NST; ++s)
            if (s < nkt) SP_SMALL_ISSUE(s);
        for (int kt = 0; kt < nkt; ++kt) {
            const int later = nkt - 1 - kt;
            if (later >= NST - 1) __builtin_amdgcn_s_waitcnt(sp_waitcnt(NI * (NST - 1), 15));
            else if (NST > 3 && later >= 2) __builtin_amdgcn_s_waitcnt(sp_waitcnt(NI * 2, 15));
            else if (NST > 2 && later >= 1) __builtin_amdgcn_s_waitcnt(sp_waitcnt(NI, 15));
            else __builtin_amdgcn_s_waitcnt(sp_waitcnt(0, 15));
            asm volatile("" ::: "memory");
            const unsigned char* cur = stages + (kt % NST) * C::STAGE;
            read_frags(cur);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (kt + NST < nkt) SP_SMALL_ISSUE(kt + NST);
            mfmas();
            // the refill's loads ride between the MFMAs: in one burst they would queue at the address
            // unit with the matrix pipe idle
#pragma unroll
            for (int i = 0; i < NMFMA; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x020, (NI + NMFMA - 1) / NMFMA, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
        }
    } else {
#pragma unroll
    for (int s = 0; s < NST - 1; ++s)
        if (s < nkt) SP_SMALL_ISSUE(s);
    for (int kt = 0; kt < nmax; ++kt) {
        // this group's tile kt has landed when at most the later tiles' loads are outstanding
        const int later = nkt - 1 - kt;
        if (later >= NST - 2) __builtin_amdgcn_s_waitcnt(sp_waitcnt(NI * (NST - 2), 0));
        else if (NST > 3 && later == 1) __builtin_amdgcn_s_waitcnt(sp_waitcnt(NI, 0));
        else __builtin_amdgcn_s_waitcnt(sp_waitcnt(0, 0));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();     // ... for every wave, and everyone is done with tile kt - 1
        asm volatile("" ::: "memory");
        if (kt + NST - 1 < nkt) SP_SMALL_ISSUE(kt + NST - 1);
        if (kt < nkt) {
            const unsigned char* cur = stages + (kt % NST) * C::STAGE;
            read_frags(cur);
            mfmas();
            // all of the tile's fragment reads first (left alone the compiler waits for each pair before its MFMA)
            __builtin_amdgcn_sched_group_barrier(0x100, KS * (TM * (AFORM == OP_KMAJOR ? 1 : 2) + TN * (WFORM == OP_KMAJOR ? 1 : 2)), 0);
            __builtin_amdgcn_sched_group_barrier(0x008, NMFMA, 0);
        }
    }
    }
#undef SP_SMALL_ISSUE
    acc_t (&acc)[TN][TM] = sums[0];
    if constexpr (NACC == 2)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[j][i] += sums[1][j][i];
    sp_lds_barrier();     // every load has been waited for, every fragment read is done: the LDS is free

    float* red = reinterpret_cast<float*>(smem);
    // partial tiles, one per group: rows of BN + 4 floats
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g = 0; g < ACC / 4; ++g) {
                // a lane's four registers of a group are four consecutive columns of one row
                const int row = C::ROW16 ? lane & 15 : (wm * TM + i) * 32 + l32;
                const int col = C::ROW16 ? j * 16 + 4 * (lane >> 4) : (wn * TN + j) * 32 + g * 8 + half * 4;
                *reinterpret_cast<float4*>(red + (grp * BM + row) * C::CSTR + col) =
                    make_float4(acc[j][i][g * 4], acc[j][i][g * 4 + 1], acc[j][i][g * 4 + 2], acc[j][i][g * 4 + 3]);
            }
    sp_lds_barrier();

    constexpr int QPR = BN_OUT / 4;       // groups of four columns per row
    for (int q = threadIdx.x; q < BM * QPR; q += C::THREADS) {
        const int r = q / QPR, c = (q % QPR) * 4;
        const int m = m0 + r, n = n0 + c;
        if (m >= p.M || n >= p.N) continue;                    // N % 8 == 0: four columns are inside or outside
        float4 rr;
        if (EPI == EPI_RESID_F32) rr = *reinterpret_cast<const float4*>(p.R + (size_t)m * p.ldr + n);
        uint2 b = make_uint2(0, 0);
        if (!SWIGLU && p.bias) b = *reinterpret_cast<const uint2*>(p.bias + n);
        float v[4] = {0.f, 0.f, 0.f, 0.f}, u[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < C::KG; ++g) {
            const float* row = red + (g * BM + r) * C::CSTR + c;
            const float4 a = *reinterpret_cast<const float4*>(row);
            v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w;
            if (SWIGLU) {
                const float4 w = *reinterpret_cast<const float4*>(row + BN_OUT);
                u[0] += w.x; u[1] += w.y; u[2] += w.z; u[3] += w.w;
            }
        }
        if (SWIGLU) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = v[e] * __builtin_amdgcn_rcpf(1.0f + __expf(-v[e])) * u[e];
        } else if (p.bias) {
            v[0] += bf_lo(b.x); v[1] += bf_hi(b.x); v[2] += bf_lo(b.y); v[3] += bf_hi(b.y);
        }
        if (EPI == EPI_GELU_BF16) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = gelu_erf(v[e]);
        }
        if (EPI == EPI_RESID_F32) { v[0] += rr.x; v[1] += rr.y; v[2] += rr.z; v[3] += rr.w; }
        if (EPI == EPI_RESID_F32 || EPI == EPI_F32)
            *reinterpret_cast<float4*>(static_cast<float*>(p.C) + (size_t)m * p.ldc + n) = make_float4(v[0], v[1], v[2], v[3]);
        else
            *reinterpret_cast<uint2*>(static_cast<bf16_t*>(p.C) + (size_t)m * p.ldc + n) =
                make_uint2(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]));
    }
}

template <class C, int EPI, int AFORM, int WFORM, int NACC>
hipError_t launch_acc(hipStream_t st, const GemmArgs& g) {
    constexpr int BN_OUT = (EPI == EPI_SWIGLU_BF16) ? C::BN / 2 : C::BN;
    static LdsLimitOnce lds_limit;
    auto kern = gemm_small_kernel<C, EPI, AFORM, WFORM, NACC>;
    hipError_t e = lds_limit.set(reinterpret_cast<const void*>(kern), C::LDS);
    if (e != hipSuccess) return e;
    GemmDev d;
    d.A = g.A; d.W = g.W; d.C = g.C; d.R = g.R; d.bias = g.bias;
    d.lda = g.lda; d.ldw = g.ldw; d.ldc = g.ldc; d.ldr = g.ldr;
    d.M = g.M; d.N = g.N; d.K = g.K;
    d.tilesM = (g.M + C::BM - 1) / C::BM;
    d.tilesN = (g.N + BN_OUT - 1) / BN_OUT;
    gemm_small_kernel<C, EPI, AFORM, WFORM, NACC><<<d.tilesM * d.tilesN, C::THREADS, C::LDS, st>>>(d);
    return hipGetLastError();
}

template <class C, int EPI, int AFORM, int WFORM>
hipError_t launch_small(hipStream_t st, const GemmArgs& g) {
    constexpr bool F32OUT = EPI == EPI_RESID_F32 || EPI == EPI_F32;
    if constexpr (F32OUT && C::KG == 4 && C::BM <= SPK_FEW_ROWS && AFORM == OP_KMAJOR && WFORM == OP_KMAJOR)
        if (g.M <= SPK_FEW_ROWS) return launch_acc<C, EPI, AFORM, WFORM, 2>(st, g);
    return launch_acc<C, EPI, AFORM, WFORM, 1>(st, g);
}

// Tile ids 14..20.  32x32 and 16x32 leave room for two work-groups per CU.
//                 BM  BN WM WN KG NST
typedef SmallCfg<16, 16, 1, 1, 8, 4> S14;
typedef SmallCfg<16, 32, 1, 1, 4, 3> S15;
typedef SmallCfg<32, 32, 1, 1, 4, 2> S16;
typedef SmallCfg<64, 32, 1, 1, 4, 3> S17;
typedef SmallCfg<64, 64, 1, 1, 4, 2> S18;
typedef SmallCfg<96, 64, 1, 1, 4, 2> S19;
typedef SmallCfg<64, 128, 2, 4, 1, 4> S20;

template <int EPI, int AFORM, int WFORM>
hipError_t launch_tile(hipStream_t st, const GemmArgs& g) {
    switch (g.tile) {
        case 16: return launch_small<S16, EPI, AFORM, WFORM>(st, g);
        case 18: return launch_small<S18, EPI, AFORM, WFORM>(st, g);
    }
    if constexpr (AFORM == OP_KMAJOR && WFORM == OP_KMAJOR) {
        switch (g.tile) {
            case 14: return launch_small<S14, EPI, AFORM, WFORM>(st, g);
            case 15: return launch_small<S15, EPI, AFORM, WFORM>(st, g);
            case 17: return launch_small<S17, EPI, AFORM, WFORM>(st, g);
            case 19: return launch_small<S19, EPI, AFORM, WFORM>(st, g);
            case 20: return launch_small<S20, EPI, AFORM, WFORM>(st, g);
        }
    }
    return hipErrorInvalidValue;
}

// Estimated time of a tile in us: launch, prologue and epilogue (a, b per unit), operand tiles (c per
// unit and 1000 of K), the weights from HBM (bw, TB/s).  A unit is one work-group on every CU.
// Fitted to 160 shapes (M 17..2560, N 256..12288, K 256..11008), rms error 7-14 %.  (Operands with the row index
// contiguous are compared with the large tiles in one table, k_gemm.hip.)
struct SmallCost { int id, bm, bn, per_cu; float a, b, c, bw; };
constexpr SmallCost kSmallK[] = {{16, 32, 32, 2, 1.9f, 0.16f, 1.52f, 13.0f}, {17, 64, 32, 1, 0.5f, 2.2f, 2.24f, 17.5f},
                                 {18, 64, 64, 1, 0.5f, 3.1f, 3.03f, 12.8f},  {19, 96, 64, 1, 0.5f, 3.95f, 3.82f, 16.6f},
                                 {20, 64, 128, 1, 0.5f, 2.9f, 5.48f, 13.9f}};
int cheapest(int epi, int M, int N, int K, float* us) {
    int best = 0;
    for (const SmallCost& t : kSmallK) {
        const int bn_out = epi == EPI_SWIGLU_BF16 ? t.bn / 2 : t.bn;
        const long tiles = (long)((M + t.bm - 1) / t.bm) * ((N + bn_out - 1) / bn_out), round = 256 * t.per_cu;
        const long units = tiles / round * t.per_cu + (tiles % round == 0 ? 0 : tiles % round <= 256 ? 1 : t.per_cu);
        const float w_mb = (epi == EPI_SWIGLU_BF16 ? 2.f : 1.f) * (float)N * (float)K * 2e-6f;
        const float c = t.a + (float)units * (t.b + t.c * (float)K * 1e-3f) + w_mb / t.bw;
        if (!best || c < *us) { best = t.id; *us = c; }
    }
    return best;
}

}  // namespace

int spk_small_gemm_tile(int epi, int a_form, int w_form, int M, int N, int K, float* us) {
    const int forms = a_form * 2 + w_form;
    if (forms == 0) {
        if (M > 16) return cheapest(epi, M, N, K, us);
        // at most 16 rows: 16 columns per work-group while that is one round of the chip (4096 x 4096,
        // 8 rows: 8.5 us against 10.6), 32 beyond (11008 x 4096 SwiGLU: 38.3 against 32.1)
        *us = 0.f;
        return (epi == EPI_SWIGLU_BF16 ? (N + 7) / 8 : (N + 15) / 16) <= 256 ? 14 : 15;
    }
    return 0;
}

hipError_t spk_launch_gemm_small(hipStream_t st, int epi, const GemmArgs& g) {
    const int forms = g.a_form * 2 + g.w_form;
    switch (epi) {
        case EPI_BF16:
            if (forms == 0) return launch_tile<EPI_BF16, OP_KMAJOR, OP_KMAJOR>(st, g);
            if (forms == 1) return launch_tile<EPI_BF16, OP_KMAJOR, OP_RMAJOR>(st, g);
            break;
        case EPI_RESID_F32:
            if (forms == 0) return launch_tile<EPI_RESID_F32, OP_KMAJOR, OP_KMAJOR>(st, g);
            break;
        case EPI_GELU_BF16:
            if (forms == 0 && g.bias) return launch_tile<EPI_GELU_BF16, OP_KMAJOR, OP_KMAJOR>(st, g);
            break;
        case EPI_SWIGLU_BF16:
            if (forms == 0 && !g.bias) return launch_tile<EPI_SWIGLU_BF16, OP_KMAJOR, OP_KMAJOR>(st, g);
            break;
        case EPI_F32:
            if (forms == 0) return launch_tile<EPI_F32, OP_KMAJOR, OP_KMAJOR>(st, g);
            if (forms == 1) return launch_tile<EPI_F32, OP_KMAJOR, OP_RMAJOR>(st, g);
            if (forms == 3) return launch_tile<EPI_F32, OP_RMAJOR, OP_RMAJOR>(st, g);
            break;
    }
    return hipErrorInvalidValue;
}
