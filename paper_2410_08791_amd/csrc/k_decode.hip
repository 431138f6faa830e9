// Autoregressive decode: key/value cache append and single-query attention over the cache.
//
// Cache of one layer (bf16):  Kt [B][Hkv][hd][max_len]   keys, position index contiguous
//                             V  [B][Hkv][max_len][hd]   values, head dimension contiguous
// Kt is stored transposed so that the score pass reads keys coalesced along the position
// (eight positions per lane); V rows are read coalesced along the head dimension by the
// weighted sum.  Both passes read every cached byte once: the kernel is HBM-bound,
// 4 n Hkv hd bytes per sequence for n cached positions.
#include "sp_common.h"
#include "sp_kernels.h"

namespace {

// Append S new positions (pos0 .. pos0+S-1) of every sequence from the fused activation
// qkv [B*S, ld] = [q | k | v].  One work-group: 64 positions of one (batch, kv head).  HBM-bound; WIDE: 16-byte
// accesses throughout, taken where rows, pointers and the first position allow (with 2-byte ones a prompt of
// 2048 tokens x 32 heads of 128 took 20.9 us for its 67 MB).
template <bool WIDE>
__global__ __launch_bounds__(256) void kv_append_kernel(const bf16_t* __restrict__ qkv, int ld, bf16_t* __restrict__ kt,
                                                        bf16_t* __restrict__ v, int S, int pos0, int Hq, int Hkv,
                                                        int hd, int max_len) {
    __shared__ __attribute__((aligned(16))) bf16_t tile[64][130];
    const int s0 = blockIdx.x * 64, h = blockIdx.y, b = blockIdx.z;
    const int ns = min(64, S - s0);
    const bf16_t* ksrc = qkv + (size_t)(b * S + s0) * ld + (size_t)(Hq + h) * hd;
    const bf16_t* vsrc = ksrc + (size_t)Hkv * hd;
    bf16_t* vdst = v + ((size_t)(b * Hkv + h) * max_len + pos0 + s0) * hd;
    bf16_t* kdst = kt + (size_t)(b * Hkv + h) * hd * max_len + pos0 + s0;
    if (WIDE) {
        const int cpr = hd / 8;
        for (int i = threadIdx.x; i < ns * cpr; i += 256) {
            const int s = i / cpr, d = (i - s * cpr) * 8;
            const u32x4_t kw = *reinterpret_cast<const u32x4_t*>(ksrc + (size_t)s * ld + d);
            *reinterpret_cast<u32x4_t*>(vdst + (size_t)s * hd + d) = *reinterpret_cast<const u32x4_t*>(vsrc + (size_t)s * ld + d);
#pragma unroll
            for (int j = 0; j < 4; ++j) *reinterpret_cast<uint32_t*>(&tile[s][d + 2 * j]) = kw[j];     // rows of 260 bytes
        }
    } else {
        for (int i = threadIdx.x; i < ns * hd; i += 256) {
            const int s = i / hd, d = i - s * hd;
            tile[s][d] = ksrc[(size_t)s * ld + d];
            vdst[(size_t)s * hd + d] = vsrc[(size_t)s * ld + d];
        }
    }
    __syncthreads();
    if (WIDE) {
        // eight positions per lane; the last, short piece of a ragged prompt position by position
        for (int i = threadIdx.x; i < hd * 8; i += 256) {
            const int d = i >> 3, s = (i & 7) * 8;
            if (s + 8 <= ns) {
                u32x4_t w;
#pragma unroll
                for (int j = 0; j < 4; ++j) w[j] = (uint32_t)tile[s + 2 * j][d] | ((uint32_t)tile[s + 2 * j + 1][d] << 16);
                *reinterpret_cast<u32x4_t*>(kdst + (size_t)d * max_len + s) = w;
            } else {
                for (int j = s; j < ns; ++j) kdst[(size_t)d * max_len + j] = tile[j][d];
            }
        }
        return;
    }
    const int s = threadIdx.x & 63;
    if (s < ns)
        for (int d = threadIdx.x >> 6; d < hd; d += 4) kdst[(size_t)d * max_len + s] = tile[s][d];
}

// Attention of one query per sequence over the cached positions [0, n), and (fresh) over the position n
// whose key and value are still in the fused activation: they are taken from there and stored into the
// cache by the way, so a decode step needs no append launch in front.
//
// One work-group = one split of the positions for one key/value head and G of the query heads that
// share it: a cached byte is read once for all G (one work-group per query head read a group's cache
// Hq / Hkv times and left most of the chip idle for few sequences: 2 x 32/8 heads over 8191 positions
// 107 us).  Each of the NW waves walks its own positions, 128 at a time, with its own running
// maximum, sum and output, and needs no barrier before the end: a lane holds 8 positions (16 bytes of a
// Kt row), the quarter-waves split the head dimension and add up by two shuffles, so every load is 16
// bytes and 16 (keys) or 8 (values) of them are in flight per lane.  A long split is dealt to the waves in
// steps of 128 positions, so that a work-group reads NW x 256 neighbouring bytes of a Kt row at a time (a run
// of its own per wave: 64 x 32 heads of 128 over 2000 positions 414 us, 389 so), a short one in NW even runs.
// Row addresses are a uniform base and one 32-bit lane offset: 64-bit addresses per row took half the
// registers (196 against 132 at G = 1).  The waves' results meet in LDS.  With
// more than one split the unnormalised rows go to `part` (fp32: HD values, reference maximum in base 2,
// denominator) and combine_kernel adds them in split order.  Without that scratch (KS > 1) one work-group of
// KS x NW waves takes all splits of a query head, KS at a time, leaves their rows in LDS and adds them in the same
// order: the same bits from fewer work-groups.
// HBM-bound: 4 n Hkv hd bytes per sequence.
//
// A score of -inf has weight 0 whichever positions a wave holds: where every score of a wave or split so far
// is -inf, 0 stands in for the maximum in the differences taken with it (-inf - -inf would make the row NaN).
__device__ __forceinline__ float finite_ref(float m) { return m == -INFINITY ? 0.f : m; }

// Element d of the result from the rows of its splits, by whole waves.  At most 64 splits (kDecodeMaxLen / 512):
// lane s weighs split s, then every thread adds its element of the rows, eight loads in flight (one dependent
// chain of loads per split took 10.5 us for 16 splits).
template <int HD>
__device__ __forceinline__ float combine_rows(const float* p, int splits, int d) {
    const int lane = threadIdx.x & 63;
    const bool on = lane < splits;
    const float2 ml = on ? *reinterpret_cast<const float2*>(p + lane * (HD + 2) + HD) : make_float2(-INFINITY, 0.f);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = j < splits ? p[j * (HD + 2) + d] : 0.f;
    const float M = finite_ref(wave_max(ml.x));
    const float f = on ? __builtin_amdgcn_exp2f(ml.x - M) : 0.f;
    const float L = wave_sum(f * ml.y);
    float acc = 0.f;
    for (int s0 = 0; s0 < splits; s0 += 8) {
        if (s0)
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = s0 + j < splits ? p[(s0 + j) * (HD + 2) + d] : 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc = fmaf(__shfl(f, s0 + j, 64), v[j], acc);     // s0 + j <= 63
    }
    return acc / L;
}

template <int HD, int G, int NW, int KS>
__global__ __launch_bounds__(NW * KS * 64) void decode_attn_kernel(
    const bf16_t* __restrict__ qkv, int ld_qkv, bf16_t* kt, bf16_t* v, bf16_t* __restrict__ o, int ld_o,
    float* __restrict__ part, int n, int fresh, int splits, int per_split, int max_len, int Hq, int Hkv, float scale_log2e) {
    constexpr int DQ = HD / 4;             // head-dimension elements per quarter-wave in the score pass
    constexpr int LPR = HD / 8;            // lanes per V row
    constexpr int RPI = 64 / LPR;          // V rows per load instruction
    constexpr int TB = 128;                // positions per wave and step
    constexpr int KBATCH = KS > 1 ? 8 : 16, VBATCH = 8;         // KS > 1: sixteen waves, 128 registers each
    constexpr bool SEQ = KS > 1;
    constexpr int MAX_SPLITS = kDecodeMaxLen / 512;
    __shared__ float qs[G][HD];
    __shared__ __attribute__((aligned(16))) float buf[NW * KS * G * TB];   // a wave's probabilities, then its output rows
    __shared__ float wm[NW * KS][G], wl[NW * KS][G];
    __shared__ __attribute__((aligned(16))) float rows_lds[SEQ ? G * MAX_SPLITS * (HD + 2) : 1];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = Hq / Hkv, ngb = (grp + G - 1) / G;
    const int wi = w % NW, sub = w / NW;   // wave of its split, split of the KS
    int split = SEQ ? sub : blockIdx.x;
    const int hk = blockIdx.y / ngb, h0 = (blockIdx.y % ngb) * G, b = blockIdx.z;
    const bf16_t* row = qkv + (size_t)b * ld_qkv;
    for (int i = threadIdx.x; i < G * HD; i += NW * KS * 64) {
        const int g = i / HD, h = min(h0 + g, grp - 1);       // heads past the group repeat its last one and are not stored
        qs[g][i % HD] = bf2f(row[(size_t)(hk * grp + h) * HD + i % HD]) * scale_log2e;
    }
    __syncthreads();

    bf16_t* K = kt + (size_t)(b * Hkv + hk) * HD * max_len;
    bf16_t* V = v + (size_t)(b * Hkv + hk) * max_len * HD;
    const int qw = lane >> 4, l16 = lane & 15;
    const int vrow = lane / LPR, dp = 8 * (lane % LPR);
    const int per_wave = (per_split / NW + 7) & ~7;
    const bool dealt = per_split >= NW * TB;
    float* ps = buf + w * G * TB;          // [position][G]
    for (;;) {                             // SEQ: KS splits at a time, past the last one a wave has no positions
    const int s1 = min(n, (split + 1) * per_split);
    const int w0 = split * per_split + wi * (dealt ? TB : per_wave), wend = dealt ? s1 : min(s1, w0 + per_wave);
    float m[G], l[G], oa[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        m[g] = -INFINITY; l[g] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) oa[g][e] = 0.f;
    }
    for (int t0 = w0; t0 < wend; t0 += dealt ? NW * TB : TB) {
        const int w1 = min(wend, t0 + TB);
        // scores.  max_len is a multiple of 8, so a lane's 8 positions lie inside the cache row.
        const int t = t0 + l16 * 8;
        float a[G][8];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 8; ++e) a[g][e] = 0.f;
        if (t < w1) {
            const unsigned kofs = qw * DQ * max_len + t;
#pragma unroll
            for (int d0 = 0; d0 < DQ; d0 += KBATCH) {
                u32x4_t kk[KBATCH];
#pragma unroll
                for (int d = 0; d < KBATCH; ++d)
                    kk[d] = *reinterpret_cast<const u32x4_t*>(K + (size_t)(d0 + d) * max_len + kofs);
                __builtin_amdgcn_sched_barrier(0);      // all loads first: paired with their uses each would be waited for
#pragma unroll
                for (int d = 0; d < KBATCH; ++d)
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const float q = qs[g][qw * DQ + d0 + d];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            a[g][2 * e] = fmaf(q, bf_lo(kk[d][e]), a[g][2 * e]);
                            a[g][2 * e + 1] = fmaf(q, bf_hi(kk[d][e]), a[g][2 * e + 1]);
                        }
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // this step's first value rows are fetched under the softmax
        const int rows = w1 - t0;
        u32x4_t vv[VBATCH];
#pragma unroll
        for (int j = 0; j < VBATCH; ++j)
            vv[j] = *reinterpret_cast<const u32x4_t*>(V + (unsigned)(min(t0 + j * RPI + vrow, w1 - 1) * HD + dp));
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float mx = -INFINITY;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float x = a[g][e];
                x += __shfl_xor(x, 16, 64);
                x += __shfl_xor(x, 32, 64);
                x = t + e < w1 ? x : -INFINITY;
                a[g][e] = x;
                mx = fmaxf(mx, x);
            }
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
            mx = fmaxf(m[g], mx);
            const float ref = finite_ref(mx);
            const float alpha = __builtin_amdgcn_exp2f(m[g] - ref);
            m[g] = mx;
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                a[g][e] = __builtin_amdgcn_exp2f(a[g][e] - ref);
                sum += a[g][e];
            }
            l[g] = fmaf(l[g], alpha, sum);               // of this lane's positions
#pragma unroll
            for (int e = 0; e < 8; ++e) oa[g][e] *= alpha;
            if (qw == (g & 3))
#pragma unroll
                for (int e = 0; e < 8; ++e) ps[(l16 * 8 + e) * G + g] = a[g][e];
        }
        __builtin_amdgcn_wave_barrier();
        // weighted sum: row groups of RPI value rows; a wave's LDS accesses are in order
        for (int r0 = 0; r0 < rows; r0 += VBATCH * RPI) {
            if (r0) {
#pragma unroll
                for (int j = 0; j < VBATCH; ++j)
                    vv[j] = *reinterpret_cast<const u32x4_t*>(V + (unsigned)(min(t0 + r0 + j * RPI + vrow, w1 - 1) * HD + dp));
                __builtin_amdgcn_sched_barrier(0);
            }
            if (r0 + VBATCH * RPI > rows) {
                // rows past the run repeat its last one: cleared, since 0 times an infinite value would be NaN
#pragma unroll
                for (int j = 0; j < VBATCH; ++j)
                    if (r0 + j * RPI + vrow >= rows) vv[j] = u32x4_t{0, 0, 0, 0};
            }
#pragma unroll
            for (int j = 0; j < VBATCH; ++j) {
                const int r = r0 + j * RPI + vrow;       // < TB; positions past the run have probability 0
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float p = ps[r * G + g];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        oa[g][2 * e] = fmaf(p, bf_lo(vv[j][e]), oa[g][2 * e]);
                        oa[g][2 * e + 1] = fmaf(p, bf_hi(vv[j][e]), oa[g][2 * e + 1]);
                    }
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (fresh && split == splits - 1 && wi == NW - 1) {
        // the new position: scored and added like a run of one, and stored (by the first head block)
        const bf16_t* kn = row + (size_t)(Hq + hk) * HD;
        const bf16_t* vn = kn + (size_t)Hkv * HD;
        constexpr int EPL = HD / 64;
        const u32x4_t nv = *reinterpret_cast<const u32x4_t*>(vn + dp);
        const u32x4_t pv = vrow == 0 ? nv : u32x4_t{0, 0, 0, 0};
        bf16_t kb[EPL];
        float kf[EPL];
#pragma unroll
        for (int e = 0; e < EPL; ++e) { kb[e] = kn[lane + 64 * e]; kf[e] = bf2f(kb[e]); }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) s = fmaf(qs[g][lane + 64 * e], kf[e], s);
            s = wave_sum(s);
            const float mx = fmaxf(m[g], s), ref = finite_ref(mx);
            const float alpha = __builtin_amdgcn_exp2f(m[g] - ref), p = __builtin_amdgcn_exp2f(s - ref);
            m[g] = mx;
            l[g] = fmaf(l[g], alpha, l16 == 0 ? p : 0.f);
            const float pr = vrow == 0 ? p : 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                oa[g][2 * e] = fmaf(pr, bf_lo(pv[e]), oa[g][2 * e] * alpha);
                oa[g][2 * e + 1] = fmaf(pr, bf_hi(pv[e]), oa[g][2 * e + 1] * alpha);
            }
        }
        if (h0 == 0) {
#pragma unroll
            for (int e = 0; e < EPL; ++e) K[(size_t)(lane + 64 * e) * max_len + n] = kb[e];
            if (vrow == 0) *reinterpret_cast<u32x4_t*>(V + (size_t)n * HD + dp) = nv;
        }
    }

    // a wave's row groups, then the waves, in a fixed order
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) l[g] += __shfl_xor(l[g], off, 64);
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int off = LPR; off < 64; off <<= 1) oa[g][e] += __shfl_xor(oa[g][e], off, 64);
    }
    __syncthreads();                       // buf changes hands
    if (vrow == 0)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 8; ++e) buf[(w * G + g) * HD + dp + e] = oa[g][e];
    if (lane == 0)
#pragma unroll
        for (int g = 0; g < G; ++g) { wm[w][g] = m[g]; wl[w][g] = l[g]; }
    __syncthreads();
    for (int i = threadIdx.x - sub * NW * 64; i < G * HD; i += NW * 64) {
        const int g = i / HD, d = i % HD, k0 = sub * NW;
        if (h0 + g >= grp || split >= splits) continue;
        float M = wm[k0][g];
#pragma unroll
        for (int k = 1; k < NW; ++k) M = fmaxf(M, wm[k0 + k][g]);
        const float ref = finite_ref(M);
        float L = 0.f, acc = 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const float f = __builtin_amdgcn_exp2f(wm[k0 + k][g] - ref);      // 0 for a wave without positions
            L = fmaf(f, wl[k0 + k][g], L);
            acc = fmaf(f, buf[((k0 + k) * G + g) * HD + d], acc);
        }
        const int hq = hk * grp + h0 + g;
        if (!SEQ && splits == 1) {
            o[(size_t)b * ld_o + hq * HD + d] = f2bf(acc / L);
        } else {
            float* pr = SEQ ? rows_lds + (g * splits + split) * (HD + 2) : part + ((size_t)(b * Hq + hq) * splits + split) * (HD + 2);
            pr[d] = acc;
            if (d == 0) { pr[HD] = M; pr[HD + 1] = L; }
        }
    }
    if (!SEQ) break;
    __syncthreads();                       // the waves' results have been read out of buf
    split += KS;
    if (split - sub >= splits) break;
    }
    if (SEQ) {
        for (int i = threadIdx.x; i < G * HD; i += NW * KS * 64) {     // whole waves per head
            const int g = i / HD, d = i % HD;
            if (h0 + g < grp)
                o[(size_t)b * ld_o + (hk * grp + h0 + g) * HD + d] = f2bf(combine_rows<HD>(rows_lds + g * splits * (HD + 2), splits, d));
        }
    }
}

template <int HD>
__global__ __launch_bounds__(HD) void combine_kernel(const float* __restrict__ part, int splits, bf16_t* __restrict__ o,
                                                     int ld_o, int Hq) {
    const int hq = blockIdx.x, b = blockIdx.y;
    o[(size_t)b * ld_o + hq * HD + threadIdx.x] = f2bf(combine_rows<HD>(part + (size_t)(b * Hq + hq) * splits * (HD + 2), splits, threadIdx.x));
}

struct DecodeCall {
    const bf16_t* qkv; int ld_qkv;
    bf16_t *kt, *v, *o; int ld_o;
    float* part;
    int B, n, fresh, max_len, Hq, Hkv;
    bool one_split;
};

template <int HD, int G, int NW, int KS>
hipError_t launch_one(hipStream_t st, const DecodeCall& c, int splits, int per) {
    const float sl2 = 1.4426950408889634f / sqrtf((float)HD);
    const dim3 grid(KS > 1 ? 1 : splits, c.Hkv * ((c.Hq / c.Hkv + G - 1) / G), c.B);
    decode_attn_kernel<HD, G, NW, KS><<<grid, NW * KS * 64, 0, st>>>(c.qkv, c.ld_qkv, c.kt, c.v, c.o, c.ld_o, c.part, c.n, c.fresh, splits,
                                                                     per, c.max_len, c.Hq, c.Hkv, sl2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || KS > 1 || splits == 1) return e;
    combine_kernel<HD><<<dim3(c.Hq, c.B), HD, 0, st>>>(c.part, splits, c.o, c.ld_o, c.Hq);
    return hipGetLastError();
}

// Splits, query heads per work-group and waves.  Splits and waves, which the order of the sums depends on, follow
// from the shapes alone; without a scratch for the splits' rows G is 1.
//   splits: none below 1024 positions (they would save less than the second launch costs).  Above, there are two plans.
//     Coarse: enough splits to fill the chip once, of at least 512 positions, in work-groups of eight waves.
//     Fine: as many as fill it twice, with at least 256 positions each, and beyond 16 of them with 512 -- more rows of
//     partial results cost the second launch more than shorter splits save -- in work-groups of two or four waves.
//     Neither has more rows than decode_scratch_floats counts.
//   G: the fewest heads whose work-groups still fit one round of the chip (fine: two rounds of small ones; else 256, or
//     1024 of two waves); a group's cache is then read again through the L2, which costs less than idle CUs.  Always
//     sharing it cost, us: 1 x 64/8 heads of 128 over 500 positions 34.3 against 9.1, 4 x 64/8 over 800 38.6 against
//     19.5; never sharing it 32 x 32/8 over 500 39.5 against 21.  More than four heads per work-group spilled registers
//     and was slower than two blocks of four (8 x 64/8 over 4096 positions 91 against 43).
//   NW: a wave with less than a step of 128 positions idles in its loads, and every wave has its part in the
//     merge: 64 x 32 heads over 16 positions 42.6 us with eight waves, 15.8 with two.  Several rounds of work-groups
//     of a split launch overlap better in small ones (8 x 64/8 over 4096, G = 4: four waves 45, two 39).
// Which of the two, by the coarse plan's work-groups (us, coarse and fine):
//   up to 120, not half the chip, or more than 256, a second round: fine (2 x 16/4 heads of 128 over 1955 positions 11.6
//     and 9.4, 8 x 48/12 over 1779 33.5 and 25.0) -- but not where the coarse one all but fills two rounds and the fine
//     one, with its larger head blocks, would begin a third (38 x 24/3 of 64 over 1053 23.4 and 24.3).
//   between: coarse.  The fine plan's work-groups, not many more than 256 of them or with the heads that read one cache
//     on different XCDs, took up to 1.39 times as long (2 x 8/2 heads of 128 over 8649 positions 13.3 and 18.5, 4 x 32/4
//     of 64 over 2139 11.0 and 14.3) as often as they were quicker.  Not so where they all but fill two rounds and share
//     a cache in multiples of eight splits: ids go round the eight XCDs, so the heads of a split then meet in
//     one L2 (2 x 32/8 of 128 over 8191 22.9 and 20.5, over 1813 15.1 and 11.3).  For the same reason a coarse plan of more
//     than a round in such splits stays where the fine one has none (2 x 64/8 of 128 over 13506 42.4 and 46.4).
// On 200 shapes drawn after the rule stood: 5.9 % quicker than coarse plans alone on average, none more than 2 % slower;
// without a scratch 4.3 %, slowest 9 x 12/6 of 64 over 3765 28.2 and 30.7 (three turns for two).  Fine plans alone, on 179
// others: 7 %, but 42 slower by more than 2 %.
// Without a scratch one work-group runs 16 / NW splits of a head at a time: where the coarse plan needs one turn, a fine
// one for a second round needs no more (2 x 44/44 heads of 64 over 1540 positions, no scratch: 14.5 us in three splits,
// 18.6 in five of four waves).
// One split: against 258 shapes (1..64 sequences, groups of 1 to 8, 20..16000 positions) 3.6 % off the best of all
// combinations on average.
struct DecodePlan { int splits, per, G, NW; };
long decode_groups(const DecodeCall& c, int G, int splits) { return (long)c.B * c.Hkv * ((c.Hq / c.Hkv + G - 1) / G) * splits; }

DecodePlan plan_splits(const DecodeCall& c, int splits, bool fine) {
    const int grp = c.Hq / c.Hkv;
    DecodePlan p;
    p.per = std::max(((c.n + splits - 1) / splits + 63) / 64 * 64, 64);
    p.splits = std::max((c.n + p.per - 1) / p.per, 1);           // none is empty
    p.NW = fine ? (p.per <= 256 ? 2 : 4) : p.per <= 128 ? 2 : p.per <= 400 ? 4 : 8;
    p.G = 1;
    while (p.G < 4 && p.G < grp && decode_groups(c, p.G, p.splits) > (fine ? 512 : p.NW == 2 ? 1024 : 256)) p.G *= 2;
    const long groups = decode_groups(c, p.G, p.splits);
    if (p.splits > 1 && groups > (fine ? 512 : 256)) p.NW = p.G == 4 && groups > 512 ? 2 : fine ? p.NW : 4;
    return p;
}

DecodePlan plan_decode(const DecodeCall& c) {
    if (c.one_split || c.n < 1024) return plan_splits(c, 1, false);
    const int room = std::max(kDecodeSplitGroups / (c.B * c.Hkv), 1);
    const DecodePlan coarse = plan_splits(c, std::min(room, c.n / 512), false);
    const int splits = std::min(std::min(room, (c.n + 255) / 256), std::max(16, (c.n + 511) / 512));
    if (splits == 1) return coarse;
    DecodePlan fine = plan_splits(c, splits, true);
    const long in_coarse = decode_groups(c, coarse.G, coarse.splits), in_fine = decode_groups(c, fine.G, fine.splits);
    const int grp = c.Hq / c.Hkv;
    if (in_coarse > 120 && in_coarse <= 256) return fine.splits % 8 == 0 && fine.G < grp && in_fine >= 448 ? fine : coarse;
    if (in_coarse > 256 && coarse.splits % 8 == 0 && coarse.G < grp && fine.splits % 8) return coarse;
    if (in_coarse > 448 && in_coarse <= 512 && in_fine > 512) return coarse;
    const int turn = 16 / fine.NW;
    if (in_coarse > 256 && coarse.splits <= 16 / coarse.NW && fine.splits > turn) fine = plan_splits(c, turn, true);
    return fine;
}

template <int HD>
hipError_t launch_decode(hipStream_t st, const DecodeCall& c) {
    const DecodePlan p = plan_decode(c);
    if (p.splits > 1 && !c.part)
        return p.NW == 2 ? launch_one<HD, 1, 2, 8>(st, c, p.splits, p.per) : p.NW == 4 ? launch_one<HD, 1, 4, 4>(st, c, p.splits, p.per)
                                                                                       : launch_one<HD, 1, 8, 2>(st, c, p.splits, p.per);
#define SP_DECODE(g, w) if (p.G == g && p.NW == w) return launch_one<HD, g, w, 1>(st, c, p.splits, p.per);
    SP_DECODE(1, 2) SP_DECODE(1, 4) SP_DECODE(1, 8) SP_DECODE(2, 2) SP_DECODE(2, 4) SP_DECODE(2, 8) SP_DECODE(4, 2) SP_DECODE(4, 4) SP_DECODE(4, 8)
#undef SP_DECODE
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t spk_launch_kv_append(hipStream_t st, const bf16_t* qkv, int ld_qkv, bf16_t* kt, bf16_t* v, int B, int S,
                                int pos0, int Hq, int Hkv, int hd, int max_len) {
    if (B < 1 || S < 1 || pos0 < 0 || pos0 + S > max_len || hd > 128 || hd < 1 || Hkv < 1 || Hq < Hkv)
        return hipErrorInvalidValue;
    const dim3 grid((S + 63) / 64, Hkv, B);
    if ((hd | ld_qkv | max_len | pos0) % 8 == 0 && (((uintptr_t)qkv | (uintptr_t)kt | (uintptr_t)v) & 15) == 0)
        kv_append_kernel<true><<<grid, 256, 0, st>>>(qkv, ld_qkv, kt, v, S, pos0, Hq, Hkv, hd, max_len);
    else
        kv_append_kernel<false><<<grid, 256, 0, st>>>(qkv, ld_qkv, kt, v, S, pos0, Hq, Hkv, hd, max_len);
    return hipGetLastError();
}

void spk_decode_plan_host(int B, int n, int Hq, int Hkv, int* out4) {
    DecodeCall c{};
    c.B = B; c.n = n; c.Hq = Hq; c.Hkv = Hkv;
    const DecodePlan p = plan_decode(c);
    out4[0] = p.splits; out4[1] = p.per; out4[2] = p.G; out4[3] = p.NW;
}

static hipError_t decode_step(hipStream_t st, const DecodeCall& c, int hd) {
    const int n = c.n + c.fresh;
    if (c.B < 1 || n < 1 || n > c.max_len || (c.max_len & 7) || c.max_len > kDecodeMaxLen || c.Hkv < 1 || c.Hq % c.Hkv ||
        ((uintptr_t)c.kt & 15) || ((uintptr_t)c.v & 15))
        return hipErrorInvalidValue;
    // queries are read one by one; the new value row, which only a step has, by 16 bytes
    if (c.fresh && (c.ld_qkv % 8 || ((uintptr_t)c.qkv & 15))) return hipErrorInvalidValue;
    if (hd == 128) return launch_decode<128>(st, c);
    if (hd == 64) return launch_decode<64>(st, c);
    return hipErrorInvalidValue;
}

hipError_t spk_launch_decode_attention(hipStream_t st, const bf16_t* qkv, int ld_qkv, const bf16_t* kt,
                                       const bf16_t* v, bf16_t* o, int ld_o, int B, int n, int max_len, int Hq,
                                       int Hkv, int hd) {
    // nothing is stored without a fresh position; no scratch, and no other form whose bits it would have to match
    return decode_step(st, DecodeCall{qkv, ld_qkv, const_cast<bf16_t*>(kt), const_cast<bf16_t*>(v), o, ld_o, nullptr, B, n, 0, max_len, Hq, Hkv,
                                      true}, hd);
}

hipError_t spk_launch_decode_step(hipStream_t st, const bf16_t* qkv, bf16_t* o, const AttnShape& a) {
    return decode_step(st, DecodeCall{qkv, a.ld_qkv, a.kt, a.v, o, a.Hq * a.hd, a.part, a.B, a.pos, 1, a.max_len, a.Hq, a.Hkv, false}, a.hd);
}
