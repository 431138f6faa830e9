// Norm backward over many rows, RMSNorm and LayerNorm: a row is held by WPR waves (1, 2, 4: rows of at most
// 2048, 4096, 8192 elements; a lane keeps at most eight float4 of da, h and dh), a work-group of eight waves
// has 8 / WPR rows in flight and walks rows with the grid.  HBM-bound: 18 bytes per element (da, h and dh in,
// dh and its bf16 copy out).  With one row per work-group the loads of a row were waited for before the next row's were issued
// and four to six barriers separated the rows: LayerNorm 8224 x 1280 123 us, RMSNorm 16384 x 4096 409 us.
//
// RMSNorm   a = h r g, r = rsqrt(mean(h^2) + eps):
//           dh_io += r (da g) - h r^3 mean(da g h),  dgain = sum_t da h r
// LayerNorm a = xhat g + b, xhat = (h - mean) r, q = da g:
//           dh_io += r (q - mean(q) - xhat mean(q xhat)),  dgain = sum_t da xhat,  dbias = sum_t da
// Partial row b of `part` (d floats, LayerNorm [dgain | dbias]) holds the sums over the work-group's rows, the
// waves' shares added in wave order: every sum has a fixed order.
#pragma once
#include "sp_common.h"
#include "sp_limits.h"

constexpr int NB_ROWS_V = 8;        // float4 per lane, at most
constexpr int NB_ROWS_WAVES = 8;

// sums over the WPR waves of a row; `red` is one float4 per wave
template <int WPR>
__device__ __forceinline__ void row_sum3(float& a, float& b, float& c, float4* red, int wave) {
    a = wave_sum(a); b = wave_sum(b); c = wave_sum(c);
    if (WPR == 1) return;
    __syncthreads();                // the previous use has been read
    if ((threadIdx.x & 63) == 0) red[wave] = make_float4(a, b, c, 0.f);
    __syncthreads();
    const int w0 = wave / WPR * WPR;
    float4 s = red[w0];
#pragma unroll
    for (int i = 1; i < WPR; ++i) {
        const float4 o = red[w0 + i];
        s.x += o.x; s.y += o.y; s.z += o.z;
    }
    a = s.x; b = s.y; c = s.z;
}

template <bool LN, int WPR, int V>
__global__ __launch_bounds__(NB_ROWS_WAVES * 64) void norm_bwd_rows_kernel(
    const float* __restrict__ da, const float* __restrict__ h, const bf16_t* __restrict__ gain, float* __restrict__ dh_io,
    bf16_t* __restrict__ dhb, float* __restrict__ part, int T, int d, float eps) {
    __shared__ float4 acc[(LN ? 2 : 1) * WPR * 64 * V];
    __shared__ float4 red[NB_ROWS_WAVES];
    constexpr int ROWS = NB_ROWS_WAVES / WPR;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sub = wave / WPR, col = wave % WPR * 64 + lane;     // float4 col, col + 64 WPR, ... of row slot `sub`
    const int nv = d >> 2;
    const float inv_d = 1.0f / (float)d;
    float4 gacc[V], bacc[LN ? V : 1];
    uint2 gv[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        gacc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (LN) bacc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        const int idx = col + i * 64 * WPR;
        gv[i] = idx < nv ? reinterpret_cast<const uint2*>(gain)[idx] : make_uint2(0, 0);
    }
    // with WPR > 1 the waves meet at barriers: every wave makes every trip, those without a row on zeros
    const int trips = (T + gridDim.x * ROWS - 1) / (gridDim.x * ROWS);
    for (int t = 0; t < trips; ++t) {
        const int row = (t * (int)gridDim.x + (int)blockIdx.x) * ROWS + sub;
        const bool on = row < T;
        const size_t base = (size_t)(on ? row : 0) * d;
        const float4* hp = reinterpret_cast<const float4*>(h + base);
        const float4* ap = reinterpret_cast<const float4*>(da + base);
        float4* op = reinterpret_cast<float4*>(dh_io + base);
        float4 hv[V], av[V], ov[V];
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int idx = col + i * 64 * WPR;
            hv[i] = av[i] = ov[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (on && idx < nv) { hv[i] = hp[idx]; av[i] = ap[idx]; ov[i] = op[idx]; }
        }
        // a lane's sums run in two chains: one of eight float4 had a 2-5 % larger error than the rows spread over a
        // whole work-group
        float mean = 0.f, mean1 = 0.f, zero0 = 0.f, zero1 = 0.f;
        if (LN) {
#pragma unroll
            for (int i = 0; i < V; ++i) (i & 1 ? mean1 : mean) += (hv[i].x + hv[i].y) + (hv[i].z + hv[i].w);
            mean += mean1;
            row_sum3<WPR>(mean, zero0, zero1, red, wave);
            mean *= inv_d;
        }
        float ss[2] = {0.f, 0.f}, dot[2] = {0.f, 0.f}, sq[2] = {0.f, 0.f};      // sums of hc^2, q hc, q with hc = h - mean
#pragma unroll
        for (int i = 0; i < V; ++i) {
            if (LN && col + i * 64 * WPR < nv) { hv[i].x -= mean; hv[i].y -= mean; hv[i].z -= mean; hv[i].w -= mean; }
            ss[i & 1] += (hv[i].x * hv[i].x + hv[i].y * hv[i].y) + (hv[i].z * hv[i].z + hv[i].w * hv[i].w);
            const float qx = av[i].x * bf_lo(gv[i].x), qy = av[i].y * bf_hi(gv[i].x), qz = av[i].z * bf_lo(gv[i].y),
                        qw = av[i].w * bf_hi(gv[i].y);
            dot[i & 1] += (qx * hv[i].x + qy * hv[i].y) + (qz * hv[i].z + qw * hv[i].w);
            if (LN) sq[i & 1] += (qx + qy) + (qz + qw);
        }
        float ss_all = ss[0] + ss[1], dot_all = dot[0] + dot[1], sq_all = sq[0] + sq[1];
        row_sum3<WPR>(ss_all, dot_all, sq_all, red, wave);
        const float r = rsqrtf(ss_all * inv_d + eps);
        const float c = (LN ? r : r * r * r) * dot_all * inv_d, m1 = LN ? sq_all * inv_d : 0.f;
        uint2* bp = reinterpret_cast<uint2*>(dhb + base);
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int idx = col + i * 64 * WPR;
            if (on && idx < nv) {
                float4 o = ov[i];
                const float gx = bf_lo(gv[i].x), gy = bf_hi(gv[i].x), gz = bf_lo(gv[i].y), gw = bf_hi(gv[i].y);
                if (LN) {
                    // fused by hand: the products with the gain exist already, and taken from there each would add a
                    // rounding (4.9e-8 relative error instead of 4.5e-8)
                    hv[i].x *= r; hv[i].y *= r; hv[i].z *= r; hv[i].w *= r;          // xhat
                    o.x = fmaf(r, fmaf(-hv[i].x, c, fmaf(av[i].x, gx, -m1)), o.x);
                    o.y = fmaf(r, fmaf(-hv[i].y, c, fmaf(av[i].y, gy, -m1)), o.y);
                    o.z = fmaf(r, fmaf(-hv[i].z, c, fmaf(av[i].z, gz, -m1)), o.z);
                    o.w = fmaf(r, fmaf(-hv[i].w, c, fmaf(av[i].w, gw, -m1)), o.w);
                } else {
                    o.x += r * av[i].x * gx - hv[i].x * c;
                    o.y += r * av[i].y * gy - hv[i].y * c;
                    o.z += r * av[i].z * gz - hv[i].z * c;
                    o.w += r * av[i].w * gw - hv[i].w * c;
                }
                op[idx] = o;
                bp[idx] = make_uint2(pack_bf2(o.x, o.y), pack_bf2(o.z, o.w));
                const float s = LN ? 1.f : r;
                gacc[i].x += av[i].x * hv[i].x * s;
                gacc[i].y += av[i].y * hv[i].y * s;
                gacc[i].z += av[i].z * hv[i].z * s;
                gacc[i].w += av[i].w * hv[i].w * s;
                if (LN) { bacc[i].x += av[i].x; bacc[i].y += av[i].y; bacc[i].z += av[i].z; bacc[i].w += av[i].w; }
            }
        }
    }
    // the row slots' partials: slot 0 stores, the others add theirs one after the other
    for (int w = 0; w < ROWS; ++w) {
        if (sub == w) {
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const int at = i * 64 * WPR + col;
                float4 g = gacc[i], b = LN ? bacc[LN ? i : 0] : g;
                if (w) {
                    const float4 o = acc[at];
                    g.x += o.x; g.y += o.y; g.z += o.z; g.w += o.w;
                }
                acc[at] = g;
                if (LN) {
                    if (w) {
                        const float4 o = acc[WPR * 64 * V + at];
                        b.x += o.x; b.y += o.y; b.z += o.z; b.w += o.w;
                    }
                    acc[WPR * 64 * V + at] = b;
                }
            }
        }
        __syncthreads();
    }
    float4* pp = reinterpret_cast<float4*>(part + (size_t)blockIdx.x * (LN ? 2 : 1) * d);
    for (int i = threadIdx.x; i < nv; i += NB_ROWS_WAVES * 64) {
        pp[i] = acc[i];
        if (LN) pp[nv + i] = acc[WPR * 64 * V + i];
    }
}

// Taken from 1024 rows on (below, the row slots of 256 work-groups are half empty and one work-group per row
// spreads better); SPK_NORM_BWD_BLOCKS partial rows.  LayerNorm rows beyond 4096 elements stay with one
// work-group per row: four waves' partials of gain and bias would take more than 64 KB of LDS.
template <bool LN>
inline bool norm_bwd_rows_fit(int T, int d) { return T >= 4 * SPK_NORM_BWD_BLOCKS && (!LN || d <= 2 * 64 * NB_ROWS_V * 4); }
template <bool LN>
void launch_norm_bwd_rows(hipStream_t st, const float* da, const float* h, const bf16_t* gain, float* dh_io, bf16_t* dhb,
                          float* part, int T, int d, float eps) {
    constexpr int NT = NB_ROWS_WAVES * 64, W = 64 * NB_ROWS_V * 4;
    // rows of at most 512 elements in two float4 per lane: eight, six of them idle, cost 8 to 12 % (8224 x 64, 8224 x 256)
    if (d <= W / 4) norm_bwd_rows_kernel<LN, 1, 2><<<SPK_NORM_BWD_BLOCKS, NT, 0, st>>>(da, h, gain, dh_io, dhb, part, T, d, eps);
    else if (d <= W) norm_bwd_rows_kernel<LN, 1, 8><<<SPK_NORM_BWD_BLOCKS, NT, 0, st>>>(da, h, gain, dh_io, dhb, part, T, d, eps);
    else if (d <= 2 * W) norm_bwd_rows_kernel<LN, 2, 8><<<SPK_NORM_BWD_BLOCKS, NT, 0, st>>>(da, h, gain, dh_io, dhb, part, T, d, eps);
    else if constexpr (!LN) norm_bwd_rows_kernel<LN, 4, 8><<<SPK_NORM_BWD_BLOCKS, NT, 0, st>>>(da, h, gain, dh_io, dhb, part, T, d, eps);
}
