// Slice sum of the convolution theorem (Eq. 13 summed over slices, algorithm
// steps 5-6 with the sum taken before the inverse transform):
//   A_b(p) = sum_k G^_{k,b}(p) S^_k(p).
// G^ is real and even in every axis, so it is stored as its non-negative
// octant and each complex product costs two real multiplies.
//
// fused_z (lc_fused_device.h): per column of the y-transformed slices, the
// forward z transform of each slice, the multiply by G^ and the sum over
// slices (in FP64 in the FP32 form) are done in registers; the
// inverse z transform follows and A is written once. Slices left in the
// parity y layout by the half-plane xy pass get their last y radix-2 step on
// the way in, two output columns per input column. The plain forms (FP64,
// plain FP32) run the same pass with plain sums.
//
// This file holds its dispatch over grid sides, the merge of split tiles and
// the FP64 source sums.
#include "lc_fused_device.h"

namespace lc {

// Workgroup: 512 / Q consecutive elements of one (tile, output, band), two per
// lane; each of its Q lane groups adds a share of the parts (eight loads in
// flight at a time) and the first adds the Q sums in order. Q is the smallest
// that leaves a group eight parts or fewer, up to 8: with few parts per tile
// the reduction only adds waiting (192^3, 4 parts: Q = 1 8.9 us, Q = 4 13.6),
// with many the loads of one group come one after another (128^3, 64 parts:
// Q = 1 21.6 us, Q = 4 11.6). The tile and the range of its parts are the
// same for a whole workgroup; found per element, with 64-bit divisions, they
// cost more than the adding (192^3: 23 us).
template <int Q>
__global__ __launch_bounds__(256) void fused_rest_merge_kernel(RestMerge m, ColSet s0, ColSet s1) {
    constexpr int LN = 256 / Q;
    __shared__ float4 red[Q > 1 ? Q - 1 : 1][LN];
    const int per = m.L * m.cpw, chunks = (per + 2 * LN - 1) / (2 * LN);
    int r = blockIdx.x;
    const int ch = r % chunks;
    r /= chunks;
    const int b = r % m.nband;
    r /= m.nband;
    const int o = r % m.no;
    const int64_t i = r / m.no;
    const int lane = threadIdx.x % LN, g = threadIdx.x / LN;
    const int e = ch * 2 * LN + 2 * lane;
    const int64_t U = m.rest * m.kmax, lo = i * m.kmax, hi = lo + m.kmax;
    // workgroups whose range starts inside the tile: w U / P in (lo, hi),
    // i.e. w in [ceil((lo + 1) P / U), ceil(hi P / U))
    const int w0 = (int)(((lo + 1) * m.P + U - 1) / U);
    const int w1 = (int)std::min<int64_t>(m.P, (hi * m.P + U - 1) / U);
    const int64_t tile = fused_slot_tile(m.full + i, s0.n_wgs, m.nrow, m.npb, m.gp);
    const int nq = (w1 - w0 + Q - 1) / Q, qa = w0 + g * nq, qb = w1 < qa + nq ? w1 : qa + nq;
    const bool ok = e < per, sparse = U < m.P;     // (sparse: some ranges are empty)
    const cx<float> *src = m.part + (int64_t)b * m.part_stride + (int64_t)o * per + (ok ? e : 0);
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int w = qa; w < qb; w += 8) {
        float4 t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int ww = w + j;
            const bool on = ww < qb && (!sparse || (int64_t)(ww + 1) * U / m.P > (int64_t)ww * U / m.P);
            t[j] = on ? *(const float4 *)(src + (int64_t)m.no * ww * per) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) v = make_float4(v.x + t[j].x, v.y + t[j].y, v.z + t[j].z, v.w + t[j].w);
    }
    if constexpr (Q > 1) {
        if (g > 0) red[g - 1][lane] = v;
        __syncthreads();
        if (g > 0) return;
#pragma unroll
        for (int q = 0; q < Q - 1; ++q) {
            const float4 u = red[q][lane];
            v = make_float4(v.x + u.x, v.y + u.y, v.z + u.z, v.w + u.w);
        }
    }
    if (!ok) return;
    const bool is_main = tile < s0.n_wgs;
    const ColSet &s = is_main ? s0 : s1;
    const int z = e / m.cpw, c = e % m.cpw;
    const int64_t col = (is_main ? tile : tile - s0.n_wgs) * m.cpw + c;
    const int64_t H = m.L / 2;
    const int64_t obase = is_main ? H * H : H;
    cx<float> *dst = m.acc + (int64_t)b * m.acc_stride + o * obase + col_base(s, col) + (int64_t)z * s.row_stride;
    if (col < s.n_cols) dst[0] = dst[0] + mk(v.x, v.y);
    if (col + 1 < s.n_cols) dst[1] = dst[1] + mk(v.z, v.w);
}

// tab[t] = the workgroup holding the second part of tile t, or -1. With
// two outputs per tile (parity layout: pair tiles, main_k of them main),
// the entries go to the tiles of both output rows, as part slots 2 w + o.
__global__ __launch_bounds__(256) void fused_split_kernel(int *__restrict__ tab, int64_t tiles, int64_t kmax,
                                                          int64_t P, int64_t W, int32_t pair, int64_t main_k) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= tiles) return;
    const int64_t lo = t * kmax;
    const int64_t wc = ((lo + 1) * P + W - 1) / W;      // first workgroup starting after lo
    int v = -1;
    if (wc < P) {
        const int64_t st = wc * W / P;
        if (st > lo && st < lo + kmax) v = (int)wc;
    }
    if (!pair) {
        tab[t] = v;
        return;
    }
    // standard tiles: main rows q < N/2 keep their index, rows q + N/2 are
    // main_k further; nyq tiles follow the 2 main_k main ones, likewise
    const int64_t nyq_k = tiles - main_k;
    const int64_t t0 = t < main_k ? t : 2 * main_k + (t - main_k);
    const int64_t t1 = t0 + (t < main_k ? main_k : nyq_k);
    tab[t0] = v < 0 ? -1 : 2 * v;
    tab[t1] = v < 0 ? -1 : 2 * v + 1;
}

void launch_fused_rest_merge(const RestMerge &m, const ColSet &s0, const ColSet &s1, hipStream_t st) {
    const int64_t parts = (m.P + m.rest - 1) / m.rest, per = (int64_t)m.L * m.cpw;   // parts per tile, its elements
#define RM_(Q)                                                                                                     \
    hipLaunchKernelGGL(fused_rest_merge_kernel<Q>, dim3((unsigned)(m.rest * m.no * m.nband * ((per * Q + 511) / 512))), \
                       dim3(256), 0, st, m, s0, s1)
    if (parts <= 8) RM_(1);
    else if (parts <= 32) RM_(4);
    else RM_(8);
#undef RM_
}

void launch_fused_split(int *tab, int64_t tiles, int64_t kmax, int64_t P, int64_t W, int32_t pair, int64_t main_k,
                        int64_t count, hipStream_t st) {
    hipLaunchKernelGGL(fused_split_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, tab, tiles, kmax, P,
                       W, pair, main_k);
}

// variants: bit 0 selects a prefetch depth of 1 (else 2) slices (fewer
// registers: the two-band instances need it), bit 1 the eight-element
// schedule where one exists (N = 384, 512: the eight-element schedule only,
// bit 0 alone). At N = 128 and 256 the last variant is the lane-exchange kernel.
int fused_variants(int n) { return n == 128 || n == 256 ? 5 : n == 64 || n == 192 ? 4 : 2; }

bool fused_parity_supported(int n) { return n == 192 || n == 256; }

int fused_max_bands(int n) { return (n == 384 || n == 512) ? 4 : 2; }

// Built-in choice: prefetch depth 2 for one band per launch, 1 for two (the
// two-band instances of depth 2 spill registers).
// (N = 128 and 256: the lane-exchange kernel; two bands at 128 the
// eight-element schedule of depth 1, 68.5 us for 24 slices against 71.)
int fused_default_variant(int n, int nband) {
    if (n == 256) return 4;
    if (n == 96) return 1;    // (depth 1: both halves of every tile fit, see fused_go; 24 slices 68 -> 49 us)
    if (n == 128) return nband > 1 ? 3 : 4;
    if (n == 384) return 1;   // depth 1 is the instance without spills there
    const int s8 = fused_variants(n) > 2 ? 2 : 0;
    return s8 + (nband > 1 ? 1 : 0);
}

static hipError_t fused_dispatch(int n, FusedForm form, const FusedArgs &a, const void *tw_full, hipStream_t st) {
    switch (n) {
        case 128: return fused_set_launch<1>(n, form, a, tw_full, st);
        case 192: return fused_set_launch<2>(n, form, a, tw_full, st);
        case 256: return fused_set_launch<3>(n, form, a, tw_full, st);
        case 384: return fused_set_launch<4>(n, form, a, tw_full, st);
        case 512: return fused_set_launch<5>(n, form, a, tw_full, st);
        default: return fused_set_launch<0>(n, form, a, tw_full, st);
    }
}

hipError_t launch_fused_z(int n, const FusedArgs &a, const void *tw_full, hipStream_t st) {
    if (a.nband < 1 || a.nband > 4) return hipErrorInvalidValue;
    return fused_dispatch(n, FusedForm::fp32, a, tw_full, st);
}

hipError_t launch_fused_plain(int n, bool t_f64, const FusedArgs &a, const void *tw_full, hipStream_t st) {
    if (a.nband < 1 || a.nband > 2) return hipErrorInvalidValue;
    return fused_dispatch(n, t_f64 ? FusedForm::plain64 : FusedForm::plain32, a, tw_full, st);
}

// ---------------------------------------------------------------------------
// FP64 mean (DC) of each band: mu_b = sum_k G^_{k,b}(0) S^_k(0) / N^3
// Stage 1: one workgroup per slice sums that slice's per-workgroup FP64
// partials of the forward x pass (fixed order: deterministic).
// Stage 2: one workgroup forms mu_b from the slice sums.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void dc_slice_kernel(const double *__restrict__ dcpart, int W,
                                                       double *__restrict__ sk, int *__restrict__ status,
                                                       int ring, int K) {
    __shared__ double red[4];
    const int k = blockIdx.x;
    double s = 0.0;
    for (int w = threadIdx.x; w < W; w += 256) s += dcpart[(int64_t)k * W + w];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        s = red[0] + red[1] + red[2] + red[3];
        sk[k] = s;
        // a NaN or infinite source value makes its slice's FP64 sum non-finite
        if (status && !isfinite(s)) {
            atomicAdd(&status[0], 1);
            atomicMin(&status[1], k >= ring ? k - ring : k - ring + K);
        }
    }
}

// One wave per slice: the (0, 0) value of every z-plane.
template <typename T>
__global__ __launch_bounds__(64) void spec_dc_kernel(const cx<T> *__restrict__ spec, int64_t stride, int n,
                                                     int64_t plane, int64_t odd, int K, double *__restrict__ sk,
                                                     int *__restrict__ status, int ring) {
    const int k = blockIdx.x;
    double v = 0.0;
    for (int z = threadIdx.x; z < n; z += 64) {
        const cx<T> *row = spec + (int64_t)k * stride + z * plane;
        v += (double)row[0].x + (odd ? (double)row[odd].x : 0.0);
    }
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if (threadIdx.x != 0) return;
    sk[k] = v;
    if (!isfinite(v)) {
        atomicAdd(&status[0], 1);
        atomicMin(&status[1], k >= ring ? k - ring : k - ring + K);
    }
}

hipError_t launch_spec_dc(int n, const void *spec, bool f64, bool parity, int64_t stride, int K, double *sk,
                          int *status, int ring, hipStream_t st) {
    if (K < 1 || ring < 0 || ring >= K) return hipErrorInvalidValue;
    const int64_t plane = (int64_t)n * (n / 2), odd = parity ? plane / 2 : 0;
    if (f64)
        hipLaunchKernelGGL(spec_dc_kernel<double>, dim3(K), dim3(64), 0, st, (const cx<double> *)spec, stride, n, plane,
                           odd, K, sk, status, ring);
    else
        hipLaunchKernelGGL(spec_dc_kernel<float>, dim3(K), dim3(64), 0, st, (const cx<float> *)spec, stride, n, plane,
                           odd, K, sk, status, ring);
    return hipGetLastError();
}

hipError_t launch_dc_reduce(const double *dcpart, int K, int W, double *sk, int *status, int ring,
                            hipStream_t st) {
    if (K < 1 || W < 1 || ring < 0 || ring >= K) return hipErrorInvalidValue;
    hipLaunchKernelGGL(dc_slice_kernel, dim3(K), dim3(256), 0, st, dcpart, W, sk, status, ring, K);
    return hipGetLastError();
}

}  // namespace lc
