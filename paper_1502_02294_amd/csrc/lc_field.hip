// Slice sum of the convolution theorem (Eq. 13 summed over slices, algorithm
// steps 5-6 with the sum taken before the inverse transform):
//   A_b(p) = sum_k G^_{k,b}(p) S^_k(p).
// G^ is real and even in every axis, so it is stored as its non-negative
// octant and each complex product costs two real multiplies.
//
// fused_z (lc_fused_device.h): per column of the y-transformed slices, the
// forward z transform of each slice, the multiply by G^ and the sum over
// slices (compensated, Kahan, in the FP32 form) are done in registers; the
// inverse z transform follows and A is written once. Slices left in the
// parity y layout by the half-plane xy pass get their last y radix-2 step on
// the way in, two output columns per input column. The plain forms (FP64,
// plain FP32) run the same pass with plain sums.
//
// This file holds its dispatch over grid sides, the merge of split tiles and
// the FP64 source sums.
#include "lc_fused_device.h"

namespace lc {

// Workgroup: 64 consecutive elements of one (tile, output, band); its four
// waves sum a quarter of the parts each (eight loads in flight at a time)
// and wave 0 adds the four partial sums in wave order.
__global__ __launch_bounds__(256) void fused_rest_merge_kernel(RestMerge m, ColSet s0, ColSet s1) {
    __shared__ cx<float> red[3][64];
    const int64_t per = (int64_t)m.L * m.cpw;
    const int64_t chunks = (per + 63) / 64;
    const int64_t g = blockIdx.x;
    const int64_t ch = g % chunks;
    int64_t r = g / chunks;
    const int b = (int)(r % m.nband);
    r /= m.nband;
    const int o = (int)(r % m.no);
    const int64_t i = r / m.no;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t e = ch * 64 + lane;
    const bool ok_e = e < per;
    const int64_t U = m.rest * m.kmax, lo = i * m.kmax, hi = lo + m.kmax;
    // workgroups whose range starts inside the tile: w U / P in (lo, hi),
    // i.e. w in [ceil((lo + 1) P / U), ceil(hi P / U))
    const int64_t w0 = ((lo + 1) * m.P + U - 1) / U;
    const int64_t w1 = std::min<int64_t>(m.P, (hi * m.P + U - 1) / U);
    const int64_t nq = (w1 - w0 + 3) / 4;
    const int64_t qa = w0 + wv * nq, qb = std::min<int64_t>(w1, qa + nq);
    const cx<float> *src = m.part + (int64_t)b * m.part_stride + o * per + (ok_e ? e : 0);
    cx<float> v = mk(0.f, 0.f);
    for (int64_t w = qa; w < qb; w += 8) {
        cx<float> t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t ww = w + j;
            const bool on = ok_e && ww < qb && (ww + 1) * U / m.P > ww * U / m.P;   // non-empty range
            t[j] = on ? src[m.no * ww * per] : mk(0.f, 0.f);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) v = v + t[j];
    }
    if (wv > 0) red[wv - 1][lane] = v;
    __syncthreads();
    if (wv > 0 || !ok_e) return;
    v = v + red[0][lane];
    v = v + red[1][lane];
    v = v + red[2][lane];
    const int z = (int)(e / m.cpw), c = (int)(e % m.cpw);
    const int64_t tile = fused_slot_tile(m.full + i, s0.n_wgs, m.nrow, m.npb, m.gp);
    const bool is_main = tile < s0.n_wgs;
    const ColSet &s = is_main ? s0 : s1;
    const int64_t col = (is_main ? tile : tile - s0.n_wgs) * m.cpw + c;
    if (col >= s.n_cols) return;
    const int64_t H = m.L / 2;
    const int64_t obase = is_main ? H * H : H;
    cx<float> *dst = m.acc + (int64_t)b * m.acc_stride + o * obase + col_base(s, col) + (int64_t)z * s.row_stride;
    *dst = *dst + v;
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
    const int64_t wgs = m.rest * m.no * m.nband * (((int64_t)m.L * m.cpw + 63) / 64);
    hipLaunchKernelGGL(fused_rest_merge_kernel, dim3((unsigned)wgs), dim3(256), 0, st, m, s0, s1);
}

void launch_fused_split(int *tab, int64_t tiles, int64_t kmax, int64_t P, int64_t W, int32_t pair, int64_t main_k,
                        int64_t count, hipStream_t st) {
    hipLaunchKernelGGL(fused_split_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, tab, tiles, kmax, P,
                       W, pair, main_k);
}

// variants: bit 0 selects a prefetch depth of 1 (else 2) slices (fewer
// registers: the two-band instances need it), bit 1 the eight-element
// schedule where one exists (N = 384, 512: the eight-element schedule only,
// bit 0 alone)
int fused_variants(int n) {
    return (n == 384 || n == 512) ? 2 : (n == 64 || n == 128 || n == 192 || n == 256) ? 4 : 2;
}

bool fused_parity_supported(int n) { return n == 192 || n == 256; }

int fused_max_bands(int n) { return (n == 384 || n == 512) ? 4 : 2; }

// Built-in choice: prefetch depth 2 for one band per launch, 1 for two (the
// two-band instances of depth 2 spill registers).
int fused_default_variant(int n, int nband) {
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
    __shared__ double red[256];
    const int k = blockIdx.x;
    double s = 0.0;
    for (int w = threadIdx.x; w < W; w += 256) s += dcpart[(int64_t)k * W + w];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        sk[k] = red[0];
        // a NaN or infinite source value makes its slice's FP64 sum non-finite
        if (status && !isfinite(red[0])) {
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
