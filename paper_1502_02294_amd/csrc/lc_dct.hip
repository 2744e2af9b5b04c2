// Cosine transforms of the kernel octant (algorithm step 3): the FP64 spectrum
// of a real even grid from its non-negative octant.
//
// A line holds x[0 .. N/2] of a real even sequence of period N; its DFT is
// real and even, X[0 .. N/2]. The line is read as the N/2 complex values
// z[j] = x[2j] + i x[2j+1] (indices past N/2 read their mirror), transformed by
// the N/2-point engine and untangled as a real row is (real parts only). The
// octant has (N/2 + 1)^3 cells, an eighth of the grid, so against the full
// real-to-complex transform of the mirrored grid a slice moves about a
// twelfth of the bytes; a batch of slices goes through one launch per axis.
// HBM bound: 2 (N/2 + 1)^3 8 bytes per slice and axis. At 128^3 a slice takes
// 4.9 us for the three axes and the store, against 53 us for the x, y and z
// passes of the mirrored grid and the fold of its complex spectrum.
//   AXIS 2: contiguous lines, lanes along the line (in place)
//   AXIS 1: lines of stride H = N/2 + 1, lanes along the H columns (in place)
//   AXIS 0: lines of stride H^2; the transformed values go straight to the
//           plan's octant store (TO, main [r][q][p < N/2] then p = N/2 as
//           [r][q]), scaled for the conserve option, G^(0) to dc
#include "lc_fft_device.h"
#include "lc_greens.h"
#include "lc_internal.h"

namespace lc {

template <int N> struct DctShape {
    static constexpr int L = N / 2, H = N / 2 + 1;
    static constexpr int TPL = Sched<L>::TPL;
    static constexpr int CPW = 16 * TPL >= 64 ? 16 : 64 / TPL;   // lines per workgroup
    static constexpr int NT = CPW * TPL;
    static constexpr int SK = 4;
    static constexpr int LS = L + (L >> SK) + 1;                 // line stride, contiguous lines
    static constexpr int ES = CPW + 1;                           // element stride, strided lines
};

template <int N, int AXIS, typename TO>
__global__ __launch_bounds__(DctShape<N>::NT) void dct_kernel(double *__restrict__ g0, int64_t n_lines,
                                                              const cx<double> *__restrict__ tw_g,
                                                              const cx<double> *__restrict__ twist_g, DctStore out) {
    using SH = DctShape<N>;
    constexpr int L = SH::L, H = SH::H, TPL = SH::TPL, CPW = SH::CPW, NT = SH::NT;
    constexpr bool ROW = AXIS == 2;
    constexpr int SK = ROW ? SH::SK : 31;
    constexpr int ES = ROW ? 1 : SH::ES;
    constexpr int64_t H2 = (int64_t)H * H;
    using EN = Engine<double, L, true, Sched<L>, SK>;
    constexpr int E = EN::E;
    __shared__ cx<double> lds[ROW ? CPW * SH::LS : L * SH::ES];
    __shared__ cx<double> tws[L], twst[L];
    for (int i = threadIdx.x; i < L; i += NT) {
        tws[i] = tw_g[i];
        twst[i] = twist_g[i];
    }
    const int c = ROW ? (int)threadIdx.x / TPL : (int)threadIdx.x % CPW;
    const int t = ROW ? (int)threadIdx.x % TPL : (int)threadIdx.x / CPW;
    const int64_t line = (int64_t)blockIdx.x * CPW + c;
    const bool ok = line < n_lines;
    const int64_t ln = ok ? line : 0;
    const int64_t b = ln / H2, f = ln % H2;   // slice of the batch, line of the slice
    const int64_t base = b * H2 * H + (AXIS == 2 ? f * H : AXIS == 1 ? (f / H) * H2 + f % H : f);
    constexpr int64_t stride = AXIS == 2 ? 1 : AXIS == 1 ? H : H2;
    const double *__restrict__ src = g0 + base;
    cx<double> x[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i0 = 2 * EN::in_pos(t, e), i1 = i0 + 1;
        x[e] = mk(src[(i0 <= L ? i0 : N - i0) * stride], src[(i1 <= L ? i1 : N - i1) * stride]);
    }
    const int lb = ROW ? c * SH::LS : c;
    EN::run(x, lds, lb, ES, t, tws);
    lds_barrier();
#pragma unroll
    for (int e = 0; e < E; ++e) lds[lb + lpos<SK>(EN::out_pos(t, e)) * ES] = x[e];
    lds_barrier();
    if (!ok) return;
    double f_scale = 1.0;
    int64_t k = 0;
    if constexpr (AXIS == 0) {
        k = out.k0 + b;
        if (out.target_over_l3[b] >= 0.0) f_scale = out.target_over_l3[b] / out.g00[k];
    }
    auto put = [&](int p, double v) {
        if constexpr (AXIS != 0) {
            g0[base + p * stride] = v;
        } else {
            TO *oct = (TO *)out.oct + (k * out.B + out.band) * (H2 * H);
            const int q = (int)(f / H), pp = (int)(f % H);
            const int64_t o = pp < L ? ((int64_t)p * H + q) * L + pp : H2 * L + (int64_t)p * H + q;
            oct[o] = (TO)(v * f_scale);
            if (f == 0 && p == 0) out.dc[k * out.B + out.band] = v * f_scale;
        }
    };
    for (int p = t; p <= L / 2; p += TPL) {
        const cx<double> A = lds[lb + lpos<SK>(p) * ES], B = lds[lb + lpos<SK>((L - p) % L) * ES];
        // E = (A + conj B) / 2, O = (A - conj B) / (2i), X[p] = E + W^p O, X[L-p] = conj(E - W^p O)
        const double ev = 0.5 * (A.x + B.x), ox = 0.5 * (A.y + B.y), oy = 0.5 * (B.x - A.x);
        const cx<double> w = twst[p];
        const double d = w.x * ox - w.y * oy;
        put(p, ev + d);
        if (p != L - p) put(L - p, ev - d);
    }
}

// G^(0) of each slice of the batch before scaling (the conserve option): the
// axis-0 line of column 0 after the other two axes' transforms.
__global__ __launch_bounds__(64) void dct_g00_kernel(const double *__restrict__ g0, int H, double *__restrict__ g00) {
    const int64_t H2 = (int64_t)H * H;
    const double *src = g0 + (int64_t)blockIdx.x * H2 * H;
    double v = 0.0;
    for (int i = threadIdx.x; i < H; i += 64) v += (i == 0 || i == H - 1 ? 1.0 : 2.0) * src[i * H2];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if (threadIdx.x == 0) g00[blockIdx.x] = v;
}

template <int N>
static hipError_t dct_t(double *oct, int count, const void *tw, const void *twist, const DctStore &out, bool oct_f64,
                        hipStream_t st) {
    using SH = DctShape<N>;
    const int64_t lines = (int64_t)count * SH::H * SH::H;
    const dim3 grid((unsigned)((lines + SH::CPW - 1) / SH::CPW)), blk(SH::NT);
    const cx<double> *t = (const cx<double> *)tw, *ts = (const cx<double> *)twist;
    hipLaunchKernelGGL((dct_kernel<N, 2, double>), grid, blk, 0, st, oct, lines, t, ts, out);
    hipLaunchKernelGGL((dct_kernel<N, 1, double>), grid, blk, 0, st, oct, lines, t, ts, out);
    if (out.conserve)
        hipLaunchKernelGGL(dct_g00_kernel, dim3((unsigned)count), dim3(64), 0, st, oct, SH::H, out.g00 + out.k0);
    if (oct_f64)
        hipLaunchKernelGGL((dct_kernel<N, 0, double>), grid, blk, 0, st, oct, lines, t, ts, out);
    else
        hipLaunchKernelGGL((dct_kernel<N, 0, float>), grid, blk, 0, st, oct, lines, t, ts, out);
    return hipGetLastError();
}

hipError_t launch_greens_dct(int n, double *oct, int count, const void *tw64_half, const void *twist64,
                             const DctStore &out, bool oct_f64, hipStream_t st) {
    if (count < 1 || count > ShellArgs::kMax) return hipErrorInvalidValue;
    switch (n) {
#define X_(N) case N: return dct_t<N>(oct, count, tw64_half, twist64, out, oct_f64, st);
        X_(8) X_(12) X_(16) X_(24) X_(32) X_(48) X_(64) X_(96) X_(128) X_(192) X_(256) X_(384) X_(512)
#undef X_
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lc
