// Device code and launch templates of the fused z pass (slice sum of the
// convolution theorem): see lc_field.hip for what it computes. Included by
// the units of lc_fused.hip, one per group of grid sides.
#pragma once

#include <algorithm>
#include <type_traits>

#include "lc_fft_device.h"
#include "lc_internal.h"

namespace lc {

__device__ __forceinline__ float fma_(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ int fold(int v, int n) { return v <= n / 2 ? v : n - v; }

// ---------------------------------------------------------------------------
// fused z pass, persistent with a balanced ("stream-K") partition
//
// The work is the sequence of (tile, slice) pairs, tile-major; tile t covers
// CPW columns and its slices k < kmax. Workgroup w of P takes the pairs
// [w W / P, (w+1) W / P), W = tiles * kmax, so every workgroup gets the same
// number of slice-tiles up to one. Since W / P >= kmax, a tile is split
// between at most two workgroups: the part starting at k = 0 is written to
// the accumulator spectrum, the other part (starting at an interior k) to a
// side buffer slot owned by the workgroup that computed it; the inverse y
// pass adds it back when it loads the tile.
// ---------------------------------------------------------------------------
template <typename T> struct FusedDev {
    const cx<T> *spec;
    int64_t spec_stride;
    const T *ghat;
    int64_t oct_stride;
    int32_t B, band0, nb;       // bands in the G^ layout, first handled band, handled bands
    int32_t Kc[4];              // kcount of the handled bands (0 past nb)
    cx<T> *acc;
    int64_t acc_stride;
    cx<T> *part;                // [band][P][L * CPW]
    int64_t part_stride;
    int32_t zero_dc;
    int32_t kmax, P;
    int64_t W;
    int32_t rounds;            // 1: whole tiles w, w+P, ... (no split tiles)
    int64_t tiles;
    const double *sk, *g0;     // band means (mu non-null): see FusedArgs
    double inv_n3;
    double *mu;
    int32_t K;
    int32_t ring;              // lookback k lives in spectrum slot (k + ring) mod K
    int32_t frozen;            // >= 0: every lookback slice reads slot `frozen` (instantaneous field)
};

// a complex value of a slice spectrum, with a non-temporal load for NT
template <bool NT, typename T> __device__ __forceinline__ cx<T> ld_spec(const char *p) {
    if constexpr (NT) {
        typedef T v2 __attribute__((ext_vector_type(2)));
        const v2 v = __builtin_nontemporal_load((const v2 *)p);
        return mk(v[0], v[1]);
    } else {
        return *(const cx<T> *)p;
    }
}

// p-blocks of CPW columns whose octant rows share a 128-byte line
__host__ __device__ constexpr int fused_gp(int cpw, int tsize) {
    return cpw * tsize >= 128 ? 1 : 128 / (cpw * tsize);
}

// Processing order of the main tiles in the rounds schedule. Main tile
// q*NPB + pb covers columns p in [pb*CPW, (pb+1)*CPW) of row q (NPB tiles
// per row). Its kernel octant rows (folded q) are CPW floats, so GP =
// 32 / CPW neighbouring p-blocks share each 128-byte octant line, and the
// rows q and q' = N - q (0 <-> N/2) fold to the same octant row: the 2*GP
// tiles {q, q'} x {GP p-blocks} read the same octant lines (and, for
// CPW < 16, the same spectrum lines). Workgroups w, w+8, w+16, ... run on
// one XCD (workgroups are dispatched to the 8 XCDs in turn), so slot s of
// a block of 16*GP consecutive slots takes member (s % (16 GP)) / 8 of
// group 8 * (s / (16 GP)) + s % 8: the readers of a line are resident
// together on one XCD and it comes from that XCD's L2 once. The p-blocks
// rotate by row, or one XCD would read the same 256 bytes of every row
// (256^3: 741 us against 757; 192^3: 177 against 182). Other tile
// counts, and tiles that do not split rows evenly (npb = 0), keep the
// identity order; the result is always a main tile when slot is one.
// With spectra in the parity layout, a tile covers rows q and q + N/2
// (q < N/2) and the same pairing runs with N/2 in place of N: the octant
// rows of tiles q and N/2 - q are {q, N/2 - q} for both.
__device__ __forceinline__ int64_t fused_slot_tile(int64_t slot, int64_t main_tiles, int n, int npb, int gp) {
    const int bs = 16 * gp;
    if (slot >= main_tiles || gp < 1 || npb < gp || npb % gp || main_tiles % bs ||
        (int64_t)n * npb != main_tiles)
        return slot;
    const int64_t blk = slot / bs;
    const int xcd = (int)(slot & 7), j = (int)((slot % bs) >> 3);
    const int64_t g = blk * 8 + xcd;
    const int ngp = npb / gp;
    const int q = (int)(g / ngp), pb = gp * (int)((g + q) % ngp) + (j % gp);
    const int row = j < gp ? q : (q == 0 ? n / 2 : n - q);
    const int64_t tile = (int64_t)row * npb + pb;
    return tile < main_tiles ? tile : slot;
}

// The tiles and slices of workgroup w, as segment(tile, first slice, end).
// rounds = 2 (few tiles): workgroup w takes a half of the slices of tile
// w mod tiles, the first or the second.
template <int L, int CPW, bool PAR, typename T, typename F>
__device__ __forceinline__ void fused_walk(const FusedDev<T> &a, const ColSet &s0, int w, F &&segment) {
    if (a.rounds == 2) {
        const int npb = (L / 2) % CPW == 0 ? (int)((L / 2) / CPW) : 0;
        const int half = w >= (int)a.tiles ? 1 : 0, mid = a.kmax / 2;
        const int64_t tile = fused_slot_tile(half ? w - a.tiles : w, s0.n_wgs, PAR ? L / 2 : L, npb,
                                             fused_gp(CPW, sizeof(T)));
        segment(tile, half ? mid : 0, half ? a.kmax : mid);
    } else if (a.rounds) {
        // whole tiles in rounds: all workgroups sweep the slices together
        // main tiles per row (0: rows do not split into whole tiles, identity order)
        const int npb = (L / 2) % CPW == 0 ? (int)((L / 2) / CPW) : 0;
        constexpr int GP = fused_gp(CPW, sizeof(T));
        const int nrow = PAR ? L / 2 : L;
        const int64_t full = a.tiles / a.P * a.P;   // slots of the whole rounds
        for (int64_t slot = w; slot < full; slot += a.P)
            segment(fused_slot_tile(slot, s0.n_wgs, nrow, npb, GP), 0, a.kmax);
        // the tiles of the remaining slots (fewer than P) would leave most
        // workgroups idle for a whole round: their (tile, slice) pairs are
        // split evenly over all workgroups instead. Only a workgroup's first
        // segment can start inside a tile; it goes to the workgroup's part
        // slot, and fused_rest_merge_kernel adds the parts of each tile.
        const int64_t U = (a.tiles - full) * a.kmax;
        int64_t u = (int64_t)w * U / a.P;
        const int64_t ue = (int64_t)(w + 1) * U / a.P;
        while (u < ue) {
            const int64_t i = u / a.kmax;
            const int k0 = (int)(u % a.kmax);
            const int k1 = (int)std::min<int64_t>(a.kmax, k0 + (ue - u));
            u += k1 - k0;
            segment(fused_slot_tile(full + i, s0.n_wgs, nrow, npb, GP), k0, k1);
        }
    } else {
        int64_t pos = (int64_t)w * a.W / a.P;
        const int64_t end = (int64_t)(w + 1) * a.W / a.P;
        while (pos < end) {
            const int64_t tile = pos / a.kmax;
            const int k0 = (int)(pos % a.kmax);
            const int k1 = (int)std::min<int64_t>(a.kmax, k0 + (end - pos));
            pos += k1 - k0;
            segment(tile, k0, k1);
        }
    }
}

// PAR: the slice spectra are in the parity layout of the half-plane xy
// shapes (rows r < N/2 of a z-plane hold the y transform E of the even rows,
// rows N/2 + r that of the odd rows O). A column (q, p) with q < N/2 then
// yields the two columns of rows q and q + N/2 of the length-N y transform,
//   T[q] = E + W_N^q O,   T[q + N/2] = E - W_N^q O
// (its last radix-2 step), formed on the way to the first butterfly: each
// input element is read once for both, and both go through the z transform,
// the kernel product and the sum. Output o of a column is at
// o * (N/2 rows) after the first; a second part goes to part slot 2 w + o.
// NTL: the spectra are read with non-temporal loads.
// KS: sums in FP64 (the FP32 form with one or two bands per launch; three or
// four bands sum in FP32: their sums would not fit in registers otherwise). A
// product and sum is a conversion and one FP64 instruction per value, where a
// compensated FP32 sum in as many registers takes four (one band of 24 slices
// of 64^3 24.3 -> 23.1 us, two of 21 slices of 96^3 65 -> 61.5), and the
// sum's error is that of its inputs. The plain forms (T = double, or float) sum
// in T in the order of the slices.
template <typename T, int L, int NB_, typename S, int PF, int IN, bool KS, bool NTL = false>
__global__ __launch_bounds__((FusedShape<T, L, S>::NT)) void fused_z_kernel(FusedDev<T> a, ColSet s0, ColSet s1,
                                                                           const cx<T> *__restrict__ tw_g) {
    // input: 0 y-transformed slices, 1 the same in the parity layout, 2
    // slices already transformed along z as well (3D spectra: no forward z
    // transform here, the slice loop is the product and the sum)
    constexpr bool PAR = IN == 1, PRE = IN == 2;
    using SH = FusedShape<T, L, S>;
    using EF = Engine<T, L, true, S>;     // forward z transform
    using EI = Engine<T, L, false, S>;    // inverse z transform
    constexpr int CPW = SH::CPW, NT = SH::NT, ES = CPW + SH::PAD, E = EF::E;
    static_assert(EI::E == E, "forward and inverse hold the same elements");
    constexpr int HP = L / 2 + 1;
    constexpr int RSTEP = NT / CPW;                        // = threads per column
    constexpr int GROWS = (HP + RSTEP - 1) / RSTEP;        // octant rows loaded per thread
    constexpr int NO = PAR ? 2 : 1;                        // output columns per input column
        constexpr int CB = sizeof(cx<T>);                      // bytes of a complex value
    // FP64 lines are twice as wide: one line buffer (a barrier more per
    // exchange) leaves room for a second workgroup on the CU
    constexpr bool DB = sizeof(T) == 4;
    // pair tiles of one band: the two outputs' transforms run interleaved
    // (Engine::first2_db / rest2_db), two barriers per slice instead of four
    constexpr bool IL = PAR && NB_ == 1 && EF::NP > 1 && sizeof(T) == 4;
    // z transform line buffers, alternated by exchange (Engine::run_db):
    // only the barriers after the writes remain in the slice loop; lds3 and
    // lds4 are the second output's pair in the interleaved form
    __shared__ cx<T> lds[L * ES], lds2[DB ? L * ES : 1];
    __shared__ cx<T> lds3[IL ? L * ES : 1], lds4[IL ? L * ES : 1];
    __shared__ cx<T> tws[L];
    // kernel octant rows of the tile (all folded z frequencies), per output:
    // rows r and L-r of a column share one entry. Double buffered by slice;
    // one buffer in the interleaved form, which stores slice k's rows after
    // the first barrier of slice k (every reader of slice k-1's rows has
    // passed it) and reads them after the second.
    constexpr int GB = IL ? 1 : 2;
    __shared__ T gl[GB][NB_ * NO][HP * CPW];
    for (int i = threadIdx.x; i < L; i += NT) tws[i] = tw_g[i];
    // the FP64 band means (DC mode), once per launch, by the first wave of
    // workgroup 0: mu_b = inv_n3 sum_k G^_{k,b}(0) S^_k(0)
    if (a.mu && blockIdx.x == 0 && threadIdx.x < 64) {
#pragma unroll
        for (int b = 0; b < NB_; ++b) {
            if (b >= a.nb) break;
            double v = 0.0;
            for (int k = threadIdx.x; k < a.K; k += 64) {
                const int slot = a.frozen >= 0 ? a.frozen : (k + a.ring < a.K ? k + a.ring : k + a.ring - a.K);
                v += a.g0[(int64_t)k * a.B + a.band0 + b] * a.sk[slot];
            }
            for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
            if (threadIdx.x == 0) a.mu[a.band0 + b] = v * a.inv_n3;
        }
    }

    const int c = threadIdx.x % CPW, t = threadIdx.x / CPW;
    const int H = L / 2;
    const int w = blockIdx.x;

    auto segment = [&](const int64_t tile, const int k0, const int k1) {

        // readers of the LDS buffers in the previous segment are done
        lds_barrier();
        const bool is_main = tile < s0.n_wgs;
        const ColSet &s = is_main ? s0 : s1;
        const int64_t col0 = (is_main ? tile : tile - s0.n_wgs) * CPW;
        const int64_t col = col0 + c;
        const bool col_ok = col < s.n_cols;
        // columns past the end compute on a valid column and are not stored
        const int64_t ccol = col_ok ? col : col0;
        const int64_t cbase = col_base(s, ccol);
        // row (y frequency) of the column; in the parity layout the second
        // output and the O input are obase elements further
        const int q = is_main ? (int)(ccol / H) : (int)ccol;
        const int64_t obase = is_main ? (int64_t)H * H : (int64_t)H;
        const cx<T> wq = tws[PAR ? q : 0];   // W_N^q

        // octant offset of this thread's column in one G^ slice; the row
        // part (folded z frequency) is added per element. The second output
        // (row q + N/2) is gdel floats further.
        int gbase, grow, gdel = 0;
        if (is_main) {
            const int cc = (int)ccol;
            gbase = fold(q, L) * H + cc % H;
            grow = HP * H;
            if constexpr (PAR) gdel = (fold(q + H, L) - fold(q, L)) * H;
        } else {
            gbase = HP * HP * H + fold(q, L);
            grow = HP;
            if constexpr (PAR) gdel = fold(q + H, L) - fold(q, L);
        }

        using A = std::conditional_t<KS, double, T>;
        cx<A> sum[NO][NB_][E];
#pragma unroll
        for (int o = 0; o < NO; ++o)
#pragma unroll
            for (int b = 0; b < NB_; ++b)
#pragma unroll
                for (int e = 0; e < E; ++e) sum[o][b][e] = mk((A)0, (A)0);

        // Byte offsets, off workgroup-uniform bases (a slice spectrum is below
        // 4 GiB): of this thread's first input element, the others being whole
        // rows further (compile-time row deltas, folded into the uniform base),
        // and of the kernel octant rows it loads (rows t + j*RSTEP of its
        // column: uniform deltas too, except the last row, which is clamped
        // for the threads past the octant's end). One offset register each
        // instead of one per element.
        // (3D spectra are read at the forward transform's output positions,
        // from the tile order their z pass writes: the tile's rows of w
        // columns contiguous, w = CPW except in a set's last tile)
        auto rowpos = [&](int e) { return PRE ? EF::out_pos(t, e) : EF::in_pos(t, e); };
        int64_t in0 = cbase, in_rs = s.row_stride;
        if constexpr (PRE) {
            const int64_t w = s.n_cols - col0 < CPW ? s.n_cols - col0 : CPW;
            in0 = (is_main ? 0 : spec_main(L)) + col0 * L + (ccol - col0);
            in_rs = w;
        }
        const uint32_t xoff0 = (uint32_t)((in0 + (int64_t)rowpos(0) * in_rs) * CB);
        const int64_t rsb = in_rs * CB;
        auto xld = [&](const char *base, int e) {
            return ld_spec<NTL, T>(base + (int64_t)(rowpos(e) - rowpos(0)) * rsb + xoff0);
        };
        constexpr bool GFULL = GROWS * RSTEP <= HP;   // every thread's last row exists
        const int rlast = t + (GROWS - 1) * RSTEP;
        const uint32_t goff0 = (uint32_t)((gbase + t * grow) * (int)sizeof(T));
        const uint32_t goffl = (uint32_t)((gbase + (rlast < HP ? rlast : 0) * grow) * (int)sizeof(T));
        const int64_t grb = (int64_t)grow * (int64_t)sizeof(T) * RSTEP;
        // LDS slot of each output element's kernel value (folded row)
        int gslot[E];
#pragma unroll
        for (int e = 0; e < E; ++e) gslot[e] = fold(EF::out_pos(t, e), L) * CPW + c;

        // The slice loop runs to a multiple of PF with no branch in its body:
        // slices past k1 read slice k1-1 again (valid, recently read memory)
        // with kernel weight 0, which leaves the sum's value
        // unchanged. Branch-free, every wait for a load counts exactly the
        // loads issued after it, so the prefetched slices stay in flight.
        const int kend = k0 + (k1 - k0 + PF - 1) / PF * PF;
        auto spec_at = [&](int k) {
            int slot = (k < k1 ? k : k1 - 1) + a.ring;
            if (slot >= a.K) slot -= a.K;
            if (a.frozen >= 0) slot = a.frozen;
            return (const char *)(a.spec + (int64_t)slot * a.spec_stride);
        };
        // first-pass inputs of the next PF slices, kept in flight in a ring of
        // register buffers (PF slices of HBM latency hidden behind compute);
        // in the parity layout ob holds the O halves
        constexpr int PO = PAR ? PF : 1;
        cx<T> xb[PF][E], ob[PO][E];
        const int64_t obytes = obase * CB;
        auto fill = [&](int j, int k) {
            const char *src = spec_at(k);
#pragma unroll
            for (int e = 0; e < E; ++e) xb[j][e] = xld(src, e);
            if constexpr (PAR) {
                const char *srco = src + obytes;
#pragma unroll
                for (int e = 0; e < E; ++e) ob[j][e] = xld(srco, e);
            }
        };
#pragma unroll
        for (int j = 0; j < PF; ++j) fill(j, k0 + j);
        // kernel octant rows of slice k are loaded one slice ahead into
        // registers and stored to LDS during slice k; a band without a kernel
        // for slice k reads a valid octant with weight 0. The weight is
        // applied at the LDS store, not at the load: arithmetic on the loaded
        // values right away would wait for every load in flight before them,
        // the prefetched slices included.
        T gn[NB_][NO][GROWS], gw[NB_];
        auto load_g = [&](int k) {
#pragma unroll
            for (int b = 0; b < NB_; ++b) {
                const int kc = a.Kc[b];
                const bool on = k < kc && k < k1;
                const int kb = on ? k : 0;
                gw[b] = on ? (T)1 : (T)0;
                // (a band past nb reads the first handled band's octant)
                const int bb = b < a.nb ? b : 0;
                const char *gp = (const char *)(a.ghat + ((int64_t)kb * a.B + a.band0 + bb) * a.oct_stride);
#pragma unroll
                for (int o = 0; o < NO; ++o) {
                    // the second output's rows are gdel floats away (gdel < 0
                    // for q > N/4): the offset is formed in 32 bits, where it
                    // wraps to the true (nonnegative) offset, before the add
                    const uint32_t od = (uint32_t)(o * gdel) * (uint32_t)sizeof(T);
#pragma unroll
                    for (int j = 0; j < GROWS; ++j)
                        gn[b][o][j] = (j < GROWS - 1 || GFULL)
                                          ? *(const T *)(gp + j * grb + (uint32_t)(goff0 + od))
                                          : *(const T *)(gp + (uint32_t)(goffl + od));
                }
            }
        };
        // octant rows of slice k go to LDS buffer k&1, whose previous
        // contents (slice k-2) were last read before the barriers of slice k-1
        auto store_g = [&](int k) {
            T *glk = &gl[(k & 1) % GB][0][0];
#pragma unroll
            for (int b = 0; b < NB_; ++b)
#pragma unroll
                for (int o = 0; o < NO; ++o)
#pragma unroll
                    for (int jj = 0; jj < GROWS; ++jj) {
                        const int rf = t + jj * RSTEP;
                        if (rf < HP) glk[(b * NO + o) * HP * CPW + rf * CPW + c] = gw[b] * gn[b][o][jj];
                    }
        };
        // sum over slices of output o
        auto mac = [&](int o, const T *glk, const cx<T>(&v)[E]) {
#pragma unroll
            for (int b = 0; b < NB_; ++b)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const T gv = glk[(b * NO + o) * HP * CPW + gslot[e]];
                    sum[o][b][e] = mk(fma_((A)gv, (A)v[e].x, sum[o][b][e].x), fma_((A)gv, (A)v[e].y, sum[o][b][e].y));
                }
        };
        load_g(k0);
        if constexpr (IL) {
            for (int kk = k0; kk < kend; kk += PF) {
#pragma unroll
                for (int j = 0; j < PF; ++j) {
                    const int k = kk + j;
                    // last radix-2 step of the y transform: E +- W_N^q O
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const cx<T> x = xb[j][e], y = ob[j][e];
                        const T ux = fma_(wq.x, y.x, -wq.y * y.y), uy = fma_(wq.x, y.y, wq.y * y.x);
                        xb[j][e] = mk(x.x + ux, x.y + uy);
                        ob[j][e] = mk(x.x - ux, x.y - uy);
                    }
                    EF::first2_db(xb[j], ob[j], lds, lds3, c, ES, t);
                    // buffer j is free: refill it with slice k + PF
                    fill(j, k + PF);
                    EF::rest2_db(
                        lds, lds2, lds3, lds4, c, ES, t, tws,
                        [&] {
                            // slice k's octant rows (loaded during slice k - 1),
                            // then slice k + 1's in flight
                            store_g(k);
                            load_g(k + 1);
                        },
                        [&](int o, const cx<T>(&v)[E]) { mac(o, &gl[0][0][0], v); });
                }
            }
        } else if constexpr (PRE) {
            store_g(k0);
            for (int kk = k0; kk < kend; kk += PF) {
#pragma unroll
                for (int j = 0; j < PF; ++j) {
                    const int k = kk + j;
                    const T *glk = &gl[k & 1][0][0];
                    load_g(k + 1);
                    // slice k's octant rows (stored at the end of slice k - 1)
                    // are visible, and every reader of slice k - 1's rows is
                    // done before they are overwritten at the end of this slice
                    lds_barrier();
                    cx<T> v[E];
#pragma unroll
                    for (int e = 0; e < E; ++e) v[e] = xb[j][e];
                    fill(j, k + PF);
                    mac(0, glk, v);
                    store_g(k + 1);
                }
            }
        } else {
            store_g(k0);
            for (int kk = k0; kk < kend; kk += PF) {
#pragma unroll
                for (int j = 0; j < PF; ++j) {
                    const int k = kk + j;
                    const T *glk = &gl[k & 1][0][0];
                    // the next slice's octant rows are in flight during this slice
                    load_g(k + 1);
                    if constexpr (PAR) {
                        // last radix-2 step of the y transform: E +- W_N^q O
#pragma unroll
                        for (int e = 0; e < E; ++e) {
                            const cx<T> x = xb[j][e], y = ob[j][e];
                            const T ux = fma_(wq.x, y.x, -wq.y * y.y), uy = fma_(wq.x, y.y, wq.y * y.x);
                            xb[j][e] = mk(x.x + ux, x.y + uy);
                            ob[j][e] = mk(x.x - ux, x.y - uy);
                        }
                    }
                    if constexpr (DB) EF::first_db(xb[j], lds, c, ES, t);
                    else EF::first(xb[j], lds, c, ES, t);
                    cx<T> v[E];
                    if constexpr (EF::NP == 1) {
#pragma unroll
                        for (int e = 0; e < E; ++e) v[e] = xb[j][e];
                        lds_barrier();    // kernel values in LDS visible
                    }
                    // buffer j is free (both halves once the second output has
                    // entered its transform): refill it with slice k + PF
                    if constexpr (!PAR) fill(j, k + PF);
                    if constexpr (EF::NP > 1) {
                        if constexpr (DB) EF::rest_db(xb[j], v, lds, lds2, c, ES, t, tws);
                        else EF::rest(xb[j], v, lds, c, ES, t, tws);
                    }
                    mac(0, glk, v);
                    if constexpr (PAR) {
                        if constexpr (DB) EF::first_db(ob[j], lds, c, ES, t);
                        else EF::first(ob[j], lds, c, ES, t);
                        if constexpr (EF::NP == 1) {
#pragma unroll
                            for (int e = 0; e < E; ++e) v[e] = ob[j][e];
                        }
                        fill(j, k + PF);
                        if constexpr (EF::NP > 1) {
                            if constexpr (DB) EF::rest_db(ob[j], v, lds, lds2, c, ES, t, tws);
                            else EF::rest(ob[j], v, lds, c, ES, t, tws);
                        }
                        mac(1, glk, v);
                    }
                    // stored at the end of the slice, after the refill loads were
                    // issued, so that waiting for them does not wait for the refill
                    store_g(k + 1);
                }
            }
        }

        // the (0,0,0) bin: row 0 of main column 0
        const bool has_dc = a.zero_dc && is_main && col == 0;
        const bool primary = k0 == 0;
        auto put = [&](int b, int o, const cx<T>(&y)[E]) {
            if (primary) {
                cx<T> *dst = a.acc + (int64_t)b * a.acc_stride + o * obase;
                if (col_ok)
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        dst[(uint32_t)(cbase + (int64_t)EI::out_pos(t, e) * s.row_stride)] = y[e];
            } else {
                cx<T> *dst = a.part + (int64_t)b * a.part_stride + (NO * (a.rounds == 2 ? tile : (int64_t)w) + o) * (L * CPW) + c;
#pragma unroll
                for (int e = 0; e < E; ++e) dst[EI::out_pos(t, e) * CPW] = y[e];
            }
        };
#pragma unroll
        for (int b = 0; b < NB_; ++b) {
            if (b >= a.nb) break;   // (uniform: the barriers below stay matched)
            cx<T> y[NO][E];
#pragma unroll
            for (int o = 0; o < NO; ++o) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    y[o][e] = mk((T)sum[o][b][e].x, (T)sum[o][b][e].y);
                    if (o == 0 && has_dc && EF::out_pos(t, e) == 0) y[o][e] = mk((T)0, (T)0);
                }
                // the last forward pass's placement is the first inverse pass's
                if constexpr (DB) EI::run_db(y[o], lds, lds2, c, ES, t, tws);
                else EI::run(y[o], lds, c, ES, t, tws);
            }
            if constexpr (PAR) {
                // first radix-2 step of the inverse y transform, split by the
                // parity s of the output rows y = 2m + s:
                //   U_0 = T[q] + T[q + N/2],  U_1 = W_N^-q (T[q] - T[q + N/2])
                // (the inverse y pass of rows of parity s is the N/2-point
                // inverse transform of U_s), stored in the places of T[q] and
                // T[q + N/2]
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const cx<T> u = y[0][e], v = y[1][e];
                    const cx<T> d = mk(u.x - v.x, u.y - v.y);
                    y[0][e] = mk(u.x + v.x, u.y + v.y);
                    y[1][e] = mk(fma_(wq.x, d.x, wq.y * d.y), fma_(wq.x, d.y, -wq.y * d.x));   // conj(W^q) d
                }
            }
#pragma unroll
            for (int o = 0; o < NO; ++o) put(b, o, y[o]);
        }
        };
    fused_walk<L, CPW, PAR>(a, s0, w, segment);
}

// ---------------------------------------------------------------------------
// The same pass with one of the z transform's two exchanges between lanes
//
// L = 8 RM 8 (128 and 256 = 8.2.8 and 8.4.8), eight elements per thread.
// Thread t of a column holds the first pass's inputs t + (L/8) r. Its outputs
// r1 = 0..7 sit at positions 8t + r1, and a middle butterfly combines the same
// r1 of the threads t, t + 8, .. (RM of them). With wave w taking the threads
// t = w + NW g (NW waves, g the lane's row of 16, one lane per column), those
// threads are rows of one wave: the exchange is a transpose between registers
// and rows of lanes (v_permlane32_swap, v_permlane16_swap: one instruction per
// 32-bit value and step instead of an LDS write, a barrier and a read). Only
// the exchange before the last pass goes through LDS, so a slice has one
// barrier, and its line buffers alternate by slice. Loads, stores and LDS
// accesses stay whole 128-byte rows.
//
// Kernel values are read straight to the registers that use them (both folds
// of a row, off one offset each), without LDS staging; the transform's
// twiddles stay in registers across slices; the next slice's inputs are in
// flight during the whole of the current one.
//
// With the spectra in cache (the instantaneous field) 256^3 x 40 takes 490 us
// of this pass against 570 for fused_z_kernel, so the instructions no longer
// bound it; streaming them from HBM it takes 741 us against 795 (4.1 TB/s: rows
// of 128 bytes 256 KiB apart; a kernel that only reads them takes 540).
// Two bands: 826 us for 20 slices against 1550, one set of line buffers and no
// spilled prefetch. 128^3 x 24: 49 us against 53 (compute bound, three
// workgroups per CU in both). 512 = 8.8.8 was slower this way (four bands of 12
// slices 4.85 ms against 4.63): its transposes need lanes 8 apart, three
// instructions a value, and four bands' kernel values two loads each.
// ---------------------------------------------------------------------------
template <int L> struct LaneShape {
    static constexpr int RM = L / 64;                       // middle radix
    static constexpr int CPW = 16;                          // columns per workgroup
    static constexpr int TPL = L / 8, NT = CPW * TPL, NW = NT / 64, Q = 8 / RM;
    static_assert(RM == 2 || RM == 4, "L = 128 or 256");
    static_assert(TPL == NW * 4, "a wave holds four threads of each column");
};

// a of the upper half of the lanes (or of the odd rows of 16) and b of the
// lower half (the even rows) change places
template <int LANES> __device__ __forceinline__ void lane_swap(float &a, float &b) {
    const unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
    static_assert(LANES == 16 || LANES == 32, "");
    const auto r = LANES == 32 ? __builtin_amdgcn_permlane32_swap(ua, ub, false, false)
                               : __builtin_amdgcn_permlane16_swap(ua, ub, false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
template <int LANES> __device__ __forceinline__ void lane_swap(cx<float> &a, cx<float> &b) {
    lane_swap<LANES>(a.x, b.x);
    lane_swap<LANES>(a.y, b.y);
}

// A 32-bit offset kept as such: extended where it is added to its uniform base
// it goes into the load instruction; extended ahead of a loop, every load
// forms a 64-bit address of its own (32 instructions and as many registers
// per slice).
__device__ __forceinline__ void keep32(uint32_t &v) { asm volatile("" : "+v"(v)); }

template <int L> struct LaneTw {
    cx<float> mid[8], last[8];   // forward twiddles: middle pass (q, r at q RM + r), last pass (r)
};

template <int L, bool FWD> struct LaneEngine {
    using SH = LaneShape<L>;
    static constexpr int RM = SH::RM, Q = SH::Q, TPL = SH::TPL;
    __device__ __forceinline__ static cx<float> wmul(cx<float> v, cx<float> w) {
        return FWD ? cmul(v, w) : cmul(v, conj(w));
    }
    // Middle butterfly q of the thread is r1(q) = element of its first pass's outputs
    __device__ __forceinline__ static int r1(int g, int q) {
        return RM == 2 ? 4 * (g >> 1) + q : 4 * q + g;
    }
    // position of output 0 of middle butterfly q (output r: 8 r further)
    __device__ __forceinline__ static int mid_pos(int w, int g, int q) {
        const int t0 = RM == 2 ? w + SH::NW * (g & 1) : w;
        return t0 * 8 * RM + r1(g, q);
    }
    // passes 1 and 2 of the line in x, stored to the line buffer
    __device__ __forceinline__ static void first(cx<float> (&x)[8], cx<float> *lds, int w, int g, int c,
                                                 const LaneTw<L> &tw) {
        dft8<FWD>(x);
        cx<float> v[Q][RM];
        if constexpr (RM == 2) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                lane_swap<32>(x[q], x[q + 4]);
                v[q][0] = x[q];
                v[q][1] = x[q + 4];
            }
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                cx<float> *a = x + 4 * q;
                lane_swap<32>(a[0], a[2]);
                lane_swap<32>(a[1], a[3]);
                lane_swap<16>(a[0], a[1]);
                lane_swap<16>(a[2], a[3]);
#pragma unroll
                for (int r = 0; r < 4; ++r) v[q][r] = a[r];
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
#pragma unroll
            for (int r = 1; r < RM; ++r) v[q][r] = wmul(v[q][r], tw.mid[q * RM + r]);
            dft<RM, FWD>(v[q]);
            const int p0 = mid_pos(w, g, q);
#pragma unroll
            for (int r = 0; r < RM; ++r) lds[(p0 + 8 * r) * SH::CPW + c] = v[q][r];
        }
    }
    // last pass: element e is the output at position t + TPL e
    __device__ __forceinline__ static void rest(cx<float> (&y)[8], const cx<float> *lds, int t, int c,
                                                const LaneTw<L> &tw) {
#pragma unroll
        for (int r = 0; r < 8; ++r) y[r] = lds[(t + TPL * r) * SH::CPW + c];
#pragma unroll
        for (int r = 1; r < 8; ++r) y[r] = wmul(y[r], tw.last[r]);
        dft8<FWD>(y);
    }
};

// NT: the spectra are read with non-temporal loads.
template <int L, int NB_, int IN, bool NT_>
__global__ __launch_bounds__((LaneShape<L>::NT)) void fused_lane_kernel(FusedDev<float> a, ColSet s0, ColSet s1,
                                                                        const cx<float> *__restrict__ tw_g) {
    static_assert(IN == 0 || IN == 1, "y-transformed slices, plain or in the parity layout");
    constexpr bool PAR = IN == 1;
    using SH = LaneShape<L>;
    using EF = LaneEngine<L, true>;
    using EI = LaneEngine<L, false>;
    constexpr int CPW = SH::CPW, TPL = SH::TPL, NO = PAR ? 2 : 1, HP = L / 2 + 1, H = L / 2;
    using A = double;   // sums in FP64, as in fused_z_kernel
    __shared__ cx<float> buf[2][NO][L * CPW];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = lane % CPW, g = lane / CPW;
    const int t = w + SH::NW * g;
    const int wg = blockIdx.x;
    LaneTw<L> tw;
#pragma unroll
    for (int q = 0; q < SH::Q; ++q)
#pragma unroll
        for (int r = 0; r < SH::RM; ++r) tw.mid[q * SH::RM + r] = tw_g[EF::r1(g, q) * (L / (8 * SH::RM)) * r];
#pragma unroll
    for (int r = 0; r < 8; ++r) tw.last[r] = tw_g[t * r];
    // the FP64 band means (DC mode), once per launch, by the first wave of
    // workgroup 0: mu_b = inv_n3 sum_k G^_{k,b}(0) S^_k(0)
    if (a.mu && wg == 0 && threadIdx.x < 64) {
#pragma unroll
        for (int b = 0; b < NB_; ++b) {
            if (b >= a.nb) break;
            double v = 0.0;
            for (int k = threadIdx.x; k < a.K; k += 64) {
                const int slot = a.frozen >= 0 ? a.frozen : (k + a.ring < a.K ? k + a.ring : k + a.ring - a.K);
                v += a.g0[(int64_t)k * a.B + a.band0 + b] * a.sk[slot];
            }
            for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
            if (threadIdx.x == 0) a.mu[a.band0 + b] = v * a.inv_n3;
        }
    }

    auto segment = [&](const int64_t tile, const int k0, const int k1) {
        lds_barrier();   // readers of the line buffers in the previous segment are done
        const bool is_main = tile < s0.n_wgs;
        const ColSet &s = is_main ? s0 : s1;
        const int64_t col0 = (is_main ? tile : tile - s0.n_wgs) * CPW;
        const int64_t col = col0 + c;
        const bool col_ok = col < s.n_cols;
        // columns past the end compute on a valid column and are not stored
        const int64_t ccol = col_ok ? col : col0;
        const int64_t cbase = col_base(s, ccol);
        // row (y frequency) of the column; in the parity layout the second
        // output and the O input are obase elements further
        const int q = is_main ? (int)(ccol / H) : (int)ccol;
        const int64_t obase = is_main ? (int64_t)H * H : (int64_t)H;
        const cx<float> wq = PAR ? tw_g[q] : mk(1.f, 0.f);   // W_N^q
        int gbase, grow, gdel = 0;
        if (is_main) {
            const int cc = (int)ccol;
            gbase = fold(q, L) * H + cc % H;
            grow = HP * H;
            if constexpr (PAR) gdel = (fold(q + H, L) - fold(q, L)) * H;
        } else {
            gbase = HP * HP * H + fold(q, L);
            grow = HP;
            if constexpr (PAR) gdel = fold(q + H, L) - fold(q, L);
        }
        cx<A> sum[NO][NB_][8];
#pragma unroll
        for (int o = 0; o < NO; ++o)
#pragma unroll
            for (int b = 0; b < NB_; ++b)
#pragma unroll
                for (int e = 0; e < 8; ++e) sum[o][b][e] = mk((A)0, (A)0);

        // byte offsets off workgroup-uniform bases: element e is e row steps
        // further; the kernel rows fold(t + TPL e) are t + TPL e for e < 4 and
        // H - t - TPL (e - 4) from there
        const uint32_t xoff = (uint32_t)((cbase + (int64_t)t * s.row_stride) * 8);
        const int64_t rsb = s.row_stride * 8 * TPL;
        const uint32_t glo = (uint32_t)((gbase + t * grow) * 4), ghi = (uint32_t)((gbase + (H - t) * grow) * 4);
        const int64_t grb = (int64_t)grow * 4 * TPL;
        const int64_t obytes = obase * 8;
        // Newest-written first: step k of the segment takes slice k0 + k1 - 1 - k,
        // since a forward pass leaves its last slices in the last-level cache
        // (128^3 x 24, 200 MB of spectra: step 157.8 -> 155.0 us; 256^3 x 40
        // unchanged).
        const int ks = k0 + k1 - 1;
        auto spec_at = [&](int k) {
            int slot = (k < k1 ? ks - k : k0) + a.ring;
            if (slot >= a.K) slot -= a.K;
            if (a.frozen >= 0) slot = a.frozen;
            return (const char *)(a.spec + (int64_t)slot * a.spec_stride);
        };
        // inputs of the next slice, in flight during the whole of the current
        // one (slices past the end read the last again)
        cx<float> xn[NO][8];
        auto fill = [&](int k) {
            const char *src = spec_at(k);
            uint32_t off = xoff;
            keep32(off);
#pragma unroll
            for (int o = 0; o < NO; ++o)
#pragma unroll
                for (int e = 0; e < 8; ++e) xn[o][e] = ld_spec<NT_, float>(src + o * obytes + e * rsb + off);
        };
        float gv[NB_][NO][8], gw[NB_];
        auto load_g = [&](int k) {
#pragma unroll
            for (int b = 0; b < NB_; ++b) {
                // a band without a kernel for slice k reads a valid octant with
                // weight 0 (one band per launch: always on); a band past nb
                // reads the first handled band's
                const bool on = NB_ == 1 || ks - k < a.Kc[b];
                gw[b] = on ? 1.f : 0.f;
                const int kb = on ? ks - k : 0, bb = b < a.nb ? b : 0;
                const char *gp = (const char *)(a.ghat + ((int64_t)kb * a.B + a.band0 + bb) * a.oct_stride);
#pragma unroll
                for (int o = 0; o < NO; ++o) {
                    // gdel < 0 for q > N/4: formed in 32 bits, where it wraps to
                    // the true (nonnegative) offset
                    const uint32_t od = (uint32_t)(o * gdel) * 4u;
                    uint32_t lo = glo + od, hi = ghi + od;
                    keep32(lo);
                    keep32(hi);
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        gv[b][o][e] = *(const float *)(gp + (e < 4 ? e * grb : -(e - 4) * grb) + (e < 4 ? lo : hi));
                }
            }
        };
        auto mac = [&](int o, const cx<float>(&v)[8]) {
#pragma unroll
            for (int b = 0; b < NB_; ++b)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float gg = NB_ == 1 ? gv[b][o][e] : gw[b] * gv[b][o][e];
                    sum[o][b][e] = mk(fma_((A)gg, (A)v[e].x, sum[o][b][e].x), fma_((A)gg, (A)v[e].y, sum[o][b][e].y));
                }
        };
        fill(k0);
        for (int k = k0; k < k1; ++k) {
            cx<float>(*lb)[L * CPW] = buf[(k - k0) & 1];
            load_g(k);
            cx<float> x[NO][8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const cx<float> u = xn[0][e];
                if constexpr (PAR) {
                    // last radix-2 step of the y transform: E +- W_N^q O
                    const cx<float> y = xn[1][e];
                    const float ux = fma_(wq.x, y.x, -wq.y * y.y), uy = fma_(wq.x, y.y, wq.y * y.x);
                    x[0][e] = mk(u.x + ux, u.y + uy);
                    x[1][e] = mk(u.x - ux, u.y - uy);
                } else {
                    x[0][e] = u;
                }
            }
            fill(k + 1);
            // a line buffer written here was last read two slices ago, before
            // the barrier that every thread has passed since
#pragma unroll
            for (int o = 0; o < NO; ++o) EF::first(x[o], lb[o], w, g, c, tw);
            lds_barrier();
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                cx<float> y[8];
                EF::rest(y, lb[o], t, c, tw);
                mac(o, y);
            }
        }

        // the (0,0,0) bin: row 0 of main column 0
        const bool has_dc = a.zero_dc && is_main && col == 0;
        const bool primary = k0 == 0;
#pragma unroll
        for (int b = 0; b < NB_; ++b) {
            if (b >= a.nb) break;   // (uniform: the barriers below stay matched)
            // the other buffer: its last readers are past a barrier
            cx<float>(*lb)[L * CPW] = buf[(k1 - k0 + b) & 1];
            cx<float> y[NO][8];
#pragma unroll
            for (int o = 0; o < NO; ++o) {
#pragma unroll
                for (int e = 0; e < 8; ++e) y[o][e] = mk((float)sum[o][b][e].x, (float)sum[o][b][e].y);
                if (o == 0 && has_dc && t == 0) y[o][0] = mk(0.f, 0.f);
                EI::first(y[o], lb[o], w, g, c, tw);
            }
            lds_barrier();
#pragma unroll
            for (int o = 0; o < NO; ++o) EI::rest(y[o], lb[o], t, c, tw);
            if constexpr (PAR) {
                // first radix-2 step of the inverse y transform, split by the
                // parity of the output rows (see fused_z_kernel)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const cx<float> u = y[0][e], v = y[1][e];
                    const cx<float> d = mk(u.x - v.x, u.y - v.y);
                    y[0][e] = mk(u.x + v.x, u.y + v.y);
                    y[1][e] = mk(fma_(wq.x, d.x, wq.y * d.y), fma_(wq.x, d.y, -wq.y * d.x));   // conj(W^q) d
                }
            }
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                if (primary) {
                    cx<float> *dst = a.acc + (int64_t)b * a.acc_stride + o * obase;
                    if (col_ok)
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            dst[(uint32_t)(cbase + (int64_t)(t + TPL * e) * s.row_stride)] = y[o][e];
                } else {
                    cx<float> *dst = a.part + (int64_t)b * a.part_stride + (int64_t)(NO * wg + o) * (L * CPW) + c;
#pragma unroll
                    for (int e = 0; e < 8; ++e) dst[(t + TPL * e) * CPW] = y[o][e];
                }
            }
        }
    };
    fused_walk<L, CPW, PAR>(a, s0, wg, segment);
}

// Parts of the tiles split by slices after the whole rounds (the rounds
// schedule's remaining slots full .. full + rest - 1): slice unit u of those
// tiles (u = i kmax + k for remaining tile i) belongs to workgroup w with
// w U / P <= u < (w + 1) U / P, U = rest kmax. The workgroup whose range holds
// unit i kmax wrote tile i to the accumulator; every other workgroup whose
// range starts inside tile i left its part in slot NO w + o (output o).
// The parts are added in a fixed order (within each share of the range in
// workgroup order, then the shares in order), so the result does not
// depend on timing.
struct RestMerge {
    cx<float> *acc;
    int64_t acc_stride;
    const cx<float> *part;
    int64_t part_stride;
    int32_t nband, no, cpw, L;
    int64_t full, rest, kmax, P;
    int32_t npb, gp, nrow;
};

void launch_fused_rest_merge(const RestMerge &m, const ColSet &s0, const ColSet &s1, hipStream_t st);
// split table of `count` entries (tiles of the launch) of a stream-K launch
void launch_fused_split(int *tab, int64_t tiles, int64_t kmax, int64_t P, int64_t W, int32_t pair, int64_t main_k,
                        int64_t count, hipStream_t st);

// Schedule of the plain forms: eight elements per thread where it exists.
template <int N> struct HasSched8 {
    static constexpr bool value = (N == 64 || N == 128 || N == 192 || N == 256 || N == 384 || N == 512);
};
template <int N, bool S8 = HasSched8<N>::value> struct PlainSchedOf { using type = Sched<N>; };
template <int N> struct PlainSchedOf<N, true> { using type = Sched8<N>; };
template <int N> using PlainSched = typename PlainSchedOf<N>::type;

// Column sets of the fused pass; with pair (parity layout) only the columns
// of rows q < N/2, each standing for rows q and q + N/2.
// T = double: the narrower tiles of the FP64 form.
template <int N, typename T = float>
static void fused_sets(ColSet &s0, ColSet &s1, bool pair = false) {
    constexpr int CPW = FusedShape<T, N, std::conditional_t<sizeof(T) == 4, FusedTiling<N>, PlainSched<N>>>::CPW;
    const int64_t H = N / 2;
    const int64_t rows = pair ? H : N;
    // main: columns (q, p) flat q*H + p; element (row r) at r*N*H + col
    s0.n_cols = rows * H; s0.W = (int64_t)N * H; s0.plane_stride = 0; s0.col_stride = 1;
    s0.row_stride = (int64_t)N * H; s0.off = 0; s0.rowfast = 0;
    // nyq: columns q; element (row r) at main + r*N + q
    s1.n_cols = rows; s1.W = N; s1.plane_stride = 0; s1.col_stride = 1; s1.row_stride = N;
    s1.off = spec_main(N); s1.rowfast = 0;
    s0.n_wgs = (int32_t)((s0.n_cols + CPW - 1) / CPW);
    s1.n_wgs = (int32_t)((s1.n_cols + CPW - 1) / CPW);
}

// Workgroups of one kernel that the device holds at a time.
template <auto KERNEL, int NT> static int fused_slots() {
    static int cached = 0;
    if (cached) return cached;
    int dev = 0, per_cu = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, KERNEL, NT, 0) != hipSuccess || per_cu < 1) per_cu = 1;
    cached = per_cu * prop.multiProcessorCount;
    return cached;
}

// Three or four bands per launch (plain sums, prefetch depth 1): compiled
// at N = 384 and 512, where the slice spectra are the largest and reading
// them once for four bands instead of twice pays most.
template <int N, int PF, int IN> constexpr bool fused_nb4() { return (N == 384 || N == 512) && PF == 1 && IN != 1; }

// Whether a launch over `tiles` tiles splits each one's slices in two: both
// halves of all tiles are resident together, a half is worth its prologue and
// its inverse transform (four slices or more), and the parts have a slot per tile.
inline bool fused_halves(int n, const FusedArgs &fa, int64_t tiles, int kmax, int64_t slots, bool par) {
    return fa.halves && fa.rounds && !par && n <= 96 && 2 * tiles <= slots && kmax >= 8 && tiles <= fa.max_parts;
}

// Launch of kernel KERNEL (one of the instances below) over the tiles.
template <int N, int CPW, int NT, bool PAR, auto KERNEL>
static hipError_t fused_go(const FusedArgs &fa, const void *tw, hipStream_t st, ColSet s0, ColSet s1, int64_t tiles,
                           int kmax) {
    static_assert(CPW == FusedShape<float, N, FusedTiling<N>>::CPW, "variants share the tiling");
    // Few tiles (N <= 96): a workgroup per tile walks all slices one after the
    // other while most SIMDs have no wave; each tile's slices go to two
    // workgroups, the second's sum to the part slot of the tile, which the
    // inverse y pass adds. Field of one band, 24 slices: 24^3 63 -> 47 us, 48^3
    // 47 -> 38, 96^3 66 -> 49; 64^3, 48 slices, 53 -> 40.
    const int64_t slots = fused_slots<KERNEL, NT>();
    const bool halves = fused_halves(N, fa, tiles, kmax, slots, PAR);
    // (two part slots per workgroup with two outputs per tile)
    const int64_t P = halves ? 2 * tiles : std::min<int64_t>(std::min<int64_t>(slots, tiles), fa.max_parts / (PAR ? 2 : 1));
    FusedDev<float> d;
    d.spec = (const cx<float> *)fa.spec; d.spec_stride = fa.spec_stride;
    d.ghat = (const float *)fa.ghat; d.oct_stride = fa.oct_stride;
    d.B = fa.B; d.band0 = fa.band0; d.nb = fa.nband;
    for (int b = 0; b < 4; ++b) d.Kc[b] = b < fa.nband ? fa.kcount[b] : 0;
    d.acc = (cx<float> *)fa.acc; d.acc_stride = fa.acc_stride;
    d.part = (cx<float> *)fa.part; d.part_stride = fa.part_stride;
    d.zero_dc = fa.zero_dc;
    d.kmax = kmax; d.P = (int32_t)P; d.W = tiles * kmax;
    d.rounds = halves ? 2 : fa.rounds; d.tiles = tiles;
    d.sk = fa.sk; d.g0 = fa.g0; d.inv_n3 = fa.inv_n3; d.mu = fa.mu; d.K = fa.K; d.ring = fa.ring; d.frozen = fa.frozen;
    // the split table serves the stream-K mode's merge in the inverse y pass;
    // the rounds mode splits no tile and its inverse pass does not read it
    if (!fa.rounds && !halves)
        launch_fused_split((int *)fa.split_tab, tiles, kmax, P, d.W, PAR ? 1 : 0, s0.n_wgs, tiles, st);
    hipLaunchKernelGGL(KERNEL, dim3((unsigned)P), dim3(NT), 0, st, d, s0, s1, (const cx<float> *)tw);
    const int64_t full = tiles / P * P;
    if (fa.halves) *fa.halves = halves;
    if (fa.rounds && !halves && full < tiles) {
        // parts of the tiles split by slices after the whole rounds
        RestMerge m;
        m.acc = (cx<float> *)fa.acc; m.acc_stride = fa.acc_stride;
        m.part = (const cx<float> *)fa.part; m.part_stride = fa.part_stride;
        m.nband = fa.nband; m.no = PAR ? 2 : 1; m.cpw = CPW; m.L = N;
        m.full = full; m.rest = tiles - full; m.kmax = kmax; m.P = P;
        m.npb = (N / 2) % CPW == 0 ? (N / 2) / CPW : 0;
        m.gp = fused_gp(CPW, sizeof(float));
        m.nrow = PAR ? N / 2 : N;
        launch_fused_rest_merge(m, s0, s1, st);
    }
    return hipGetLastError();
}

template <int N, typename S, int PF, int IN>
static hipError_t fused_launch(const FusedArgs &fa, const void *tw, hipStream_t st, ColSet s0, ColSet s1,
                               int64_t tiles, int kmax) {
    using SH = FusedShape<float, N, S>;
#define GO_(NB) return fused_go<N, SH::CPW, SH::NT, IN == 1, fused_z_kernel<float, N, NB, S, PF, IN, (NB <= 2)>>(fa, tw, st, s0, s1, tiles, kmax)
    if (fa.nband > 2) {
        if constexpr (fused_nb4<N, PF, IN>()) GO_(4);
        else return hipErrorInvalidValue;
    }
    if (fa.nband == 2) GO_(2);
    // (non-temporal loads beyond the last-level cache, as in fused_lane_launch)
    if constexpr (N == 192)
        if ((fa.frozen >= 0 ? 1 : kmax) * fa.spec_stride * 8 > ((int64_t)256 << 20))
            return fused_go<N, SH::CPW, SH::NT, IN == 1, fused_z_kernel<float, N, 1, S, PF, IN, true, true>>(
                fa, tw, st, s0, s1, tiles, kmax);
    GO_(1);
#undef GO_
}

// Grid sides with the lane-exchange kernel, the last variant there.
template <int N> constexpr bool fused_lane() { return N == 128 || N == 256; }
constexpr int kLaneVariant = 4;

template <int N, int IN>
static hipError_t fused_lane_launch(const FusedArgs &fa, const void *tw, hipStream_t st, ColSet s0, ColSet s1,
                                    int64_t tiles, int kmax) {
    using SH = LaneShape<N>;
    // Spectra that the last-level cache (256 MB) cannot hold stream past it: at
    // 256^3 x 40 (2.7 GB) 741 us with non-temporal loads against 784; slices
    // that do fit are found there (128^3 x 24, 200 MB: 57 us against 49).
    const bool nt = (fa.frozen >= 0 ? 1 : kmax) * fa.spec_stride * 8 > ((int64_t)256 << 20);
#define GO_(NB, NT_)                                                                                               \
    return fused_go<N, SH::CPW, SH::NT, IN == 1, fused_lane_kernel<N, NB, IN, NT_>>(fa, tw, st, s0, s1, tiles, kmax)
    if (fa.nband == 2) {
        if (nt) GO_(2, true);
        GO_(2, false);
    }
    if (fa.nband != 1) return hipErrorInvalidValue;
    if (nt) GO_(1, true);
    GO_(1, false);
#undef GO_
}

// parity-layout input: compiled where a half-plane xy shape exists (the
// pair tiles need rows that split into whole tiles)
template <int N> constexpr bool fused_par() { return N == 192 || N == 256; }
static_assert((256 / 2) % FusedShape<float, 256, FusedTiling<256>>::CPW == 0, "pair tiles cover whole rows");
static_assert((192 / 2) % FusedShape<float, 192, FusedTiling<192>>::CPW == 0, "pair tiles cover whole rows");

template <int N, int IN>
static hipError_t fused_sched(const FusedArgs &fa, const void *tw, hipStream_t st, ColSet s0, ColSet s1,
                              int64_t tiles, int kmax) {
    // variant = 2 * schedule + (prefetch depth 1 ? 1 : 0); schedule 1 = Sched8
    // (N = 384, 512 compile only the Sched8 pair)
    // (three or four bands per launch: prefetch depth 1 only)
    if constexpr (fused_lane<N>() && IN != 2) {
        if (fa.variant == kLaneVariant) return fused_lane_launch<N, IN>(fa, tw, st, s0, s1, tiles, kmax);
    }
    // (slices transformed along z already: the lane variant stands for the
    // eight-element schedule with two slices prefetched, the fastest there)
    const int var = fused_lane<N>() && fa.variant == kLaneVariant ? 2 : fa.variant;
    const int sched = fused_sched8_only<N>() ? 1 : var / 2, pf = var % 2 || fa.nband > 2 ? 1 : 2;
    if constexpr (HasSched8<N>::value) {
        if (sched == 1)
            return pf == 1 ? fused_launch<N, Sched8<N>, 1, IN>(fa, tw, st, s0, s1, tiles, kmax)
                           : fused_launch<N, Sched8<N>, 2, IN>(fa, tw, st, s0, s1, tiles, kmax);
    }
    if constexpr (!fused_sched8_only<N>()) {
        return pf == 1 ? fused_launch<N, Sched<N>, 1, IN>(fa, tw, st, s0, s1, tiles, kmax)
                       : fused_launch<N, Sched<N>, 2, IN>(fa, tw, st, s0, s1, tiles, kmax);
    }
    return hipErrorInvalidValue;
}

template <int N>
static hipError_t fused_t(const FusedArgs &fa, const void *tw, hipStream_t st) {
    if (fa.parity && (fa.pre || !fused_par<N>())) return hipErrorInvalidValue;
    ColSet s0, s1;
    fused_sets<N>(s0, s1, fa.parity != 0);
    const int64_t tiles = s0.n_wgs + s1.n_wgs;
    const int64_t std_tiles = fa.parity ? 2 * tiles : tiles;
    int kmax = 0;
    for (int b = 0; b < fa.nband; ++b) kmax = std::max(kmax, fa.kcount[b]);
    if (kmax <= 0) {
        // no slice contributes: the accumulators are zero (and so are the
        // kernels' DC values, hence the means)
        if (fa.mu) {
            hipError_t e = launch_fill_f64(fa.mu + fa.band0, fa.nband, 0.0, st);
            if (e != hipSuccess) return e;
        }
        for (int b = 0; b < fa.nband; ++b) {
            hipError_t e = launch_fill_bytes((char *)fa.acc + (size_t)b * fa.acc_stride * 8,
                                             fa.acc_stride * 8, st);
            if (e != hipSuccess) return e;
        }
        if (!fa.rounds)   // no tile split: every entry -1
            launch_fused_split((int *)fa.split_tab, std_tiles, 1, 1, std_tiles, 0, 0, std_tiles, st);
        return hipGetLastError();
    }
    if constexpr (fused_par<N>()) {
        if (fa.parity) return fused_sched<N, 1>(fa, tw, st, s0, s1, tiles, kmax);
    }
    if (fa.pre) return fused_sched<N, 2>(fa, tw, st, s0, s1, tiles, kmax);
    return fused_sched<N, 0>(fa, tw, st, s0, s1, tiles, kmax);
}

// Plain forms (FP64, plain FP32): one workgroup per tile walks all slices
// (no tile is split, so no parts and no merge), one or two bands per launch.
template <typename T, int N>
static hipError_t fused_plain_t(const FusedArgs &fa, const void *tw, hipStream_t st) {
    using S = PlainSched<N>;
    using SH = FusedShape<T, N, S>;
    if (fa.parity && !fused_par<N>()) return hipErrorInvalidValue;
    ColSet s0, s1;
    fused_sets<N, T>(s0, s1, fa.parity != 0);
    // (the plain FP32 tiles follow the schedule's own width)
    s0.n_wgs = (int32_t)((s0.n_cols + SH::CPW - 1) / SH::CPW);
    s1.n_wgs = (int32_t)((s1.n_cols + SH::CPW - 1) / SH::CPW);
    const int64_t tiles = s0.n_wgs + s1.n_wgs;
    int kmax = 0;
    for (int b = 0; b < fa.nband; ++b) kmax = std::max(kmax, fa.kcount[b]);
    if (kmax <= 0) {
        for (int b = 0; b < fa.nband; ++b) {
            hipError_t e = launch_fill_bytes((char *)fa.acc + (size_t)b * fa.acc_stride * sizeof(cx<T>),
                                             fa.acc_stride * (int64_t)sizeof(cx<T>), st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    FusedDev<T> d{};
    d.spec = (const cx<T> *)fa.spec; d.spec_stride = fa.spec_stride;
    d.ghat = (const T *)fa.ghat; d.oct_stride = fa.oct_stride;
    d.B = fa.B; d.band0 = fa.band0; d.nb = fa.nband;
    for (int b = 0; b < 4; ++b) d.Kc[b] = b < fa.nband ? fa.kcount[b] : 0;
    d.acc = (cx<T> *)fa.acc; d.acc_stride = fa.acc_stride;
    d.kmax = kmax; d.P = (int32_t)tiles; d.W = tiles * kmax;
    d.rounds = 1; d.tiles = tiles; d.K = fa.K; d.ring = fa.ring; d.frozen = fa.frozen;
    // (beyond the last-level cache the spectra stream past it, as in
    // fused_lane_launch)
    const bool nt = SH::CPW * sizeof(cx<T>) >= 128 &&
                    (fa.frozen >= 0 ? 1 : kmax) * fa.spec_stride * (int64_t)sizeof(cx<T>) > ((int64_t)256 << 20);
#define FP_(NB, IN)                                                                                               \
    do {                                                                                                          \
        if (nt)                                                                                                   \
            hipLaunchKernelGGL((fused_z_kernel<T, N, NB, S, 1, IN, false, true>), dim3((unsigned)tiles), dim3(SH::NT), \
                               0, st, d, s0, s1, (const cx<T> *)tw);                                              \
        else                                                                                                      \
            hipLaunchKernelGGL((fused_z_kernel<T, N, NB, S, 1, IN, false>), dim3((unsigned)tiles), dim3(SH::NT), 0, st, \
                               d, s0, s1, (const cx<T> *)tw);                                                     \
    } while (0)
    if constexpr (fused_par<N>()) {
        if (fa.parity) {
            if (fa.nband == 2) FP_(2, 1);
            else FP_(1, 1);
            return hipGetLastError();
        }
    }
    if (fa.nband == 2) FP_(2, 0);
    else FP_(1, 0);
#undef FP_
    return hipGetLastError();
}

}  // namespace lc
