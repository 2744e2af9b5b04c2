// Periodic retarded-time shell kernel G_k (Eq. 10, algorithm step 2) and the
// folding of its FP64 spectrum (step 3), plus small utility kernels.
//
// Builder: the cells of the non-negative octant c in [0, N/2]^3, a batch of
// consecutive shells per launch. For every periodic image u whose cell box
// can reach the batch's shells the m^3 subpoints are summed, each into the
// shell whose [T_k, T_{k+1}) holds its exact integer squared distance n
// (units of the half-subcell h = L/(2 m N)), weighing
// pref * phi(rho) / (4 pi rho^2) / m^3, rho = sqrt(n) h. G is real and even in
// every axis, so its spectrum is the cosine transform of the octant along
// each axis (lc_dct.hip): no mirrored grid and no complex spectrum is formed.
#include <algorithm>

#include "lc_fft_device.h"
#include "lc_greens.h"
#include "lc_internal.h"

namespace lc {

__device__ __forceinline__ double phi_eval(int kind, double r, double a, double s, double p,
                                           double c, double cut) {
    if (kind == 0) return 1.0;
    const double v = a * exp(-pow(r / s, p)) - c;
    if (kind == 1) return v > 0.0 ? v : 0.0;
    return r <= cut ? v : 0.0;
}

// ---------------------------------------------------------------------------
// Exact cell average (rule 1)
//
// For an image cell [x0,x1] x [y0,y1] x [z0,z1] of the unit source at the
// origin, cylindrical coordinates about the z axis (radius R) and
// w = asinh(z / R) (so r = R cosh w and dz / r^2 = dw / (R cosh w)) give
//   pref / l^3 int_cell phi(r) / (4 pi r^2) [r_lo <= r < r_sup] d^3x
//     = pref / (4 pi l^3) int Q(R) V(R) dR,
//   Q(R) = angle of the circle of radius R inside [x0,x1] x [y0,y1],
//   V(R) = int phi(R cosh w) / cosh w dw over w in [asinh(z0/R), asinh(z1/R)]
//          with R cosh w in [r_lo, r_sup).
// Q is formed by inclusion-exclusion over the rectangle's corners of the
// arcs {R cos t >= a} and {R sin t >= b}; V is atan(sinh w) at the interval
// ends for phi = 1, else a 16-point rule on pieces of at most 2 in w (|w|
// <= 40: the weight 1 / cosh w is below 1e-17 beyond). The R integral is
// split where Q or V change form (edge and corner distances of the
// rectangle, r_lo, r_sup, sqrt(r^2 - z^2) for the z faces); each piece takes
// the 16-point rule after R = Ra + (Rb - Ra)(1 - cos u) / 2, which smooths the
// square-root behaviour at piece ends, on parts graded towards any such
// point that lies just outside it. In the cell holding the source,
// V(R) ~ V(0) - C R^p near R = 0 (the r^p cusp of phi at r = 0), so the
// piece from R = 0 is split geometrically at Rb 2^-j, j < 50, each part
// with the same substitution.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double arc_overlap(double a, double b, double c, double d) {
    const double lo = fmax(a, c), hi = fmin(b, d);
    return hi > lo ? hi - lo : 0.0;
}

// angle of {t : R cos t >= a and R sin t >= b}: the arc [-al, al] against
// the arc [be, pi - be] (and its copy one turn lower)
__device__ double arc_quarter(double R, double a, double b) {
    const double pi = 3.141592653589793238;
    const double al = acos(fmin(1.0, fmax(-1.0, a / R)));
    const double be = asin(fmin(1.0, fmax(-1.0, b / R)));
    return arc_overlap(-al, al, be, pi - be) + arc_overlap(-al, al, be - 2.0 * pi, -pi - be);
}

__device__ double circle_in_rect(double R, double x0, double x1, double y0, double y1) {
    return arc_quarter(R, x0, y0) - arc_quarter(R, x1, y0) - arc_quarter(R, x0, y1) + arc_quarter(R, x1, y1);
}

__device__ double exact_v(const ExactShell &e, const GaussRule &g, double R, double z0, double z1) {
    if (!(R < e.r_sup)) return 0.0;
    const double wH = acosh(e.r_sup / R), wL = R < e.r_lo ? acosh(e.r_lo / R) : 0.0;
    const double wa = asinh(z0 / R), wb = asinh(z1 / R);
    double acc = 0.0;
    for (int side = 0; side < 2; ++side) {
        double lo = side ? fmax(wa, wL) : fmax(wa, -wH);
        double hi = side ? fmin(wb, wH) : fmin(wb, -wL);
        if (!(hi > lo)) continue;
        if (e.kind == 0) {
            acc += atan(sinh(hi)) - atan(sinh(lo));
            continue;
        }
        lo = fmax(lo, -40.0);
        hi = fmin(hi, 40.0);
        if (!(hi > lo)) continue;
        const int pieces = (int)ceil((hi - lo) * 0.5);
        const double len = (hi - lo) / pieces;
        for (int q = 0; q < pieces; ++q) {
            const double w0 = lo + q * len;
            double sq = 0.0;
            for (int j = 0; j < 16; ++j) {
                const double w = w0 + len * g.x[j], ch = cosh(w), r = R * ch;
                const double v = e.a * exp(-pow(r / e.s, e.p)) - e.c;
                const double ph = (e.kind == 1 && v < 0.0) ? 0.0 : v;   // (kind 2: r < r_sup <= cut)
                sq += g.w[j] * ph / ch;
            }
            acc += len * sq;
        }
    }
    return acc;
}

__device__ double cell_exact(const ExactShell &e, const GaussRule &g, double x0, double x1, double y0, double y1, double z0,
                             double z1) {
    if (!(e.r_sup > e.r_lo)) return 0.0;
    const double nx = x0 > 0.0 ? x0 : (x1 < 0.0 ? -x1 : 0.0);
    const double ny = y0 > 0.0 ? y0 : (y1 < 0.0 ? -y1 : 0.0);
    const double Rmin = sqrt(nx * nx + ny * ny);
    const double fx = fmax(fabs(x0), fabs(x1)), fy = fmax(fabs(y0), fabs(y1));
    const double Rmax = fmin(sqrt(fx * fx + fy * fy), e.r_sup);
    if (!(Rmax > Rmin)) return 0.0;
    // every R where Q or V may change form (sing), and those inside the
    // range, sorted by insertion (br)
    double sing[20], br[20];
    int ns = 0, nb = 0;
    auto add = [&](double v) {
        sing[ns++] = v;
        if (!(v > Rmin && v < Rmax)) return;
        int i = nb++;
        while (i > 0 && br[i - 1] > v) { br[i] = br[i - 1]; --i; }
        br[i] = v;
    };
    const double xs[2] = {x0, x1}, ys[2] = {y0, y1}, zs[2] = {z0, z1}, rs[2] = {e.r_lo, e.r_sup};
    for (int i = 0; i < 2; ++i) {
        add(fabs(xs[i]));
        add(fabs(ys[i]));
        for (int j = 0; j < 2; ++j) {
            add(sqrt(xs[i] * xs[i] + ys[j] * ys[j]));
            if (rs[i] > fabs(zs[j])) add(sqrt(rs[i] * rs[i] - zs[j] * zs[j]));
        }
    }
    add(e.r_lo);
    add(e.r_sup);
    add(0.0);
    const bool source_cell = nx == 0.0 && ny == 0.0 && z0 <= 0.0 && z1 >= 0.0;
    // 16-point rule on [lo, hi] after the cosine substitution
    auto piece = [&](double lo, double hi) {
        const double pi = 3.141592653589793238;
        double sq = 0.0;
        for (int j = 0; j < 16; ++j) {
            const double u = pi * g.x[j];
            const double R = lo + 0.5 * (hi - lo) * (1.0 - cos(u));
            const double jac = pi * 0.5 * (hi - lo) * sin(u);
            sq += g.w[j] * jac * circle_in_rect(R, x0, x1, y0, y1) * exact_v(e, g, R, z0, z1);
        }
        return sq;
    };
    double acc = 0.0;
    double Ra = Rmin;
    for (int pc = 0; pc <= nb; ++pc) {
        const double Rb = pc < nb ? br[pc] : Rmax;
        if (!(Rb > Ra)) continue;
        if (Ra == 0.0 && source_cell) {
            // (the top piece keeps the substitution: R = Rb may be a square-root end)
            double hi = Rb;
            for (int i = 0; i < 50; ++i) {
                acc += piece(0.5 * hi, hi);
                hi *= 0.5;
            }
        } else {
            // A change of form just outside the piece, at distance dl < len
            // from Ra (a shell radius close to an edge distance, say), slows
            // the rule's convergence. The piece is then halved, and the half
            // at Ra is cut into parts graded towards it: [Ra, Ra + dl], then
            // parts as long as their distance to Ra (which, being a piece
            // end, may itself be such a point), up to the middle. The same
            // towards Rb with dr.
            double dl = 1e300, dr = 1e300;
            for (int i = 0; i < ns; ++i) {
                if (sing[i] < Ra) dl = fmin(dl, Ra - sing[i]);
                if (sing[i] > Rb) dr = fmin(dr, sing[i] - Rb);
            }
            const double len = Rb - Ra;
            if (dl >= len && dr >= len) {
                acc += piece(Ra, Rb);
            } else {
                const double mid = Ra + 0.5 * len;
                double lo = Ra;
                if (dl < mid - lo) {
                    acc += piece(lo, lo + dl);
                    lo += dl;
                    for (int i = 0; i < 64 && lo - Ra < mid - lo; ++i) {
                        const double d = lo - Ra;
                        acc += piece(lo, lo + d);
                        lo += d;
                    }
                }
                acc += piece(lo, mid);
                double hi = Rb;
                if (dr < hi - mid) {
                    acc += piece(hi - dr, hi);
                    hi -= dr;
                    for (int i = 0; i < 64 && Rb - hi < hi - mid; ++i) {
                        const double d = Rb - hi;
                        acc += piece(hi - d, hi);
                        hi -= d;
                    }
                }
                acc += piece(mid, hi);
            }
        }
        Ra = Rb;
    }
    const double four_pi = 12.566370614359172954;
    return e.pref * acc / (four_pi * e.l * e.l * e.l);
}

// Shells of a batch, all at once. A group of LPC lanes takes one octant cell:
// the images that can reach the batch are found once per cell (a few; the
// ranges of u are computed, not searched), and each subpoint's shell from its
// exact squared distance, so the radial factor is evaluated once per subpoint
// however many shells the batch holds. Arithmetic bound (FP64 pow, exp and
// sqrt per subpoint). One launch per shell, every cell testing every image,
// took 220 us a shell at 128^3 (24 shells, m = 4); the batches take 11.6 us.
// G is the same for every order of a cell's three indices (cubic box, cells and
// subpoints), so only cells ci <= cj <= ck are summed, a sixth of them, and the
// sum goes to the up to six cells of the other orders: 11.6 us a shell without
// this, 4.0 us with. A group adds to these cells itself, which no other group
// touches: no atomics, and the result does not depend on timing. LPC = 8
// spreads the m^3 subpoints of a cell over eight lanes (m = 1 has one, the
// exact rule works cell by cell: LPC = 1).
template <int LPC, bool EXACT>
__global__ __launch_bounds__(256) void greens_shells_kernel(ShellArgs a) {
    constexpr int KM = ShellArgs::kMax;
    // (three more edges, equal to the last: empty shells past the batch's end)
    __shared__ double T[KM + 4], r[KM + 4];
    __shared__ ExactShell sh[KM];
    __shared__ double cut[KM];
    __shared__ GaussRule rule16;
    const int cnt = a.count;
    if (threadIdx.x < KM + 4) {
        const int i = (int)threadIdx.x < cnt ? (int)threadIdx.x : cnt;
        T[threadIdx.x] = a.T[i];
        r[threadIdx.x] = a.r[i];
    }
    if ((int)threadIdx.x < cnt) {
        sh[threadIdx.x] = a.sh[threadIdx.x];
        cut[threadIdx.x] = a.cut[threadIdx.x];
    }
    if (EXACT && threadIdx.x < 16) {
        rule16.x[threadIdx.x] = a.rule16.x[threadIdx.x];
        rule16.w[threadIdx.x] = a.rule16.w[threadIdx.x];
    }
    __syncthreads();
    const int n = a.n, H = n / 2 + 1;
    const int64_t cells = (int64_t)H * H * H;
    const int64_t cell = ((int64_t)blockIdx.x * 256 + threadIdx.x) / LPC;
    const int sub = threadIdx.x % LPC;
    const int ci = (int)(cell / ((int64_t)H * H)), cj = (int)((cell / H) % H), ck = (int)(cell % H);
    if (cell >= cells || ci > cj || cj > ck) return;   // (a whole group leaves together)
    // add v to the cells of slice k with these indices in any order: order o of
    // (ci, cj, ck), ikj, jik, jki, kij, kji, those that differ
    double *__restrict__ G = a.oct;
    const int orders = ci == ck ? 0x01 : ci == cj ? 0x13 : cj == ck ? 0x0D : 0x3F;
    auto add = [&](int k, double v) {
#pragma unroll
        for (int o = LPC == 1 ? 0 : sub; o < 6; o += LPC) {
            if (!(orders >> o & 1)) continue;
            const int x = o < 2 ? ci : o < 4 ? cj : ck;
            const int y = o == 0 || o == 5 ? cj : o == 1 || o == 3 ? ck : ci;
            const int z = ci + cj + ck - x - y;
            G[k * cells + ((int64_t)x * H + y) * H + z] += v;
        }
    };
    const int m = a.m, m3 = m * m * m;
    const double l = a.l, r_lo = r[0], r_hi = r[cnt];
    const double four_pi = 12.566370614359172954;
    const double margin = 1e-9 * (r_hi + l);
    // |c + u n| <= reach, in cells, for every image that meets the batch
    const int reach = (int)ceil(r_hi / l + 1.5);
    auto u_first = [&](int c) { return -((reach + c) / n); };
    auto u_last = [&](int c) { return reach >= c ? (reach - c) / n : -1; };
    auto axis = [&](int x, double &lo, double &hi, double &nr, double &fr) {
        lo = (x - 0.5) * l;
        hi = (x + 0.5) * l;
        nr = lo > 0 ? lo : (hi < 0 ? -hi : 0.0);
        fr = fmax(fabs(lo), fabs(hi));
    };
    for (int u0 = u_first(ci); u0 <= u_last(ci); ++u0) {
        const int x0 = ci + u0 * n;
        double lo0, hi0, nr0, fr0;
        axis(x0, lo0, hi0, nr0, fr0);
        for (int u1 = u_first(cj); u1 <= u_last(cj); ++u1) {
            const int x1 = cj + u1 * n;
            double lo1, hi1, nr1, fr1;
            axis(x1, lo1, hi1, nr1, fr1);
            for (int u2 = u_first(ck); u2 <= u_last(ck); ++u2) {
                const int x2 = ck + u2 * n;
                double lo2, hi2, nr2, fr2;
                axis(x2, lo2, hi2, nr2, fr2);
                const double dmin = sqrt(nr0 * nr0 + nr1 * nr1 + nr2 * nr2);
                const double dmax = sqrt(fr0 * fr0 + fr1 * fr1 + fr2 * fr2);
                if (dmin > r_hi + margin || dmax < r_lo - margin) continue;
                // shells ka .. kb of the batch that this image cell can meet
                int ka = 0, kb = cnt - 1;
                while (ka < kb) {
                    const int mid = (ka + kb) / 2;
                    if (r[mid + 1] + margin < dmin) ka = mid + 1;
                    else kb = mid;
                }
                while (kb + 1 < cnt && r[kb + 1] <= dmax + margin) ++kb;
                if constexpr (EXACT) {
                    for (int k = ka; k <= kb; ++k)
                        if (sh[k].pref != 0.0) add(k, cell_exact(sh[k], rule16, lo0, hi0, lo1, hi1, lo2, hi2));
                } else {
                    if (a.self_pair && x0 == 0 && x1 == 0 && x2 == 0) {
                        // the source's own cell belongs to slice 0
                        if (a.has_first && sub == 0) G[0] += a.self_val;
                        continue;
                    }
                    for (int kk = ka; kk <= kb; kk += 3) {
                        const double t0 = T[kk], t1 = T[kk + 1], t2 = T[kk + 2], t3 = T[kk + 3];
                        double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0;
                        for (int s = sub; s < m3; s += LPC) {
                            const int a0 = s / (m * m), a1 = (s / m) % m, a2 = s % m;
                            // (whole numbers below 2^53: exact in any order)
                            const double q0 = 2.0 * m * x0 + (2 * a0 + 1 - m);
                            const double q1 = 2.0 * m * x1 + (2 * a1 + 1 - m);
                            const double q2 = 2.0 * m * x2 + (2 * a2 + 1 - m);
                            const double dn = q0 * q0 + q1 * q1 + q2 * q2;
                            if (dn >= t0 && dn < t3) {
                                const int j = (dn >= t1 ? 1 : 0) + (dn >= t2 ? 1 : 0);
                                const ExactShell &f = sh[kk + j];
                                const double rho = sqrt(dn) * a.h;
                                const double v = f.pref / (double)m3 *
                                                 phi_eval(f.kind, rho, f.a, f.s, f.p, f.c, cut[kk + j]) /
                                                 (four_pi * rho * rho);
                                acc0 += j == 0 ? v : 0.0;
                                acc1 += j == 1 ? v : 0.0;
                                acc2 += j == 2 ? v : 0.0;
                            }
                        }
#pragma unroll
                        for (int o = LPC / 2; o > 0; o >>= 1) {
                            acc0 += __shfl_xor(acc0, o, 64);
                            acc1 += __shfl_xor(acc1, o, 64);
                            acc2 += __shfl_xor(acc2, o, 64);
                        }
                        if (acc0 != 0.0) add(kk, acc0);
                        if (acc1 != 0.0) add(kk + 1, acc1);
                        if (acc2 != 0.0) add(kk + 2, acc2);
                    }
                }
            }
        }
    }
}

hipError_t launch_greens_shells(const ShellArgs &a, hipStream_t st) {
    if (a.count < 1 || a.count > ShellArgs::kMax || a.m < 1) return hipErrorInvalidValue;
    const int64_t H = a.n / 2 + 1, cells = H * H * H;
    hipError_t e = launch_fill_f64(a.oct, cells * a.count, 0.0, st);
    if (e != hipSuccess) return e;
    if (a.rule == 1)
        hipLaunchKernelGGL((greens_shells_kernel<1, true>), dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, st, a);
    else if (a.m == 1)
        hipLaunchKernelGGL((greens_shells_kernel<1, false>), dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((greens_shells_kernel<8, false>), dim3((unsigned)((cells * 8 + 255) / 256)), dim3(256), 0, st,
                           a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// near-field (particle-mesh) correction
//
// A source with a position inside its cell (x_s, in length units) is
// deposited to its nearest node c_s = round(x_s / l) mod N. For target nodes
// x = c_s + o, 0 < |o|_inf <= R, its mesh contribution L G_k(o) has a
// primary-image part that the correction replaces by the retarded kernel at
// the exact distance: J(x) += L (F_k(|x l - x_s|) - G^prim_k(o)), with
// F_k(rho) = [r_k <= rho < r_{k+1}] pref phi(rho) / (4 pi rho^2) and
// G^prim_k(o) the m^3-subpoint average of the image u = 0 (the same rule as
// the builder). The source's own node keeps the mesh value. Distances are
// formed without fused multiply-adds so that shell membership is decided
// on the same rounded values as a plain FP64 evaluation.
// ---------------------------------------------------------------------------
#pragma clang fp contract(off)
// index in [0, n) of node coordinate c (a whole number), wrapped periodically
__device__ __forceinline__ int64_t wrap_node(double c, int n) {
    double v = fmod(c, (double)n);
    if (v < 0.0) v += (double)n;
    if (v >= (double)n) v -= (double)n;
    return (int64_t)v;
}

// Primary-image mesh kernels of a batch of slices, a wave per entry (its
// lanes take the m^3 subpoints; the exact rule has one lane work).
__global__ __launch_bounds__(256) void near_table_kernel(NearArgs a) {
    const int R = a.R, W = R + 1, W3 = W * W * W;
    const int64_t e = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64;
    const int sub = threadIdx.x % 64;
    if (e >= (int64_t)a.count * W3) return;   // (the whole wave)
    const int k = (int)(e / W3), o = (int)(e % W3);
    const int d0 = o / (W * W), d1 = (o / W) % W, d2 = o % W;
    const int m = a.m, m3 = m * m * m;
    const double four_pi = 12.566370614359172954;
    const ExactShell &f = a.sh[k];
    double acc = 0.0;
    if (a.rule == 1) {
        const double l = a.l;
        if ((d0 | d1 | d2) && sub == 0)
            acc = cell_exact(f, a.rule16, (d0 - 0.5) * l, (d0 + 0.5) * l, (d1 - 0.5) * l, (d1 + 0.5) * l, (d2 - 0.5) * l,
                             (d2 + 0.5) * l);
    } else if (d0 | d1 | d2) {
        const double wm = f.pref / (double)m3, t_lo = a.t_lo[k], t_hi = a.t_hi[k];
        for (int s = sub; s < m3; s += 64) {
            const int a0 = s / (m * m), a1 = (s / m) % m, a2 = s % m;
            const int64_t q0 = 2 * m * (int64_t)d0 + (2 * a0 + 1 - m);
            const int64_t q1 = 2 * m * (int64_t)d1 + (2 * a1 + 1 - m);
            const int64_t q2 = 2 * m * (int64_t)d2 + (2 * a2 + 1 - m);
            const double dn = (double)(q0 * q0 + q1 * q1 + q2 * q2);
            if (dn >= t_lo && dn < t_hi) {
                const double rho = sqrt(dn) * a.h;
                acc += wm * phi_eval(f.kind, rho, f.a, f.s, f.p, f.c, a.cut[k]) / (four_pi * rho * rho);
            }
        }
#pragma unroll
        for (int x = 32; x > 0; x >>= 1) acc += __shfl_xor(acc, x, 64);
    }
    if (sub == 0) a.table[e] = acc;
}

// Corrections of a batch of slices: work item = (slice, source, offset).
__global__ __launch_bounds__(256) void near_corr_kernel(NearArgs a) {
    __shared__ int64_t first[NearArgs::kMax + 1];
    if ((int)threadIdx.x <= a.count) first[threadIdx.x] = a.first[threadIdx.x];
    __syncthreads();
    const int R = a.R, D = 2 * R + 1, W = R + 1;
    const int64_t V = (int64_t)D * D * D;
    const int n = a.n;
    const double four_pi = 12.566370614359172954;
    const int64_t total = first[a.count] * V;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t g = e / V;
        const int o = (int)(e % V);
        const int o0 = o / (D * D) - R, o1 = (o / D) % D - R, o2 = o % D - R;
        if (!(o0 | o1 | o2)) continue;
        int k = 0, hi = a.count - 1;      // slice of source g
        while (k < hi) {
            const int mid = (k + hi + 1) / 2;
            if (first[mid] <= g) k = mid;
            else hi = mid - 1;
        }
        const int64_t s = g - first[k];
        const double *__restrict__ pos = a.pos[k];
        const double p0 = pos[3 * s], p1 = pos[3 * s + 1], p2 = pos[3 * s + 2];
        // a non-finite position has no cell (its slice is flagged by the deposit)
        if (!isfinite(p0) || !isfinite(p1) || !isfinite(p2)) continue;
        const double L = a.lum_f64[k] ? ((const double *)a.lum[k])[s] : (double)((const float *)a.lum[k])[s];
        const double c0 = floor(p0 / a.l + 0.5), c1 = floor(p1 / a.l + 0.5), c2 = floor(p2 / a.l + 0.5);
        const double y0 = (c0 + o0) * a.l - p0, y1 = (c1 + o1) * a.l - p1, y2 = (c2 + o2) * a.l - p2;
        const double rho = sqrt(y0 * y0 + y1 * y1 + y2 * y2);
        const ExactShell &f = a.sh[k];
        double F = 0.0;
        if (rho >= f.r_lo && rho < a.r_hi[k])
            F = f.pref * phi_eval(f.kind, rho, f.a, f.s, f.p, f.c, a.cut[k]) / (four_pi * rho * rho);
        const int t0 = o0 < 0 ? -o0 : o0, t1 = o1 < 0 ? -o1 : o1, t2 = o2 < 0 ? -o2 : o2;
        const double M = a.table[(((int64_t)k * W + t0) * W + t1) * W + t2];
        const double dv = L * (F - M);
        if (dv == 0.0) continue;
        const int64_t cell =
            (wrap_node(c0 + o0, n) * n + wrap_node(c1 + o1, n)) * n + wrap_node(c2 + o2, n);
        atomicAdd(&a.corr[cell], dv);
    }
}

// nearest-node deposit of positioned sources (positions in length units,
// wrapped periodically)
template <typename TL>
__global__ __launch_bounds__(256) void deposit_pos_kernel(double *__restrict__ grid, int64_t n_pts,
                                                          const double *__restrict__ pos,
                                                          const TL *__restrict__ lum, int n, double l) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_pts;
         e += (int64_t)gridDim.x * blockDim.x) {
        const double p0 = pos[3 * e], p1 = pos[3 * e + 1], p2 = pos[3 * e + 2];
        if (!isfinite(p0) || !isfinite(p1) || !isfinite(p2)) {
            // no cell: make the slice's sum non-finite so that the check flags it
            atomicAdd(&grid[0], (double)NAN);
            continue;
        }
        const int64_t cell = (wrap_node(floor(p0 / l + 0.5), n) * n + wrap_node(floor(p1 / l + 0.5), n)) * n +
                             wrap_node(floor(p2 / l + 0.5), n);
        atomicAdd(&grid[cell], (double)lum[e]);
    }
}
// Compact-row deposit of a batch of slices (PointTab). A dense FP64 grid per
// slice costs its clearing and reading whatever the points: 134 MB each at
// 256^3, 20 us and 56 us, for 200 to 46,000 points. The rows hold 2 KB per point
// at most, and the forward pass reads only those that exist.
__global__ __launch_bounds__(256) void point_rows_kernel(PointTab t) {
    __shared__ int64_t first[PointTab::kMax + 1];
    if ((int)threadIdx.x <= t.count) first[threadIdx.x] = t.first[threadIdx.x];
    __syncthreads();
    const int n = t.n;
    const int64_t n2 = (int64_t)n * n, n3 = n2 * n, total = first[t.count];
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        int j = 0, hi = t.count - 1;      // slice of point e
        while (j < hi) {
            const int mid = (j + hi + 1) / 2;
            if (first[mid] <= e) j = mid;
            else hi = mid - 1;
        }
        const int64_t i = e - first[j];
        double v = t.lum_f64[j] ? ((const double *)t.lum[j])[i] : (double)((const float *)t.lum[j])[i];
        int64_t cell;
        if (t.positioned[j]) {
            const double *pos = (const double *)t.where[j];
            const double p0 = pos[3 * i], p1 = pos[3 * i + 1], p2 = pos[3 * i + 2];
            if (!isfinite(p0) || !isfinite(p1) || !isfinite(p2)) {
                // no cell: make the slice's sum non-finite so that the check flags it
                cell = 0;
                v = (double)NAN;
            } else {
                cell = (wrap_node(floor(p0 / t.l + 0.5), n) * n + wrap_node(floor(p1 / t.l + 0.5), n)) * n +
                       wrap_node(floor(p2 / t.l + 0.5), n);
            }
        } else {
            cell = ((const int64_t *)t.where[j])[i];
            if (cell < 0 || cell >= n3) continue;
        }
        const int64_t r = cell / n;
        int32_t *m = t.map + j * n2 + r;
        int slot;
        if (t.whole[j]) {
            slot = t.slot0[j] + (int)r;
            *m = slot;                    // (every point of the row writes the same)
        } else {
            const int mine = t.slot0[j] + (int)i;
            const int old = atomicCAS(m, -1, mine);
            slot = old == -1 ? mine : old;
        }
        atomicAdd(&t.rows[(int64_t)slot * n + (cell - r * n)], v);
    }
}
#pragma clang fp contract(on)

template <typename TO>
__global__ __launch_bounds__(256) void add_grid_kernel(TO *__restrict__ out, const double *__restrict__ corr,
                                                       int64_t count) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
         e += (int64_t)gridDim.x * blockDim.x)
        if (corr[e] != 0.0) out[e] = (TO)((double)out[e] + corr[e]);
}

hipError_t launch_near(const NearArgs &a, hipStream_t st) {
    if (a.count < 1 || a.count > NearArgs::kMax) return hipErrorInvalidValue;
    const int64_t W = a.R + 1, D = 2 * a.R + 1;
    const int64_t lanes = 64 * a.count * W * W * W;
    hipLaunchKernelGGL(near_table_kernel, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, st, a);
    const int64_t work = a.first[a.count] * D * D * D;
    const int wgs = (int)std::min<int64_t>((work + 255) / 256, 16384);
    hipLaunchKernelGGL(near_corr_kernel, dim3(wgs), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_deposit_pos(double *grid, int64_t n_pts, const double *pos, const void *lum, bool lum_f64, int n,
                              double l, hipStream_t st) {
    if (n_pts <= 0) return hipSuccess;
    const int wgs = (int)std::min<int64_t>((n_pts + 255) / 256, 8192);
    if (lum_f64)
        hipLaunchKernelGGL(deposit_pos_kernel<double>, dim3(wgs), dim3(256), 0, st, grid, n_pts, pos,
                           (const double *)lum, n, l);
    else
        hipLaunchKernelGGL(deposit_pos_kernel<float>, dim3(wgs), dim3(256), 0, st, grid, n_pts, pos,
                           (const float *)lum, n, l);
    return hipGetLastError();
}

// map to -1, slots to zero, 16 bytes per lane and turn
__global__ __launch_bounds__(256) void clear_rows_kernel(int4 *__restrict__ map, int64_t n_map, int4 *__restrict__ rows,
                                                         int64_t n_rows) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_map + n_rows;
         e += (int64_t)gridDim.x * blockDim.x) {
        if (e < n_map) map[e] = make_int4(-1, -1, -1, -1);
        else rows[e - n_map] = make_int4(0, 0, 0, 0);
    }
}

hipError_t launch_point_rows(const PointTab &t, hipStream_t st) {
    if (t.count < 1 || t.count > PointTab::kMax || t.n % 2) return hipErrorInvalidValue;
    const int64_t n_map = (int64_t)t.count * t.n * t.n / 4, n_rows = (int64_t)t.slot0[t.count] * t.n / 2;
    const int64_t total = t.first[t.count];
    int wgs = (int)std::min<int64_t>((n_map + n_rows + 255) / 256, 16384);
    hipLaunchKernelGGL(clear_rows_kernel, dim3(wgs), dim3(256), 0, st, (int4 *)t.map, n_map, (int4 *)t.rows, n_rows);
    if (total > 0) {
        wgs = (int)std::min<int64_t>((total + 255) / 256, 8192);
        hipLaunchKernelGGL(point_rows_kernel, dim3(wgs), dim3(256), 0, st, t);
    }
    return hipGetLastError();
}

hipError_t launch_add_grid(void *out, bool out_f64, const double *corr, int64_t count, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    const int wgs = (int)std::min<int64_t>((count + 255) / 256, 16384);
    if (out_f64)
        hipLaunchKernelGGL(add_grid_kernel<double>, dim3(wgs), dim3(256), 0, st, (double *)out, corr, count);
    else
        hipLaunchKernelGGL(add_grid_kernel<float>, dim3(wgs), dim3(256), 0, st, (float *)out, corr, count);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// utilities
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void fill_f64_kernel(double *__restrict__ p, int64_t count, double v) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
         e += (int64_t)gridDim.x * blockDim.x)
        p[e] = v;
}

__global__ __launch_bounds__(256) void fill_u32_kernel(uint32_t *__restrict__ p, int64_t count) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
         e += (int64_t)gridDim.x * blockDim.x)
        p[e] = 0u;
}

__global__ __launch_bounds__(256) void fill_i32_kernel(int32_t *__restrict__ p, int64_t count, int32_t v) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
         e += (int64_t)gridDim.x * blockDim.x)
        p[e] = v;
}

hipError_t launch_fill_i32(int32_t *p, int64_t count, int32_t v, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    const int wgs = (int)std::min<int64_t>((count + 255) / 256, 16384);
    hipLaunchKernelGGL(fill_i32_kernel, dim3(wgs), dim3(256), 0, st, p, count, v);
    return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(256) void fdiff_kernel(const T *__restrict__ j, const T *__restrict__ ji,
                                                    T *__restrict__ out, int64_t count) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
         e += (int64_t)gridDim.x * blockDim.x) {
        const double a = (double)j[e], b = (double)ji[e];
        out[e] = (T)(a != 0.0 ? (b - a) / a : 0.0);
    }
}

hipError_t launch_fdiff(const void *j, const void *j_inst, void *out, int64_t count, bool f64, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    const int wgs = (int)std::min<int64_t>((count + 255) / 256, 16384);
    if (f64)
        hipLaunchKernelGGL(fdiff_kernel<double>, dim3(wgs), dim3(256), 0, st, (const double *)j,
                           (const double *)j_inst, (double *)out, count);
    else
        hipLaunchKernelGGL(fdiff_kernel<float>, dim3(wgs), dim3(256), 0, st, (const float *)j,
                           (const float *)j_inst, (float *)out, count);
    return hipGetLastError();
}

hipError_t launch_fill_f64(double *p, int64_t count, double v, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    const int wgs = (int)std::min<int64_t>((count + 255) / 256, 16384);
    hipLaunchKernelGGL(fill_f64_kernel, dim3(wgs), dim3(256), 0, st, p, count, v);
    return hipGetLastError();
}

hipError_t launch_fill_bytes(void *p, int64_t bytes, hipStream_t st) {
    if (bytes <= 0) return hipSuccess;
    if (bytes % 4) return hipErrorInvalidValue;
    const int64_t count = bytes / 4;
    const int wgs = (int)std::min<int64_t>((count + 255) / 256, 16384);
    hipLaunchKernelGGL(fill_u32_kernel, dim3(wgs), dim3(256), 0, st, (uint32_t *)p, count);
    return hipGetLastError();
}

template <typename TL>
__global__ __launch_bounds__(256) void deposit_kernel(double *__restrict__ grid, int64_t n_pts,
                                                      const int64_t *__restrict__ cell,
                                                      const TL *__restrict__ lum, int64_t n_cells) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_pts;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = cell[e];
        if (c >= 0 && c < n_cells) atomicAdd(&grid[c], (double)lum[e]);
    }
}

hipError_t launch_deposit(double *grid, int64_t n_pts, const int64_t *cell, const void *lum,
                          bool lum_f64, int64_t n_cells, hipStream_t st) {
    if (n_pts <= 0) return hipSuccess;
    const int wgs = (int)std::min<int64_t>((n_pts + 255) / 256, 8192);
    if (lum_f64)
        hipLaunchKernelGGL(deposit_kernel<double>, dim3(wgs), dim3(256), 0, st, grid, n_pts, cell,
                           (const double *)lum, n_cells);
    else
        hipLaunchKernelGGL(deposit_kernel<float>, dim3(wgs), dim3(256), 0, st, grid, n_pts, cell,
                           (const float *)lum, n_cells);
    return hipGetLastError();
}

}  // namespace lc
