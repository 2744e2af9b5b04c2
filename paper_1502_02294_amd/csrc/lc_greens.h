// Interface between the host plan code and the builder, deposit and near-field
// kernels (lc_greens.hip, lc_dct.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lc {

// Radial factor and shell of one slice, as the exact cell average (kernel rule
// 1, the m -> infinity limit of the subpoint average) takes them: pref / l^3
// times the integral of phi(r) / (4 pi r^2) over the part of an image cell
// inside [r_lo, r_sup), r_sup = min(r_{k+1}, end of phi's support).
struct ExactShell {
    double l, r_lo, r_sup, pref;
    double a, s, p, c;
    int32_t kind, reserved;
};
struct GaussRule {          // 16-point Gauss-Legendre rule on [0, 1]
    double x[16], w[16];
};

// Shell kernel builder (FP64): G_k of `count` consecutive slices on the octant
// [0, N/2]^3, slice j of the batch at oct + j (N/2+1)^3. Passed by value (no
// device table to write before the launch).
struct ShellArgs {
    static constexpr int kMax = 24;
    double *oct;
    int32_t n, m, count;
    int32_t rule;             // 0: m^3 subpoints; 1: exact cell average
    int32_t self_pair;        // rule 0, r_0 == 0: the own cell is replaced by self_val (slice 0)
    int32_t has_first;        // the batch starts at slice 0
    double self_val;
    double l, h;
    double r[kMax + 1], T[kMax + 1];   // shell edges r_k and thresholds T_k
    double cut[kMax];
    ExactShell sh[kMax];      // pref = 0: no kernel
    GaussRule rule16;
};
hipError_t launch_greens_shells(const ShellArgs &a, hipStream_t st);

// Cosine transforms of the octants of `count` slices (overwritten), the last
// axis storing into the plan's octant layout: slice k0 + j of the batch to
// oct + ((k0 + j) B + band) (N/2+1)^3 in FP64 or FP32, scaled by
// target_over_l3[j] / G^(0) where target_over_l3[j] >= 0 (else 1; G^(0) then
// from g00[k0 + j], FP64 scratch); the scaled G^(0) in FP64 to dc[(k0+j) B + band].
struct DctStore {
    void *oct;
    double *dc, *g00;
    int64_t k0;
    int32_t B, band, conserve;
    double target_over_l3[ShellArgs::kMax];
};
hipError_t launch_greens_dct(int n, double *oct, int count, const void *tw64_half, const void *twist64,
                             const DctStore &out, bool oct_f64, hipStream_t st);

// Near-field (particle-mesh) correction of a batch of slices with sources:
// their shells, radial factors and positioned point lists. Two launches per
// batch (one pair per slice took 20 us each, 16 slices of 128^3).
struct NearArgs {
    static constexpr int kMax = 24;
    int32_t n, m, R;           // grid side, subpoints per axis, near radius in cells
    int32_t count;
    int32_t rule, reserved;    // mesh kernel rule of the box (ShellArgs::rule)
    double l, h;
    double *table;             // count x (R+1)^3 primary-image mesh kernels (device)
    double *corr;              // N^3 FP64 correction accumulator (device)
    double t_lo[kMax], t_hi[kMax];     // T_k, T_{k+1}
    double r_hi[kMax], cut[kMax];      // r_{k+1} (r_k in sh)
    ExactShell sh[kMax];
    const double *pos[kMax];
    const void *lum[kMax];
    int64_t first[kMax + 1];   // sources before slice j of the batch; first[count] = all
    uint8_t lum_f64[kMax];
    GaussRule rule16;
};
hipError_t launch_near(const NearArgs &a, hipStream_t st);
hipError_t launch_deposit_pos(double *grid, int64_t n_pts, const double *pos, const void *lum, bool lum_f64, int n,
                              double l, hipStream_t st);
hipError_t launch_add_grid(void *out, bool out_f64, const double *corr, int64_t count, hipStream_t st);
hipError_t launch_deposit(double *grid, int64_t n_pts, const int64_t *cell, const void *lum,
                          bool lum_f64, int64_t n_cells, hipStream_t st);
// out = (j_inst - j) / j elementwise (0 where j == 0), FP64 arithmetic
hipError_t launch_fdiff(const void *j, const void *j_inst, void *out, int64_t count, bool f64, hipStream_t st);

// Device point lists of up to kMax slices of one box, deposited into compact
// rows instead of dense grids. Row r = z n + y of slice j has its n FP64 cells
// at rows + slot n, slot = map[j n^2 + r]; slot -1 stands for an empty row. A
// slice has at most min(points, n^2) rows: the first point that meets an empty
// row gives it the slot of its own index (slot0[j] + i), or with whole[j]
// (points >= n^2) row r has slot slot0[j] + r. One launch clears the map and
// the slots, one deposits (FP64 atomics, as launch_deposit).
struct PointTab {
    static constexpr int kMax = 64;
    const void *where[kMax];   // int64 cells, or with positioned[j] FP64 positions
    const void *lum[kMax];
    int64_t first[kMax + 1];   // points before slice j; first[count] = all
    int32_t slot0[kMax + 1];   // slots before slice j; slot0[count] = all
    uint8_t lum_f64[kMax], positioned[kMax], whole[kMax];
    int32_t count, n;
    double l;
    int32_t *map;              // count n^2 (16-byte aligned)
    double *rows;              // slot0[count] n (16-byte aligned)
};
hipError_t launch_point_rows(const PointTab &t, hipStream_t st);

}  // namespace lc
