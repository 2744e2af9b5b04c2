"""Kernels built in batches of consecutive shells (algorithm steps 2-3).

The builder takes as many shells per launch as the plan's scratch holds, at
most 24, and transforms each batch's octants by cosine transforms. Cases on
the edges of the batches: a plan whose scratch holds ten octants with 25
slices (two whole batches and one of five), rescaled to the shell integral,
with several periodic images; and a plan whose second, larger box leaves room
for the full 24 (49 slices: 24 + 24 + 1), with thin shells several of which
meet one cell, five subpoints an axis and two slices without a kernel.
FP64 against route D with the oracle's kernels on the full grid. Tolerance
e_max <= 1e-12: the kernel sums and transforms round at 1e-16 times a few
hundred operations, as for the other FP64 comparisons.
"""
import dataclasses

import numpy as np
import pytest

import lc_inputs as li
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("case", ["conserve_images", "zero_slices_two_boxes"])
def test_batched_builder_matches_oracle(case):
    import paper_1502_02294_amd as lc
    if case == "conserve_images":
        n, K, m, conserve, r0, r1, zero, others = 12, 25, 3, 1, 0.0, 2.6, (), ()
    else:
        n, K, m, conserve, r0, r1, zero, others = 8, 49, 5, 0, 0.05, 0.9, (10, 30), (48,)
    L = 0.78125 * n
    radii = np.linspace(r0 * L, r1 * L, K + 1)
    at = li.Atten(kind=1, s=4.0 * L)
    attens = [dataclasses.replace(at, prefactor=0.0 if k in zero else 1.0 + 0.01 * k) for k in range(K)]
    srcs = [li.random_sources([91, n, k], n, 4) for k in range(K)]
    box = li.Box(n=n, box=L, radii=radii, supersample=m, bands=[at], sources=srcs, conserve=conserve)
    more = [li.Box(n=v, box=0.78125 * v, radii=np.array([0.0, 5.0, 10.0]), supersample=1, bands=[at], sources=[])
            for v in others]
    if conserve:
        attens = [at] * K
        G = oracle.build_G(n, L, radii, m, at, conserve=1)
    else:
        G = oracle.build_G_slices(n, L, radii, m, attens)
    Jr = oracle.field_direct(G, srcs, np.arange(n ** 3)).reshape((n,) * 3)
    plan = lc.Plan([box] + more, precision=lc.LC_PREC_FP64)
    print(f"case builder batches {case}", flush=True)
    plan.build_greens_slices(0, 0, attens)
    keep = [plan.push_points(0, k, torch.from_numpy(c).cuda(), torch.from_numpy(v).cuda()) for k, (c, v) in enumerate(srcs)]
    J = plan.field(0, 0).cpu().numpy()
    e_max, e_rms = oracle.rel_errors(J, Jr)
    print(f"  e_max={e_max:.3e} e_rms={e_rms:.3e}", flush=True)
    assert e_max <= 1e-12
    dc = np.array(plan.greens_dc(0, 0))
    ref = G.reshape(K, -1).sum(axis=1)
    assert np.all(np.abs(dc - ref) <= 1e-12 * np.abs(ref).max())
    assert all(dc[k] == 0.0 for k in zero)
    assert plan.greens_imag_ratio(0, 0) <= 1e-12
    del keep
    plan.close()
