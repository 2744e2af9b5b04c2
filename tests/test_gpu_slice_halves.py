"""Grids with few tiles: each tile's slices summed in two halves.

Up to N = 96 a launch of the slice sum with eight slices or more gives the two
halves of a tile's slices to different workgroups, and the inverse y pass adds
the second sum. Slice counts around the rule (7 and 8), odd counts, two bands
of which one has a kernel only in the first half, FP32 and FP64 outputs,
and the field from frozen sources. Against the FP64 form on the same grids:
e_rms <= 1e-6, the FP32 transforms' rounding (5e-8 to 2e-7 measured at these
sizes against the oracle) with a margin of five.
"""
import numpy as np
import pytest

import lc_inputs as li
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,K,bands", [(8, 8, 1), (24, 7, 1), (24, 17, 2), (32, 8, 1), (48, 23, 2), (64, 9, 1),
                                       (64, 40, 2), (96, 8, 1), (96, 25, 2)])
def test_halved_slices_match_fp64(n, K, bands):
    import paper_1502_02294_amd as lc
    L = 0.78125 * n
    radii = np.linspace(0.3, 0.48 * L, K + 1)
    ats = [li.Atten(), li.lw_band(0.2 * L)][:bands]
    srcs = [li.random_sources([31, n, k], n, 60) for k in range(K)]
    box = li.Box(n=n, box=L, radii=radii, supersample=1, bands=ats, sources=srcs)
    grids = [torch.from_numpy(li.dense_grid(n, c, v, np.float64)).cuda() for c, v in srcs]
    fields = {}
    for prec in (lc.LC_PREC_FP64, lc.LC_PREC_FP32):
        plan = lc.Plan([box], precision=prec)
        plan.build_all()
        print(f"case slice halves n={n} K={K} bands={bands} prec={prec}", flush=True)
        out = [torch.empty((n,) * 3, dtype=torch.float64, device="cuda") for _ in range(bands)]
        plan.step(grids, out)
        one = torch.empty((n,) * 3, dtype=torch.float32, device="cuda")
        plan.field(0, bands - 1, out=one)
        frozen = plan.field_frozen(0, 0, K - 1, dtype=torch.float64)
        fields[prec] = [o.cpu().numpy() for o in out] + [one.double().cpu().numpy(), frozen.cpu().numpy()]
        plan.close()
    for i, (a, r) in enumerate(zip(fields[lc.LC_PREC_FP32], fields[lc.LC_PREC_FP64])):
        e_max, e_rms = oracle.rel_errors(a, r)
        print(f"  field {i}: e_max={e_max:.3e} e_rms={e_rms:.3e}", flush=True)
        assert e_rms <= 1e-6
