"""Near-field correction of more slices than one launch takes (24).

K = 30 thin shells inside the corrected cubes, some slices without sources,
FP32 and FP64 luminosities mixed, a slice whose factor is zero. FP64 field
against route D plus the oracle's correction, e_max <= 1e-12 (FP64 sums of at
most a few hundred terms).
"""
import dataclasses

import numpy as np
import pytest

import lc_inputs as li
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,R,m", [(24, 3, 3), (48, 8, 1)])
def test_near_field_of_many_slices(n, R, m):
    import paper_1502_02294_amd as lc
    K, L = 30, 0.78125 * n
    radii = np.linspace(0.2, 0.45 * L, K + 1)
    at = li.lw_band(0.4 * L)
    attens = [dataclasses.replace(at, prefactor=0.0 if k == 5 else 1.0 + 0.02 * k) for k in range(K)]
    positioned = []
    for k in range(K):
        p, v = li.positioned_sources([93, n, k], L, 0 if k in (0, 11, 25) else 3 + k % 5)
        positioned.append((p, v.astype(np.float32).astype(np.float64)))
    cells = [(oracle.ngp_cells(n, L, p), v) for p, v in positioned]
    box = li.Box(n=n, box=L, radii=radii, supersample=m, bands=[at], sources=cells)
    plan = lc.Plan([box], precision=lc.LC_PREC_FP64)
    print(f"case near batches n={n} R={R} m={m}", flush=True)
    plan.build_greens_slices(0, 0, attens)
    dev = [lc.Positioned(torch.from_numpy(np.ascontiguousarray(p)).cuda(),
                         torch.from_numpy(v.astype(np.float32) if k % 2 else v).cuda())
           for k, (p, v) in enumerate(positioned)]
    keep = [plan.push_positioned(0, k, s.pos, s.lum) for k, s in enumerate(dev)]
    J = plan.field(0, 0)
    plan.near_field(0, 0, dev, R, J)
    J = J.cpu().numpy()
    G = oracle.build_G_slices(n, L, radii, m, attens)
    Jr = oracle.field_direct(G, cells, np.arange(n ** 3)).reshape((n,) * 3)
    Jr = Jr + oracle.near_correction(n, L, radii, m, attens, positioned, R)
    e_max, e_rms = oracle.rel_errors(J, Jr)
    print(f"  e_max={e_max:.3e} e_rms={e_rms:.3e}", flush=True)
    assert e_max <= 1e-12
    del keep
    plan.close()
