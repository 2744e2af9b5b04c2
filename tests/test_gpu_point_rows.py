"""Point lists through compact rows against the same sources as dense grids.

Luminosities are small whole numbers, so the FP64 sums of coincident points are
exact in any order and the field must be the same bit for bit as with dense
FP64 grids. Slice sizes on the edges of the row map: no point, one point, N^2
- 1 and N^2 + 5 points (rows claimed one by one, and the whole map), many
points of few cells; cells outside the grid are ignored; FP32 and FP64
luminosities, flat cells and positions, in one captured step and as single
pushes.
"""
import numpy as np
import pytest

import lc_inputs as li

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _lists(n, L, K):
    rng = np.random.default_rng([23, n])
    dev, grids = [], []
    for k, count in enumerate([0, 1, n * n - 1, n * n + 5, 5000][:K]):
        cells = rng.integers(0, n ** 3, size=count) if k != 4 else rng.integers(0, 40, size=count) * (n + 3)
        lum = rng.integers(1, 9, size=count).astype(np.float32 if k % 2 else np.float64)
        g = np.bincount(cells, weights=lum.astype(np.float64), minlength=n ** 3).astype(np.float64)   # (no point: whole numbers)
        grids.append(torch.from_numpy(g).cuda())
        if k == 4:
            # positions within their cells, some outside the box (wrapped)
            c = np.stack([cells // (n * n), cells // n % n, cells % n], 1).astype(np.float64)
            pos = (c + rng.uniform(-0.4, 0.4, size=c.shape) + n * rng.integers(-1, 2, size=c.shape)) * (L / n)
            dev.append(("pos", torch.from_numpy(pos).cuda(), torch.from_numpy(lum).cuda()))
        else:
            if k == 2:
                cells, lum = np.append(cells, [-1, n ** 3]), np.append(lum, lum[:2])
            dev.append(("cells", torch.from_numpy(cells.astype(np.int64)).cuda(), torch.from_numpy(lum).cuda()))
    return dev, grids


@pytest.mark.parametrize("form", ["fp64", "fp32", "plain"])
@pytest.mark.parametrize("n", [64, 96, 128, 192, 256])
def test_point_rows_equal_dense_grids(n, form):
    import paper_1502_02294_amd as lc
    K, L = 5, 0.78125 * n
    prec = {"fp64": lc.LC_PREC_FP64, "fp32": lc.LC_PREC_FP32, "plain": lc.LC_PREC_FP32_PLAIN}[form]
    box = li.Box(n=n, box=L, radii=np.linspace(0.0, 0.3 * L, K + 1), supersample=1, bands=[li.Atten()],
                 sources=[None] * K)
    dev, grids = _lists(n, L, K)
    plan = lc.Plan([box], precision=prec, use_graph=True)
    plan.build_all()
    shapes = [None]
    if form == "fp32" and n >= 192:
        shapes = [0, {192: 2, 256: 4}[n]]       # whole planes, rows of one parity
    for shape in shapes:
        if shape is not None:
            plan.set_schedule(0, xy_variant=shape)
        for k, g in enumerate(grids):
            plan.push_grid(0, k, g)
        ref = plan.field(0, 0)
        assert torch.isfinite(ref).all() and ref.abs().max() > 0
        for rep in range(2):
            print(f"case point rows n={n} {form} shape={shape} rep={rep}", flush=True)
            out = [torch.full_like(ref, float("nan"))]
            keep = plan.step([lc.Positioned(a, v) if kind == "pos" else (a, v) for kind, a, v in dev], out)
            assert torch.equal(out[0], ref)
        for k, (kind, a, v) in enumerate(dev):
            plan.push_grid(0, k, torch.ones_like(grids[k]))
            if kind == "pos":
                plan.push_positioned(0, k, a, v)
            else:
                plan.push_points(0, k, a, v)
        assert torch.equal(plan.field(0, 0), ref)
        # a non-finite position has no cell but is reported
        bad = dev[4][1].clone()
        bad[7, 1] = float("inf")
        plan.push_positioned(0, 4, bad, dev[4][2])
        plan.field(0, 0)
        with pytest.raises(lc.LCError) as err:
            plan.check_sources(0)
        assert err.value.code == lc.LC_ENONFINITE
        del keep
    plan.close()


@pytest.mark.parametrize("n,K", [(192, 24), (256, 10)])
def test_point_rows_stored_past_the_cache(n, K):
    """FP32 steps whose spectra are stored non-temporally (more than 640 MiB):
    bit for bit the field of dense FP64 grids, on two passes."""
    import paper_1502_02294_amd as lc
    L = 0.78125 * n
    box = li.Box(n=n, box=L, radii=np.linspace(0.0, 0.9 * L, K + 1), supersample=1, bands=[li.Atten()],
                 sources=[None] * K)
    plan = lc.Plan([box], precision=lc.LC_PREC_FP32)
    plan.build_all()
    for seed in (1, 2):
        rng = np.random.default_rng([seed, n])
        dev = []
        for k in range(K):
            cells = rng.integers(0, n ** 3, size=300 * k)
            lum = rng.integers(1, 9, size=300 * k).astype(np.float64)
            g = torch.zeros(n ** 3, dtype=torch.float64, device="cuda")
            g.index_add_(0, torch.from_numpy(cells).cuda(), torch.from_numpy(lum).cuda())
            plan.push_grid(0, k, g)
            dev.append((torch.from_numpy(cells).cuda(), torch.from_numpy(lum).cuda()))
        ref = plan.field(0, 0)
        out = [torch.empty((n,) * 3, device="cuda")]
        plan.step(dev, out)
        assert torch.isfinite(ref).all() and ref.abs().max() > 0
        assert torch.equal(ref, out[0])
    plan.close()
