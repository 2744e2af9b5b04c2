"""Order of a plan's work against torch's streams.

Until a program asks for `plan.stream`, calls run on torch's current stream;
afterwards on the plan's stream, ordered against the current one. Whatever
the current stream of each call (default, side streams, the plan's stream, a
stream under capture), a call must see the inputs produced before it on the
current stream, the earlier calls' state, and be seen by what follows. Each
case gives the same field, bit for bit, as calls on the default stream with
a device synchronisation around each.
"""
import numpy as np
import pytest

import lc_inputs as li

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, K = 64, 4


def _setup(use_graph=False, forms=None):
    import paper_1502_02294_amd as lc
    srcs = [li.random_sources([17, k], N, 3000) for k in range(K)]
    box = li.Box(n=N, box=50.0, radii=np.linspace(0.0, 40.0, K + 1), supersample=2, bands=[li.Atten()], sources=srcs)
    grids = [torch.from_numpy(li.dense_grid(N, c, v, np.float32)).reshape(N, N, N).cuda() for c, v in srcs]
    plan = lc.Plan([box], precision=lc.LC_PREC_FP32, use_graph=use_graph)
    plan.build_all()
    return lc, plan, grids


def _reference(plan, grids, out):
    for k, g in enumerate(grids):
        torch.cuda.synchronize()
        plan.push_grid(0, k, g)
    torch.cuda.synchronize()
    plan.field(0, 0, out=out)
    torch.cuda.synchronize()
    return out.clone()


def _late_copy(g):
    """g, produced late on the current stream (after a long run of kernels)."""
    t = torch.zeros_like(g)
    for _ in range(50):
        t.add_(1.0)
    return t.zero_().add_(g)


@pytest.mark.parametrize("ask", ["never", "first", "midway", "current"])
def test_calls_from_changing_streams(ask):
    lc, plan, grids = _setup()
    out = torch.empty((N,) * 3, device="cuda")
    ref = _reference(plan, grids, out)
    streams = [torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    if ask == "first":
        plan.stream
    if ask == "current":
        streams.append(plan.stream)
    for rep in range(3):
        print(f"case streams {ask} rep={rep}", flush=True)
        plan.push_grid(0, 0, torch.zeros_like(grids[0]))
        out.fill_(float("nan"))
        prev = torch.cuda.current_stream()
        keep = []
        for k, g in enumerate(grids):
            st = streams[(k + rep) % len(streams)]
            st.wait_stream(prev)
            with torch.cuda.stream(st):
                keep.append(_late_copy(g))
                plan.push_grid(0, k, keep[-1])
            prev = st
            if ask == "midway" and k == 1:
                plan.stream
        streams[0].wait_stream(prev)
        plan.field(0, 0, out=out)
        doubled = out * 2.0          # on the current stream, after the call
        assert torch.equal(doubled, ref * 2.0)
        torch.cuda.synchronize()
        del keep
    plan.close()


def test_plans_stream_object_sees_earlier_calls():
    lc, plan, grids = _setup()
    out = torch.empty((N,) * 3, device="cuda")
    ref = _reference(plan, grids, out)
    out.fill_(float("nan"))
    late = _late_copy(grids[0])
    plan.push_grid(0, 0, late)
    plan.field(0, 0, out=out)
    plan.stream.synchronize()        # everything enqueued so far
    got = torch.empty_like(out)
    with torch.cuda.stream(plan.stream):
        got.copy_(out)
    plan.stream.synchronize()
    assert torch.equal(got, ref)
    plan.close()


@pytest.mark.parametrize("where", ["plan_elsewhere", "plan_on_the_captured_stream"])
def test_calls_under_capture(where):
    lc, plan, grids = _setup()
    out = torch.empty((N,) * 3, device="cuda")
    ref = _reference(plan, grids, out)
    buf = torch.zeros_like(grids[0])
    st = torch.cuda.Stream()
    if where == "plan_on_the_captured_stream":
        st.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(st):
            plan.push_grid(0, 0, buf)
        torch.cuda.current_stream().wait_stream(st)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        plan.push_grid(0, 0, buf)
        plan.field(0, 0, out=out)
    for rep in range(3):
        print(f"case capture {where} replay={rep}", flush=True)
        buf.copy_(grids[0] * (rep + 1.0))
        out.fill_(float("nan"))
        g.replay()
        got = out.clone()
        # eager work between the replays
        keep = plan.push_grid(0, 0, grids[0] * (rep + 1.0))
        out.fill_(float("nan"))
        plan.field(0, 0, out=out)
        assert torch.equal(got, out)
        torch.cuda.synchronize()
        del keep
    buf.copy_(grids[0])
    g.replay()
    assert torch.equal(out, ref)
    plan.close()


def test_graph_step_from_changing_streams():
    lc, plan, grids = _setup(use_graph=True)
    out = [torch.empty((N,) * 3, device="cuda")]
    ref = _reference(plan, grids, out[0])
    bufs = [torch.empty_like(g) for g in grids]
    streams = [torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    prev = streams[0]
    for rep in range(4):
        print(f"case graph step rep={rep}", flush=True)
        st = streams[rep % 3]
        st.wait_stream(prev)
        with torch.cuda.stream(st):
            out[0].fill_(float("nan"))
            for b, g in zip(bufs, grids):
                b.copy_(_late_copy(g))
            keep = plan.step(bufs, out)
            got = out[0] + 0.0
        prev = st
        st.synchronize()
        assert torch.equal(got, ref)
        del keep
    plan.close()
