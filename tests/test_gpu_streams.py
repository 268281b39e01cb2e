"""Chain launches of several streams at once: the ranks of a unit's workgroup
group wait for each other, so a launch must not start on CUs that another one's
incomplete groups hold (the launches are cooperative, also inside a captured
graph); every call must end with its waits met and the results it gives when it
runs alone, bit for bit."""
import pytest
import torch

from paper_2608_21308_amd import e2ttt, workloads as WL
from tests.gpu_util import config_of, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fw,d,dh,C", [(0, 64, 256, 64), (1, 64, 172, 64), (0, 128, 512, 32)])
def test_concurrent_streams_equal_one_stream(fw, d, dh, C):
    # 128 units of two, three and eight workgroups: each launch alone fills the device
    w = WL.WORKLOADS[1].with_(fw=fw, B=8, H=16, T=256, d=d, dh=dh, C=C, backward=True, seed=4300 + dh)
    cfg = config_of(w)
    t = to_dev(WL.make_inputs(w, with_grads=True), w.io)
    args = t["q"], t["k"], t["v"], t["eta"], t["beta"], t["gamma"], t["w_in"], None

    def step():
        out, wo, mo, ws = e2ttt.forward(cfg, *args, save_for_backward=True)
        scratch = torch.empty(e2ttt.backward_scratch_bytes(cfg), dtype=torch.uint8, device="cuda")
        g = e2ttt.backward(cfg, *args, ws, t["d_out"], scratch=scratch)
        return [out, wo, mo, *[g[n] for n in sorted(g)]], ws, scratch

    ref = step()[0]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    res = []
    for s in streams:
        with torch.cuda.stream(s):
            res.append(step())
    for s, (got, ws, scratch) in zip(streams, res):
        with torch.cuda.stream(s):
            assert e2ttt.wait_status(cfg, ws, scratch) == 0
        s.synchronize()
        for a, b in zip(got, ref):
            assert torch.equal(a, b)


@pytest.mark.parametrize("fw,d,dh,C", [(0, 64, 256, 64), (1, 64, 172, 64), (0, 128, 512, 32)])
def test_concurrent_graphs_equal_one_stream(fw, d, dh, C):
    # a training step captured per stream, the graphs replayed at once
    w = WL.WORKLOADS[1].with_(fw=fw, B=8, H=16, T=256, d=d, dh=dh, C=C, backward=True,
                              seed=4350 + dh)
    cfg = config_of(w)
    t = to_dev(WL.make_inputs(w, with_grads=True), w.io)
    args = t["q"], t["k"], t["v"], t["eta"], t["beta"], t["gamma"], t["w_in"], None

    def step(ws, scratch):
        out, wo, mo, _ = e2ttt.forward(cfg, *args, workspace=ws, save_for_backward=True)
        g = e2ttt.backward(cfg, *args, ws, t["d_out"], scratch=scratch)
        return [out, wo, mo, *[g[n] for n in sorted(g)]]

    def buffers():
        return (e2ttt.alloc_workspace(cfg, True),
                torch.empty(e2ttt.backward_scratch_bytes(cfg), dtype=torch.uint8, device="cuda"))

    ref = step(*buffers())
    runs = []
    for _ in range(3):
        s, bufs, graph = torch.cuda.Stream(), buffers(), torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            got = step(*bufs)
        runs.append((s, got, bufs, graph))
    for _ in range(3):
        for s, got, _, graph in runs:
            with torch.cuda.stream(s):
                for g in got:
                    g.fill_(float("nan"))
                graph.replay()
        for s, got, (ws, scratch), _ in runs:
            with torch.cuda.stream(s):
                assert e2ttt.wait_status(cfg, ws, scratch) == 0
            for a, b in zip(got, ref):
                assert torch.equal(a, b)
