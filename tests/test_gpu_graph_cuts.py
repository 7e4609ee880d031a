"""GPU: every cut of the work into units -- queued with the setup in one launch and in three, single, halved and
paired direct units -- recorded into a HIP graph after a call of the same shape class (head dimension, ragged or not)
that takes another cut: one call prepares its class.  Replays give the bits of the eager calls on new data."""
import pytest
import torch

import workloads
from gpu_util import to_device

pytestmark = pytest.mark.gpu


def _step(w):
    import paper_2410_01359_amd as fm
    _, dev, vecs = to_device(w)
    x = [dev[n].clone() for n in ("q", "k", "v", "dout")]
    ws = torch.empty(max(fm.flashmask_workspace_bytes(p, w.B, w.H, w.N, w.d) for p in (fm.FM_PASS_FWD, fm.FM_PASS_BWD)),
                     dtype=torch.uint8, device="cuda")

    def step():
        out, lse = fm.flashmask_fwd(*x[:3], *vecs, w.scale, workspace=ws)
        return (out, lse, *fm.flashmask_bwd(*x[:3], out, lse, x[3], *vecs, w.scale, workspace=ws))

    return x, step


# B, H, N of the call outside the capture and of the captured one, at 128-row units on 256 compute units:
@pytest.mark.parametrize("warm,size,d", [
    ((1, 2, 512), (4, 40, 1024), 128),     # halved -> queued, setup in one launch
    ((1, 2, 512), (1, 10, 8192), 128),     # halved -> queued forward, setup in three launches
    ((1, 2, 500), (4, 40, 1000), 64),      # the same at ragged lengths, d = 64
    ((4, 40, 1024), (2, 16, 1024), 128),   # queued -> paired
    ((4, 40, 1024), (2, 32, 1024), 128),   # queued -> direct
    ((4, 40, 1000), (1, 4, 1000), 64),     # queued -> halved
])
def test_graph_of_another_cut_than_the_call_before_it(warm, size, d):
    def load(shape, seed):
        return workloads.small_workload("causal_document", shape[2], seed=seed, B=shape[0], H=shape[1], d=d)

    _step(load(warm, 31))[1]()             # outside the capture
    x, step = _step(load(size, 32))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = step()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    for trial in range(3):
        for t in x:
            t.copy_(torch.randn(t.shape, device="cuda", generator=gen).bfloat16())
        eager = [y.clone() for y in step()]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for name, a, b in zip(("out", "lse", "dq", "dk", "dv"), eager, captured):
            assert torch.equal(a, b), f"replay {trial}: {name} differs from the eager call"
