"""GPU: partially masked tiles of every kind the element mask tells apart -- one interval pair or both, each decided by one
bound (its intervals run to the edge of the rows) or by two -- against the oracle, in direct and queued units, at lengths
that are and are not multiples of the tiles.  Neighbouring heads hold the same tensors, so the first one stands for all."""
import numpy as np
import pytest
import torch

import paper_2410_01359_amd as fm
import workloads
from gpu_util import bf16_to_np, check_bwd, check_fwd, f64, to_device
from oracle import flashmask_oracle as orc

pytestmark = pytest.mark.gpu


def _bounds(mode, N):
    j = np.arange(N)
    none = np.full(N, N), np.full(N, N), np.zeros(N, int), np.zeros(N, int)
    lts, lte, uts, ute = none
    if mode in ("lower_edge", "both_edges"):       # row >= LTS decides
        lts = np.minimum(j + 37, N)
    if mode in ("upper_edge", "both_edges"):       # row < UTE decides
        ute = np.maximum(j - 41, 0)
    if mode in ("lower_inside", "both_inside"):    # starts and ends within a tile's rows
        lts, lte = np.minimum(j + 20, N), np.minimum(j + 20 + j % 70, N)
    if mode in ("upper_inside", "both_inside"):
        uts, ute = np.maximum(j - 90, 0), np.maximum(j - 90, 0) + j % 60
    return tuple(v.astype(np.int32) for v in (lts, lte, uts, ute))


@pytest.mark.parametrize("mode", ["lower_edge", "upper_edge", "both_edges", "lower_inside", "upper_inside", "both_inside"])
@pytest.mark.parametrize("H,N,d", [(3, 450, 128), (3, 512, 64), (24, 1024, 128), (160, 1000, 128), (160, 1024, 128), (200, 1152, 64)])
def test_mask_mode(mode, H, N, d):
    w = workloads.small_workload("causal", N, seed=11 + N, B=1, H=1, d=d)
    w.vectors = [_bounds(mode, N)]
    bits, dev, vecs = to_device(w)
    x = {n: dev[n].expand(1, H, N, d).contiguous() for n in ("q", "k", "v", "dout")}
    out, lse = fm.flashmask_fwd(x["q"], x["k"], x["v"], *vecs, w.scale)
    dq, dk, dv = fm.flashmask_bwd(x["q"], x["k"], x["v"], out, lse, x["dout"], *vecs, w.scale)
    torch.cuda.synchronize()
    for name, t in (("out", out), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv)):
        assert torch.equal(t, t[:, :1].expand_as(t)), f"{name}: heads differ"
    rdq, rdk, rdv, ro, rl = orc.backward(*(f64(bits[n][0, 0]) for n in ("q", "k", "v", "dout")), *w.vectors[0], w.scale)
    what = f"{mode} H={H} N={N} d={d}"
    check_fwd(bf16_to_np(out[0, 0]), lse[0, 0].cpu().numpy(), ro, rl, what)
    for name, got, ref in (("dq", dq, rdq), ("dk", dk, rdk), ("dv", dv, rdv)):
        check_bwd(bf16_to_np(got[0, 0]), ref, name, what)
