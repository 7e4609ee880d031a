"""GPU: the cuts of a tile loop's work between halved units and unit queues (units of 128 rows or keys without setup
launches, alone or with their tiles shared by two groups of four waves), at the unit counts on both sides of each line
for 256 compute units and at lengths where a group has no tile, an odd tile or a few real rows.  The same tensors in
every head: one head against the oracle, all others bit for bit."""
import numpy as np
import pytest
import torch

import paper_2410_01359_amd as fm
import workloads
from gpu_util import bf16_to_np, check_bwd, check_fwd, f64, to_device
from oracle import flashmask_oracle as orc

pytestmark = pytest.mark.gpu


def _heads_alike(w, H, Hk, strided, what):
    """Forward and backward of w's one head copied into H query and Hk K/V heads."""
    bits, dev, vecs = to_device(w)
    N, d = w.N, w.d
    x = {n: dev[n].expand(1, Hk if n in ("k", "v") else H, N, d) for n in ("q", "k", "v", "dout")}
    if strided:
        x = {n: t.transpose(1, 2).contiguous().transpose(1, 2) for n, t in x.items()}
        out, lse = fm.flashmask_fwd_ex(x["q"], x["k"], x["v"], *vecs, w.scale)
        dq, dk, dv = fm.flashmask_bwd_ex(x["q"], x["k"], x["v"], out, lse, x["dout"], *vecs, w.scale)
    else:
        x = {n: t.contiguous() for n, t in x.items()}
        out, lse = fm.flashmask_fwd(x["q"], x["k"], x["v"], *vecs, w.scale)
        dq, dk, dv = fm.flashmask_bwd(x["q"], x["k"], x["v"], out, lse, x["dout"], *vecs, w.scale)
    torch.cuda.synchronize()
    for name, t in (("out", out), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv)):
        assert torch.equal(t, t[:, :1].expand_as(t)), f"{what}: {name}: heads differ"
    rdq, rdk, rdv, ro, rl = orc.backward(*(f64(bits[n][0, 0]) for n in ("q", "k", "v", "dout")), *w.vectors[0], w.scale)
    check_fwd(bf16_to_np(out[0, 0]), lse[0, 0].cpu().numpy(), ro, rl, what)
    for name, got, ref in (("dq", dq, rdq), ("dk", dk, rdk * (H // Hk)), ("dv", dv, rdv * (H // Hk))):
        check_bwd(bf16_to_np(got[0, 0]), ref, name, what)


# units of 128 rows: 129 and 256 (two groups of four waves, d = 128), 257 and 512 (units alone), 513, 768 and 1025, 2049
# (short sequences on both sides of the line); lengths of one tile, of an odd number of tiles, with a few rows in the last
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,N", [(129, 64), (129, 128), (128, 256), (43, 330), (17, 1920), (15, 2112), (257, 128), (86, 321),
                                 (64, 1024), (52, 1100), (171, 384), (192, 500), (205, 576), (512, 512), (513, 400)])
@pytest.mark.parametrize("kind", ["full", "shared_question", "random_intervals"])
def test_cuts(kind, H, N, d):
    if kind == "shared_question" and N < 500:
        kind = "causal_document"
    _heads_alike(workloads.small_workload(kind, N, seed=H + N, B=1, H=1, d=d), H, H, False, f"{kind} H={H} N={N} d={d}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,Hk,N", [(80, 40, 400), (136, 34, 520), (20, 10, 1664), (64, 32, 1030)])
def test_cuts_strided_grouped(H, Hk, N, d):
    w = workloads.small_workload("causal", N, seed=H + N, B=1, H=1, d=d)
    lts, lte, uts, ute = (v.copy() for v in w.vectors[0])
    uts[:], ute[:] = 0, np.maximum(ute, 3)                 # rows 0..2 see nothing
    w.vectors = [(lts, lte, uts, ute)]
    _heads_alike(w, H, Hk, True, f"H={H}/{Hk} N={N} d={d}")


# How fm_direct_order.h deals the units, with groups of query heads and without, odd slices to two, four and eight XCDs: runs
# (12 on 3, 12 on 6 and 42 on 14 at d = 128), whole slices and units one by one (36 on 9; 42 on 14 at d = 64), turns that begin
# one XCD further on and a block after the last turn (20 alone and 12 on 6 at d = 64).
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,Hk,N", [(12, 3, 1100), (42, 14, 640), (36, 9, 1000), (12, 6, 2100), (20, 20, 1300)])
def test_deals(H, Hk, N, d):
    w = workloads.small_workload("document", N, seed=H + N, B=1, H=1, d=d)
    _heads_alike(w, H, Hk, H != Hk, f"H={H}/{Hk} N={N} d={d}")
