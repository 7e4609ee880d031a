"""GPU: the bands of sizes between the cuts of the work that the small sizes of the other tests do not reach -- queues of
one round, queues for one of the backward's loops only, long sequences of few units.  Each size names the cuts it is
there for, so that a line that moves shows here.  The same tensors in every head: one head against the oracle on sampled
rows and columns, all others bit for bit."""
import numpy as np
import pytest
import torch

import paper_2410_01359_amd as fm
import workloads
from gpu_util import bf16_to_np, check_bwd, check_fwd, f64, to_device
from oracle import flashmask_oracle as orc
from test_gpu_configs import sample_cols, sample_rows

Q, D, H2, P2 = fm.FM_CUT_QUEUED, fm.FM_CUT_DIRECT, fm.FM_CUT_HALVED, fm.FM_CUT_PAIRED

# H, N, d and the cuts of forward, dQ and dK/dV on 256 compute units
BANDS = [
    (16, 4096, 128, (Q, Q, D)),     # one round of 128-row units off the queues, setup in one launch, for the rows only
    (15, 4000, 128, (Q, Q, D)),     # the same, ragged
    (8, 8192, 128, (Q, Q, D)),      # the same with the setup in three launches
    (20, 2500, 128, (Q, Q, D)),
    (3, 16320, 64, (Q, Q, H2)),     # d = 64: queued dQ with halved keys
    (3, 16512, 64, (Q, Q, Q)),      # one round of keys, long: queued
    (1, 24576, 128, (P2, P2, Q)),   # queues and setup for the keys only
    (1, 40960, 64, (Q, Q, Q)),
    (2, 16384, 128, (P2, P2, H2)),  # the longest halved keys of a full round
    (1, 24500, 128, (P2, P2, H2)),  # ragged: halved at any length
    (520, 640, 128, (Q, Q, Q)),     # many slices: setup of short sequences in three launches
    (1100, 200, 64, (Q, Q, Q)),
]
IDS = [f"{H}x{N}-d{d}" for H, N, d, _ in BANDS]


@pytest.mark.parametrize("H,N,d,cuts", BANDS, ids=IDS)
def test_band_takes_its_cuts(H, N, d, cuts):
    passes = (fm.FM_PASS_FWD, fm.FM_PASS_BWD_DQ, fm.FM_PASS_BWD_DKDV)
    assert tuple(fm.flashmask_work_cut(p, 1, H, H, N, d, compute_units=256) for p in passes) == cuts


def test_queued_keys_never_meet_direct_rows():
    """The backward's cuts go together as they are: where the keys are queued, the rows are queued, halved or paired."""
    seen = set()
    for cus in (32, 104, 256, 304):
        for d in (64, 128):
            for N in (1, 128, 500, 512, 513, 1024, 2048, 2176, 3000, 4096, 8192, 8200, 16384, 32768, 131072):
                for Hk in (1, 2, 7, 16, 64, 255, 600, 2100):
                    for group in (1, 4):
                        size = (1, Hk * group, Hk, N, d)
                        if size[1] * N > 1 << 27:
                            continue
                        dq, dkdv = (fm.flashmask_work_cut(p, *size, compute_units=cus)
                                    for p in (fm.FM_PASS_BWD_DQ, fm.FM_PASS_BWD_DKDV))
                        seen.add((dq, dkdv))
                        assert (dq, dkdv) != (D, Q), size
    assert {(Q, Q), (Q, D), (Q, H2), (P2, Q), (H2, H2), (D, D)} <= seen


# B, H, H_kv, N, d; launches of the forward's and of the backward's setup on 256 compute units
@pytest.mark.parametrize("B,H,Hk,N,d,launches", [
    (1, 2, 2, 512, 128, (0, 0)), (16, 4, 4, 2048, 128, (1, 1)), (1, 16, 16, 4096, 128, (1, 1)), (1, 8, 8, 8192, 128, (3, 3)),
    (1, 24, 24, 4224, 64, (3, 3)),
    (1, 503, 503, 640, 128, (1, 3)), (1, 504, 504, 640, 128, (3, 3)),       # 256 and 264 workgroups a pass
    (4, 60, 60, 640, 64, (1, 1)), (4, 62, 62, 640, 64, (1, 3)), (8, 256, 128, 200, 64, (3, 3)), (1, 1500, 1500, 128, 128, (3, 3)),
])
def test_setup_launches(B, H, Hk, N, d, launches):
    assert tuple(fm.flashmask_setup_launches(p, B, H, Hk, N, d, compute_units=256)
                 for p in (fm.FM_PASS_FWD, fm.FM_PASS_BWD)) == launches


@pytest.mark.gpu
@pytest.mark.parametrize("H,N,d,cuts", BANDS, ids=IDS)
def test_band(H, N, d, cuts):
    w = workloads.small_workload("causal_document", N, seed=H + N, B=1, H=1, d=d)
    bits, dev, vecs = to_device(w)
    x = {n: dev[n].expand(1, H, N, d).contiguous() for n in ("q", "k", "v", "dout")}
    out, lse = fm.flashmask_fwd(x["q"], x["k"], x["v"], *vecs, w.scale)
    dq, dk, dv = fm.flashmask_bwd(x["q"], x["k"], x["v"], out, lse, x["dout"], *vecs, w.scale)
    torch.cuda.synchronize()
    for name, t in (("out", out), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv)):
        assert torch.equal(t, t[:, :1].expand_as(t)), f"{name}: heads differ"
        assert torch.isfinite(t).all(), f"{name} has non-finite values"
    rng = np.random.default_rng(H + N)
    vec = w.vectors[0]
    rows, cols = sample_rows(w, vec, rng, 48), sample_cols(w, vec, rng, 2048)
    host = [f64(bits[n][0, 0]) for n in ("q", "k", "v", "dout")]
    what = f"H={H} N={N} d={d}"
    ro, rl = orc.forward_rows(*host[:3], *vec, w.scale, rows)
    check_fwd(bf16_to_np(out[0, 0])[rows], lse[0, 0].cpu().numpy()[rows], ro, rl, what)
    check_bwd(bf16_to_np(dq[0, 0])[rows], orc.backward_rows(*host, *vec, w.scale, rows), "dq", what)
    rdk, rdv = orc.backward_cols(*host, *vec, w.scale, cols)
    check_bwd(bf16_to_np(dk[0, 0])[cols], rdk, "dk", what)
    check_bwd(bf16_to_np(dv[0, 0])[cols], rdv, "dv", what)


@pytest.mark.gpu
@pytest.mark.parametrize("H,N,d,cut", [(2, 512, 64, H2), (3, 1500, 128, H2), (24, 1024, 128, P2), (64, 1024, 128, D),
                                       (160, 1000, 128, Q), (200, 1152, 64, Q)])
def test_same_call_same_bits(H, N, d, cut):
    """Every cut repeats itself bit for bit, whatever the workspace holds."""
    assert fm.flashmask_work_cut(fm.FM_PASS_FWD, 1, H, H, N, d, compute_units=256) == cut
    w = workloads.small_workload("random_intervals", N, seed=3, B=1, H=H, d=d)
    _, dev, vecs = to_device(w)
    x = [dev[n] for n in ("q", "k", "v", "dout")]
    ws = torch.empty(max(fm.flashmask_workspace_bytes(p, 1, H, N, d) for p in (fm.FM_PASS_FWD, fm.FM_PASS_BWD)),
                     dtype=torch.uint8, device="cuda")
    first = None
    for fill in (0, 255, 127):
        ws.fill_(fill)
        out, lse = fm.flashmask_fwd(*x[:3], *vecs, w.scale, workspace=ws)
        ws.fill_(fill)
        results = (out, lse, *fm.flashmask_bwd(*x[:3], out, lse, x[3], *vecs, w.scale, workspace=ws))
        torch.cuda.synchronize()
        first = first or results
        for name, a, b in zip(("out", "lse", "dq", "dk", "dv"), first, results):
            assert torch.equal(a, b), f"{name} differs from the first call"
