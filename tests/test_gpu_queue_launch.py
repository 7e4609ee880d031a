"""GPU: launches over the unit queues at the unit counts where the handing out of tickets changes: a few more units than
run at once, slices (batch row, head) that do not fill a round of eight queues.  (Launches of one round, where every
workgroup has its ticket in its number: test_gpu_cut_bands.py.)"""
import numpy as np
import pytest
import torch

import paper_2410_01359_amd as fm
import workloads
from gpu_util import bf16_to_np, check_bwd, check_fwd, f64, to_device
from oracle import flashmask_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,N", [(64, 1024), (65, 1024), (43, 1536), (103, 640), (129, 700), (7, 16384 - 64)])
def test_every_head_alike(H, N, d):
    """The same tensors in every head: one head against the oracle, all others bit for bit."""
    w = workloads.small_workload("causal_document", N, seed=H + N, B=1, H=1, d=d)
    bits, dev, vecs = to_device(w)
    x = {n: dev[n].expand(1, H, N, d).contiguous() for n in ("q", "k", "v", "dout")}
    out, lse = fm.flashmask_fwd(x["q"], x["k"], x["v"], *vecs, w.scale)
    dq, dk, dv = fm.flashmask_bwd(x["q"], x["k"], x["v"], out, lse, x["dout"], *vecs, w.scale)
    torch.cuda.synchronize()
    for name, t in (("out", out), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv)):
        assert torch.equal(t, t[:, :1].expand_as(t)), f"{name}: heads differ"
    if N > 4096:
        return
    q, k, v, do = (f64(bits[n][0, 0]) for n in ("q", "k", "v", "dout"))
    rdq, rdk, rdv, ro, rl = orc.backward(q, k, v, do, *w.vectors[0], w.scale)
    check_fwd(bf16_to_np(out[0, 0]), lse[0, 0].cpu().numpy(), ro, rl, f"H={H} N={N} d={d}")
    for name, got, ref in (("dq", dq, rdq), ("dk", dk, rdk), ("dv", dv, rdv)):
        check_bwd(bf16_to_np(got[0, 0]), ref, name, f"H={H} N={N} d={d}")


# Some of the sizes above take direct units; these reach the queues, with a few units more than a loop runs at once (two or
# three workgroups to a compute unit in the row-parallel loops, two for the keys at d = 64) and one, three or five slices more than
# fill rounds of eight queues.
Q, D = fm.FM_CUT_QUEUED, fm.FM_CUT_DIRECT
PAST_ONE_ROUND = [(17, 4096, 128, (Q, Q, Q)), (19, 3500, 128, (Q, Q, Q)), (13, 5250, 128, (Q, Q, Q)), (25, 4096, 64, (Q, Q, Q)),
                  (27, 3650, 64, (Q, Q, Q)), (17, 4224, 64, (D, Q, Q))]


@pytest.mark.parametrize("H,N,d,cuts", PAST_ONE_ROUND, ids=[f"{H}x{N}-d{d}" for H, N, d, _ in PAST_ONE_ROUND])
def test_every_head_alike_past_one_round(H, N, d, cuts):
    passes = (fm.FM_PASS_FWD, fm.FM_PASS_BWD_DQ, fm.FM_PASS_BWD_DKDV)
    assert tuple(fm.flashmask_work_cut(p, 1, H, H, N, d, compute_units=256) for p in passes) == cuts
    test_every_head_alike(H, N, d)


@pytest.mark.parametrize("B,H,N", [(1, 64, 1024), (1, 7, 640), (3, 5, 384), (2, 12, 1152), (1, 1, 128)])
def test_units_lie_within_the_tickets(B, H, N):
    """No queue is longer than the launch's ticket count: whole rounds of slices, then a half, a quarter and an eighth
    (rounded up) of the slices left over."""
    w = workloads.small_workload("causal", N, seed=1, B=B, H=H, d=64)
    vecs = [torch.from_numpy(v).cuda() for v in w.stacked_vectors()]
    for pass_id in (fm.FM_PASS_FWD, fm.FM_PASS_BWD_DQ, fm.FM_PASS_BWD_DKDV):
        rec = fm.flashmask_unit_queues(pass_id, *vecs, H, 64).cpu().numpy()
        slices, units = B * H, (N + 127) // 128
        r = slices % 8
        longest = slices // 8 * units + (r & 4 and -(-units // 2)) + (r & 2 and -(-units // 4)) + (r & 1 and -(-units // 8))
        assert (rec[8 * longest:, 0] == -1).all()
        assert np.array_equal(np.sort(rec[rec[:, 0] >= 0, 0]), np.arange(slices * units))


@pytest.mark.parametrize("B,H,N", [(1, 3, 64), (2, 1, 2049), (9, 1, 700), (7, 3, 1153), (3, 16, 2048), (2, 8, 4096), (1, 2, 4097),
                                   (2, 9, 4224), (3, 176, 130), (2, 250, 384)])
@pytest.mark.parametrize("kind", ["document", "random_intervals", "sliding_window"])
def test_records_on_both_sides_of_the_one_launch_setup(kind, B, H, N):
    """Every unit's live range is what Equation 4 gives, in the one-launch setup (N <= 4096, few slices) and beyond it."""
    w = workloads.small_workload(kind, N, seed=B + H + N, B=B, H=H, d=64)
    vecs = [torch.from_numpy(v).cuda() for v in w.stacked_vectors()]
    n_pad = -(-N // 128) * 128
    for pass_id in (fm.FM_PASS_FWD, fm.FM_PASS_BWD_DQ, fm.FM_PASS_BWD_DKDV):
        br, bc = fm.flashmask_tile_shape(pass_id, 64)
        rec = fm.flashmask_unit_queues(pass_id, *vecs, H, 64).cpu().numpy()
        rec = rec[rec[:, 0] >= 0]
        rec = rec[np.argsort(rec[:, 0])]
        units = n_pad // 128
        assert len(rec) == B * H * units
        for b in range(B):
            # The columns past the end: masked for every row by both pairs where they are keys of a row; a dK/dV block
            # has the keys that exist (repeating the last one adds nothing to a min or max).
            i32 = np.iinfo(np.int32)
            mm = []
            for v, p in zip(w.stacked_vectors(), (i32.min, i32.max, i32.min, i32.max)):
                how = {"mode": "edge"} if pass_id == fm.FM_PASS_BWD_DKDV else {"constant_values": p}
                mm.append(np.pad(v[b].astype(np.int64), (0, n_pad - N), **how).reshape(-1, bc))
            r0 = np.arange(0, N, br)[:, None]
            r1 = np.minimum(r0 + br, N)
            full = ((r0 >= mm[0].max(1)) & (r1 <= mm[1].min(1))) | ((r0 >= mm[2].max(1)) & (r1 <= mm[3].min(1)))
            live = ~full if pass_id != fm.FM_PASS_BWD_DKDV else ~full.T
            lo = np.where(live.any(1), live.argmax(1), 0)
            hi = np.where(live.any(1), live.shape[1] - live[:, ::-1].argmax(1), 0)
            for h in range(H):
                got = rec[(b * H + h) * units:(b * H + h + 1) * units]
                assert np.array_equal(got[:, 1], lo) and np.array_equal(got[:, 2], hi), (pass_id, b, h)


# every loop queued, ragged and not: setup in one launch, in three, and in three for short sequences in many slices
@pytest.mark.parametrize("H,N,d,launches", [(160, 1000, 128, 1), (200, 1100, 64, 1), (24, 4099, 64, 3), (24, 4352, 128, 3),
                                            (520, 600, 128, 3), (1100, 200, 64, 3)])
@pytest.mark.parametrize("kind", ["document", "random_intervals", "sliding_window"])
def test_calls_follow_these_records(kind, H, N, d, launches):
    """What flashmask_unit_queues returns is what an attention call builds: the call's workspace holds the same records in the
    same queues (the forward's, and both of the backward's, whose tables one launch forms together)."""
    w = workloads.small_workload(kind, N, seed=H + N, B=1, H=1, d=d)
    _, dev, vecs = to_device(w)
    x = {n: dev[n].expand(1, H, N, d).contiguous() for n in ("q", "k", "v", "dout")}
    for p in (fm.FM_PASS_FWD, fm.FM_PASS_BWD):
        assert fm.flashmask_setup_launches(p, 1, H, H, N, d) == launches
    ws = [torch.zeros(fm.flashmask_workspace_bytes(p, 1, H, N, d), dtype=torch.uint8, device="cuda")
          for p in (fm.FM_PASS_FWD, fm.FM_PASS_BWD)]
    out, lse = fm.flashmask_fwd(x["q"], x["k"], x["v"], *vecs, w.scale, workspace=ws[0])
    fm.flashmask_bwd(x["q"], x["k"], x["v"], out, lse, x["dout"], *vecs, w.scale, workspace=ws[1])
    held = [t.cpu().numpy().view(np.int32).reshape(-1, 4) for t in ws]
    for pass_id, where in ((fm.FM_PASS_FWD, 0), (fm.FM_PASS_BWD_DQ, 1), (fm.FM_PASS_BWD_DKDV, 1)):
        assert fm.flashmask_work_cut(pass_id, 1, H, H, N, d) == fm.FM_CUT_QUEUED
        rec = fm.flashmask_unit_queues(pass_id, *vecs, H, d).cpu().numpy()
        assert _holds(held[where], rec), f"pass {pass_id}: the call's records are others"


def _by_queue(rec):
    """Records by queue and unit: units of one rank have no fixed order within their queue."""
    rows = np.column_stack([np.arange(len(rec)) % 8, rec])
    return rows[np.lexsort(rows.T[::-1])]


def _holds(rows, rec):
    """Whether a stretch of `rows` is `rec` up to the order within a queue; where its columns add up to rec's, it is compared."""
    sums = np.vstack([np.zeros((1, 4), np.int64), np.cumsum(rows, axis=0, dtype=np.int64)])
    starts = np.nonzero((sums[len(rec):] - sums[:-len(rec)] == rec.sum(axis=0, dtype=np.int64)).all(axis=1))[0]
    return any(np.array_equal(_by_queue(rows[i:i + len(rec)]), _by_queue(rec)) for i in starts)
