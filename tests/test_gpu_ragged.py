"""GPU: sequence lengths that are not a multiple of 128, several batch rows (so that the rows of the bound vectors
start at addresses that are only 4-byte aligned), and bounds at the ends of the int32 range."""
import numpy as np
import pytest
import torch

import paper_2410_01359_amd as fm
import workloads
from test_gpu_backward import compare_all, run_fwd_bwd

pytestmark = pytest.mark.gpu


# one row past a tile, one short of it, a last row block with one real row in its last wave, and long enough for a
# last row block whose live key blocks are a small part of the sequence
@pytest.mark.parametrize("kind", ["document", "causal_document", "sliding_window", "random_intervals"])
@pytest.mark.parametrize("N,d", [(65, 128), (127, 64), (225, 128), (1283, 64), (1283, 128)])
def test_ragged_batches(kind, N, d):
    w = workloads.small_workload(kind, N, seed=17 + N, B=3, H=2, d=d)
    compare_all(w, *run_fwd_bwd(w), f"{kind} N={N} d={d} B=3")


@pytest.mark.parametrize("N,d", [(384, 128), (300, 64)])
def test_bounds_at_the_ends_of_int32(N, d):
    """An interval as long as int32 allows masks its key for every row, like any other that covers all rows."""
    w = workloads.small_workload("causal", N, seed=29, B=1, H=2, d=d)
    lts, lte, uts, ute = (v.copy() for v in w.vectors[0])
    i32 = np.iinfo(np.int32)
    lts[5:90:3], lte[5:90:3] = i32.min, i32.max
    uts[100:200:7], ute[100:200:7] = i32.min, i32.max
    lts[201:260:5], lte[201:260:5] = i32.max, i32.min      # empty
    uts[3:50:9] = i32.min                                   # from row 0, as before
    w.vectors = [(lts, lte, uts, ute)]
    compare_all(w, *run_fwd_bwd(w), f"int32 ends N={N} d={d}")


@pytest.mark.parametrize("H,N,d", [(1, 24576, 128), (12, 4096, 128), (2, 24576, 64)])
def test_the_columns_that_do_not_exist_add_no_tiles(H, N, d):
    """dK/dV units that run without queues: a window over one key less takes about as long as over N keys (if the last
    key block's padded columns counted as masked keys, its chain would be the whole sequence: 2 to 6 times as long)."""
    times = []
    for n in (N, N - 1):
        vecs = [torch.from_numpy(x).cuda()[None] for x in workloads.sliding_window_mask(n, 256)]
        q, k, v, dout = (torch.randn((1, H, n, d), device="cuda", dtype=torch.bfloat16) for _ in range(4))
        out, lse = fm.flashmask_fwd(q, k, v, *vecs, d ** -0.5)
        passes = []
        for _ in range(8):
            ends = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ends[0].record()
            fm.flashmask_bwd(q, k, v, out, lse, dout, *vecs, d ** -0.5)
            ends[1].record()
            ends[1].synchronize()
            passes.append(ends[0].elapsed_time(ends[1]))
        times.append(min(passes))
    assert times[1] < 1.7 * times[0], times


@pytest.mark.parametrize("H,N,d", [(40, 8192, 128), (16, 32768, 64), (16, 4224, 64)])
def test_the_columns_that_do_not_exist_add_no_tiles_to_queued_units(H, N, d):
    """The same for dK/dV units off the queues.  (With the last key block live for every row above the diagonal, one key
    less took 1.71, 2.96 and 2.28 times as long at these sizes; it takes 1.10, 1.06 and 1.05 times.)  And exactly, in the
    live ranges: the last key block reaches as far as its rows, and a row block no further than its own diagonal."""
    n = N - 1
    assert fm.flashmask_work_cut(fm.FM_PASS_BWD_DKDV, 1, H, H, n, d, compute_units=256) == fm.FM_CUT_QUEUED
    vecs = [torch.from_numpy(x).cuda()[None] for x in workloads.sliding_window_mask(n, 256)]
    for pass_id in (fm.FM_PASS_FWD, fm.FM_PASS_BWD_DQ, fm.FM_PASS_BWD_DKDV):
        br, bc = fm.flashmask_tile_shape(pass_id, d)
        rec = fm.flashmask_unit_queues(pass_id, *vecs, H, d).cpu().numpy()
        rec = rec[np.argsort(rec[:, 0])][-H * (N // 128):]
        if pass_id == fm.FM_PASS_BWD_DKDV:
            last = rec[rec[:, 0] % (N // bc) == N // bc - 1]
            assert np.array_equal(last[:, 1:3], np.tile([(N - bc) // br, N // br], (H, 1)))
        else:
            assert np.array_equal(rec[:, 2] * bc, (rec[:, 0] % (N // br) + 1) * br)
    test_the_columns_that_do_not_exist_add_no_tiles(H, N, d)
