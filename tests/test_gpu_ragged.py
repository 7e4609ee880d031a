"""GPU: sequence lengths that are not a multiple of 128, several batch rows (so that the rows of the bound vectors
start at addresses that are only 4-byte aligned), and bounds at the ends of the int32 range."""
import numpy as np
import pytest

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
