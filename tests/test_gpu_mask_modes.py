"""GPU: partially masked tiles of every kind the element mask tells apart -- one interval pair or both, each decided by one
bound (its intervals run to the edge of the rows) or by two -- against the oracle, in every cut of the work, at lengths that
are and are not multiples of the tiles, contiguous and with grouped K/V heads in strided storage.  Neighbouring heads hold
the same tensors, so the first one stands for all."""
import numpy as np
import pytest

import paper_2410_01359_amd as fm
import workloads
from oracle import flashmask_oracle as orc
from test_gpu_direct_cuts import _heads_alike

Q, D, H2, P2 = fm.FM_CUT_QUEUED, fm.FM_CUT_DIRECT, fm.FM_CUT_HALVED, fm.FM_CUT_PAIRED

# mask: the pairs that a tile needs (1 = LT, 2 = UT), those of them that one bound decides
MODES = {"lower_edge": (1, 1), "upper_edge": (2, 2), "both_edges": (3, 3), "lower_inside": (1, 0), "upper_inside": (2, 0),
         "both_inside": (3, 0), "lower_edge_upper_inside": (3, 1), "lower_inside_upper_edge": (3, 2)}

# H, H_kv, N, d and the cuts of forward, dQ and dK/dV on 256 compute units
SHAPES = [(3, 3, 450, 128, (H2, H2, H2)), (3, 3, 512, 64, (H2, H2, H2)), (3, 3, 333, 64, (H2, H2, H2)),
          (24, 24, 1024, 128, (P2, P2, D)), (64, 64, 1024, 128, (D, D, D)), (64, 64, 1000, 64, (D, D, D)),
          (160, 160, 1000, 128, (Q, Q, Q)), (160, 160, 1024, 128, (Q, Q, Q)), (200, 200, 1152, 64, (Q, Q, Q)),
          (200, 200, 1100, 64, (Q, Q, Q)),
          (6, 3, 450, 128, (H2, H2, H2)), (64, 32, 1000, 128, (D, D, D)), (64, 32, 1024, 64, (D, D, H2)),
          (160, 80, 1000, 128, (Q, Q, Q)), (160, 80, 1024, 128, (Q, Q, Q)), (200, 100, 1100, 64, (Q, Q, Q))]


def _bounds(mode, N):
    j = np.arange(N)
    lts, lte, uts, ute = np.full(N, N), np.full(N, N), np.zeros(N, int), np.zeros(N, int)
    if mode.startswith(("lower_edge", "both_edges")):       # row >= LTS decides
        lts = np.minimum(j + 37, N)
    if mode.endswith(("upper_edge", "both_edges")):         # row < UTE decides
        ute = np.maximum(j - 41, 0)
    if mode.startswith(("lower_inside", "both_inside")):    # starts and ends within a tile's rows
        lts, lte = np.minimum(j + 20, N), np.minimum(j + 20 + j % 70, N)
    if mode.endswith(("upper_inside", "both_inside")):
        uts, ute = np.maximum(j - 50, 0), np.maximum(j - 50, 0) + j % 60
    return tuple(v.astype(np.int32) for v in (lts, lte, uts, ute))


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_shape_takes_its_cuts(shape):
    H, Hk, N, d, cuts = shape
    passes = (fm.FM_PASS_FWD, fm.FM_PASS_BWD_DQ, fm.FM_PASS_BWD_DKDV)
    assert tuple(fm.flashmask_work_cut(p, 1, H, Hk, N, d, compute_units=256) for p in passes) == cuts


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("N,br,bc", [(450, 64, 64), (512, 64, 64), (333, 64, 64), (1000, 128, 64), (1024, 128, 64),
                                     (1100, 128, 128), (1152, 128, 128)])
def test_masks_have_tiles_of_their_kind(mode, N, br, bc):
    """At the tiles of the row-parallel loops, there are tiles that need these pairs, with one bound for these of them."""
    mm = orc.minmax_tables(*_bounds(mode, N), bc)
    need = orc.classify_tiles_fast(mm, N, br, bc) >> 4
    r0 = np.arange(0, N, br)[:, None]
    single = 1 * (mm[3] >= np.minimum(r0 + br, N)) + 2 * (mm[4] <= r0)     # min LTE, max UTS
    pairs, one_bound = MODES[mode]
    assert ((need == pairs) & ((single & pairs) == one_bound)).any()


@pytest.mark.gpu
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_mask_mode(mode, shape):
    H, Hk, N, d, _ = shape
    w = workloads.small_workload("causal", N, seed=11 + N, B=1, H=1, d=d)
    w.vectors = [_bounds(mode, N)]
    _heads_alike(w, H, Hk, Hk != H, f"{mode} H={H}/{Hk} N={N} d={d}")
