"""GPU: sizes on the direct side of the lines up to which blocks taken in step need no order (fm_in_step, forward units that all
run at once, keys of two rounds at 16384 tokens), against the oracle like the bands of test_gpu_cut_bands.py."""
import pytest

import test_gpu_cut_bands as bands
from test_gpu_cut_bands import D, H2, Q

# H, N, d and the cuts of forward, dQ and dK/dV on 256 compute units
SIZES = [
    (48, 2048, 128, (D, D, D)), (40, 1921, 128, (D, D, D)), (150, 600, 128, (D, D, D)),   # up to three units a compute unit
    (24, 4096, 64, (D, D, D)), (20, 4000, 64, (D, D, D)), (150, 600, 64, (D, D, D)),
    (12, 8192, 64, (D, Q, Q)), (11, 8115, 64, (D, Q, Q)),                                 # forward alone: one round
    (4, 16384, 128, (Q, Q, D)), (4, 16290, 128, (Q, Q, D)),
    (49, 2048, 128, (Q, Q, Q)), (25, 4096, 64, (Q, Q, Q)), (16, 4096, 64, (H2, H2, H2)),  # beyond, and the halved ones below
]
IDS = [f"{H}x{N}-d{d}" for H, N, d, _ in SIZES]


@pytest.mark.parametrize("H,N,d,cuts", SIZES, ids=IDS)
def test_size_takes_its_cuts(H, N, d, cuts):
    bands.test_band_takes_its_cuts(H, N, d, cuts)


@pytest.mark.parametrize("H,Hk,N,cut", [(12, 6, 8192, D), (12, 6, 8115, Q), (16, 4, 5200, Q), (16, 4, 5100, D), (12, 12, 8115, D)])
def test_forward_of_one_round_with_grouped_heads(H, Hk, N, cut):
    """d = 64: ragged lengths of grouped heads are queued beyond 5120 tokens, where direct units took 1.05 times as long."""
    assert bands.fm.flashmask_work_cut(bands.fm.FM_PASS_FWD, 1, H, Hk, N, 64, compute_units=256) == cut


@pytest.mark.gpu
@pytest.mark.parametrize("H,N,d,cuts", SIZES, ids=IDS)
def test_size(H, N, d, cuts):
    bands.test_band(H, N, d, cuts)
