"""GPU: problems small enough for direct units (no setup launches, halved units whose tiles are dealt to two pairs of
waves) against the oracle, at the sizes where the split can go wrong: one tile (one pair of waves has nothing), odd
tile counts, row blocks with a few real rows, several passes over the list of key blocks."""
import numpy as np
import pytest
import torch

import workloads
from gpu_util import bf16_to_np, check_bwd, check_fwd, f64, to_device
from oracle import flashmask_oracle as orc
from test_gpu_backward import compare_all, run_fwd_bwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["full", "causal", "shared_question", "random_intervals"])
@pytest.mark.parametrize("N,d", [(64, 128), (128, 128), (192, 64), (450, 128), (2176, 64), (2176, 128)])
def test_direct_units(kind, N, d):
    w = workloads.small_workload(kind, N, seed=41 + N, B=1, H=3, d=d)
    compare_all(w, *run_fwd_bwd(w), f"{kind} N={N} d={d}")


@pytest.mark.parametrize("kind", ["causal", "document"])
def test_direct_units_grouped_heads(kind):
    """Strided storage and grouped K/V heads on the direct path, dead rows included."""
    import paper_2410_01359_amd as fm
    B, H, Hk, N, d = 1, 6, 2, 520, 128
    w = workloads.small_workload(kind, N, seed=7, B=B, H=H, d=d)
    lts, lte, uts, ute = (v.copy() for v in w.vectors[0])
    uts[:], ute[:] = 0, np.maximum(ute, 3)                 # rows 0..2 see nothing
    w.vectors = [(lts, lte, uts, ute)]
    bits, dev, vecs = to_device(w)
    strided = {n: (dev[n][:, :Hk] if n in ("k", "v") else dev[n]).transpose(1, 2).contiguous().transpose(1, 2)
               for n in ("q", "k", "v", "dout")}
    out, lse = fm.flashmask_fwd_ex(strided["q"], strided["k"], strided["v"], *vecs, w.scale)
    dq, dk, dv = fm.flashmask_bwd_ex(strided["q"], strided["k"], strided["v"], out, lse, strided["dout"], *vecs, w.scale)
    torch.cuda.synchronize()
    for hk in range(Hk):
        heads = range(hk * H // Hk, (hk + 1) * H // Hk)
        k, v = f64(bits["k"][0, hk]), f64(bits["v"][0, hk])
        sdk, sdv = np.zeros((N, d)), np.zeros((N, d))
        for h in heads:
            rdq, rdk, rdv, ro, rl = orc.backward(f64(bits["q"][0, h]), k, v, f64(bits["dout"][0, h]), *w.vectors[0], w.scale)
            check_fwd(bf16_to_np(out[0, h]), lse[0, h].cpu().numpy(), ro, rl, f"{kind} h={h}")
            check_bwd(bf16_to_np(dq[0, h]), rdq, "dq", f"{kind} h={h}")
            sdk += rdk
            sdv += rdv
        check_bwd(bf16_to_np(dk[0, hk]), sdk, "dk", f"{kind} hk={hk}")
        check_bwd(bf16_to_np(dv[0, hk]), sdv, "dv", f"{kind} hk={hk}")


def test_direct_units_long_list():
    """More key blocks than one pass over the list holds (65536 columns), forward."""
    import paper_2410_01359_amd as fm
    N, d = 65536 + 200, 64
    w = workloads.small_workload("sliding_window", N, seed=3, B=1, H=1, d=d)
    j = np.arange(N)
    lts, lte, uts, ute = (v.copy() for v in w.vectors[0])
    lts[:] = np.minimum(j + 70, N)
    lts[::4096] = N                                        # a few keys stay visible: live blocks all over the sequence
    w.vectors = [(lts, lte, uts, ute)]
    bits, dev, vecs = to_device(w, ("q", "k", "v"))
    out, lse = fm.flashmask_fwd(dev["q"], dev["k"], dev["v"], *vecs, w.scale)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(0, 70), np.arange(32700, 32840), np.arange(N - 130, N)]))
    q, k, v = (f64(bits[n][0, 0]) for n in ("q", "k", "v"))
    for r in rows:
        seen = ~(((r >= lts) & (r < lte)) | ((r >= uts) & (r < ute)))
        s = (k[seen] @ q[r]) * w.scale
        p = np.exp(s - s.max())
        ref_o, ref_l = (p @ v[seen]) / p.sum(), s.max() + np.log(p.sum())
        check_fwd(bf16_to_np(out[0, 0, r:r + 1]), lse[0, 0, r:r + 1].cpu().numpy(), ref_o[None], np.array([ref_l]), f"row {r}")
