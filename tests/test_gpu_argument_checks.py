"""GPU: every tensor argument of the contiguous entry points with a wrong type, a wrong shape, a wrong stride or on the
host is refused with a FlashMaskError before anything is launched."""
import pytest
import torch

pytestmark = pytest.mark.gpu

B, H, N, D = 2, 3, 160, 64


def _arguments(call):
    big = {n: torch.zeros((B, H, N, D), dtype=torch.bfloat16, device="cuda") for n in ("q", "k", "v", "out", "dout")}
    big["lse"] = torch.zeros((B, H, N), dtype=torch.float32, device="cuda")
    bounds = {n: torch.zeros((B, N), dtype=torch.int32, device="cuda") for n in ("lts", "lte", "uts", "ute")}
    names = {"fwd": ("q", "k", "v"), "fwd_noalloc": ("q", "k", "v"), "bwd": ("q", "k", "v", "out", "lse", "dout")}[call]
    args = {n: big[n] for n in names} | bounds | {"scale": 0.125}
    return args | ({"out": big["out"], "lse": big["lse"]} if call == "fwd_noalloc" else {})


@pytest.mark.parametrize("call", ["fwd", "fwd_noalloc", "bwd"])
def test_each_wrong_tensor_is_refused(call):
    import paper_2410_01359_amd as fm
    entry = getattr(fm, "flashmask_" + call)
    args = _arguments(call)
    entry(**args)
    for name, t in args.items():
        if name == "scale":
            continue
        longer = torch.zeros((*t.shape[:2], t.shape[2] + 8, *t.shape[3:]) if t.dim() > 2 else (B, N + 8),
                             dtype=t.dtype, device="cuda")
        strided = torch.zeros((*t.shape[:-1], 2 * t.shape[-1]), dtype=t.dtype, device="cuda")[..., ::2]
        for wrong in (t.cpu(), t.to(torch.float16), strided, longer):
            with pytest.raises(fm.FlashMaskError):
                entry(**(args | {name: wrong}))
    torch.cuda.synchronize()
