"""Performance cases of the FlashMask attention path, through the package's public entry points.

A case is one pass of what a user of the library has it do: a training step's attention (forward,
then backward with the upstream gradient) or a forward alone (prefill).  The cases run from a call that
is all latency (N = 512, two heads) to one head group of a 131072-token sequence, over both head
dimensions, lengths that are and are not multiples of 128, contiguous [B,H,N,d] tensors, [B,N,H,d]
storage with grouped K/V heads, and the mask families of the paper's own kernel benchmark.

Fields of a case:
  mode    "train" (flashmask_fwd + flashmask_bwd), "forward" (flashmask_fwd) or "noalloc"
          (flashmask_fwd_noalloc: outputs and scratch that exist before the call)
  packed  tensors stored [B,N,H,d] and passed as strided views to the *_ex entry points; Hk <= H then
          counts the K/V heads (otherwise Hk == H)
  B, H, Hk, N, d
  mask    family; `size` is its parameter (documents or samples per sequence, window, prefix length) and
          `mask_seed` draws the document lengths.  The mask belongs to the case, the tensors to the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2410_01359_amd as fm

_MODES = ("train", "forward", "noalloc")


def _case(name, mode, B, H, N, d, mask, size=0, Hk=None, packed=False, mask_seed=7):
    return {"name": name, "mode": mode, "B": B, "H": H, "Hk": Hk or H, "N": N, "d": d, "mask": mask, "size": size,
            "packed": packed, "mask_seed": mask_seed}


def listed():
    return [
        # the smallest training call: three packed documents, two heads; nothing but latency
        _case("train_docs_512", "train", 1, 2, 512, 64, "causal_document", 3),
        # a short prompt of odd length into buffers that a serving loop already holds
        _case("prefill_prompt_333", "noalloc", 1, 8, 333, 128, "causal"),
        # fine-tuning micro-batch, packed to a length that is no multiple of any tile
        _case("train_docs_1000", "train", 4, 8, 1000, 128, "causal_document", 5),
        # the usual fine-tuning shape: projections stored [B,N,H,d], four query heads to a K/V head,
        # preference data (one question, several answers)
        _case("train_gqa_answers_2048", "train", 2, 32, 2048, 128, "shared_question", 2, Hk=8, packed=True),
        # encoder: bidirectional documents, head dimension 64, odd length
        _case("train_encoder_4099", "train", 1, 16, 4099, 64, "document", 6),
        # prefill of one long prompt with grouped K/V heads
        _case("prefill_gqa_8192", "forward", 1, 32, 8192, 128, "causal", Hk=8, packed=True),
        # training on packed documents, two rows of 8192 tokens
        _case("train_docs_8192", "train", 2, 32, 8192, 128, "causal_document", 11),
        # reward-model training, questions with answers packed to 16384 tokens
        _case("train_answers_16384", "train", 1, 32, 16384, 128, "shared_question", 4),
        # long sequence with a causal window: many short rows of tiles
        _case("train_window_32768", "train", 1, 16, 32768, 128, "sliding_window", 1024),
        # prefix-LM, the densest long case, at both head dimensions
        _case("train_prefix_32768", "train", 1, 16, 32768, 128, "prefix_lm", 4096),
        _case("train_prefix_32768_d64", "train", 1, 32, 32768, 64, "prefix_lm", 4096),
        # long-context training: documents of very different lengths in one 131072-token sequence
        _case("train_docs_131072", "train", 1, 8, 131072, 128, "skewed_document", 34),
    ]


_MOST_FLOPS = 16.0e12   # no drawn case costs more than the largest listed one


def draw(rng):
    while True:
        mode = rng.choice(("train", "train", "train", "forward", "noalloc"))
        packed = mode != "noalloc" and rng.random() < 0.35
        N = int(round(math.exp(rng.uniform(math.log(192), math.log(131072)))))
        if rng.random() < 0.5:
            N = max(128, N // 128 * 128)
        d = rng.choice((64, 128, 128))
        H = rng.choice((2, 4, 8, 12, 16, 32))
        Hk = H // rng.choice([g for g in (1, 2, 4) if H % g == 0]) if packed else H
        B = rng.choice((1, 1, 2, 4)) if N <= 16384 else 1
        mask = rng.choice(("causal", "causal_document", "document", "shared_question", "sliding_window", "prefix_lm",
                           "skewed_document"))
        if mask == "shared_question" and N < 512:
            mask = "causal"
        size = 0
        if mask in ("causal_document", "document"):
            size = rng.randint(2, max(2, min(20, N // 128)))
        elif mask == "skewed_document":
            size = rng.randint(2, max(2, min(48, N // 256)))
        elif mask == "shared_question":
            size = rng.randint(1, max(1, min(8, N // 1024)))
        elif mask == "sliding_window":
            size = int(round(math.exp(rng.uniform(math.log(64), math.log(max(128, N // 4))))))
        elif mask == "prefix_lm":
            size = rng.randint(1, max(1, N // 2))
        case = _case("", mode, B, H, N, d, mask, size, Hk=Hk, packed=packed, mask_seed=rng.randint(0, 1 << 30))
        del case["name"]
        if work(case)["flops"] <= _MOST_FLOPS and B * H * N * d <= 8 * 131072 * 128:
            return case


# --- masks: four int32 bounds per key column; row i does not see column j iff LTS <= i < LTE or UTS <= i < UTE
def _partition(rng, N, parts):
    """N as a uniformly drawn sum of `parts` lengths, each at least an eighth of an equal share."""
    floor = max(1, N // (8 * parts))
    cuts = np.sort(rng.integers(0, N - floor * parts + 1, size=parts - 1))
    edges = np.concatenate(([0], cuts, [N - floor * parts]))
    return floor + np.diff(edges)


def _skewed(rng, N, parts):
    """Log-uniform lengths that sum to N: a few documents hold most of the sequence."""
    floor = max(1, min(512, N // (2 * parts)))
    raw = np.exp(rng.uniform(math.log(floor), math.log(N), size=parts))
    lens = np.maximum(np.floor(raw * ((N - floor * parts) / raw.sum())).astype(np.int64) + floor, 1)
    lens[int(np.argmax(lens))] += N - int(lens.sum())
    return lens


def _bounds(case, row):
    """The four bound vectors of one batch row."""
    N, mask, size = case["N"], case["mask"], case["size"]
    rng = np.random.default_rng([case["mask_seed"], row])
    j = np.arange(N, dtype=np.int64)
    lts, lte, uts, ute = np.full(N, N), np.full(N, N), np.zeros(N, np.int64), j.copy()   # causal
    if mask in ("causal_document", "document", "skewed_document"):
        lens = (_skewed if mask == "skewed_document" else _partition)(rng, N, size)
        ends = np.cumsum(lens)
        lts = np.repeat(ends, lens)
        if mask == "document":
            ute = np.repeat(ends - lens, lens)
    elif mask == "shared_question":
        # samples of a question (two fifths) and three answers that do not see each other
        pos = 0
        for total in _partition(rng, N, size):
            question = int(total) * 2 // 5
            end = pos + int(total)
            answers = pos + question + (int(total) - question) * np.arange(4) // 3
            lts[pos:pos + question] = end
            for a0, a1 in zip(answers[:-1], answers[1:]):
                lts[a0:a1] = a1
            pos = end
    elif mask == "sliding_window":
        lts = np.minimum(j + size, N)
    elif mask == "prefix_lm":
        ute[:size] = 0
    return [v.astype(np.int32) for v in (lts, lte, uts, ute)]


def _unmasked(case):
    """Score elements that are not masked, over the batch (per head)."""
    total = 0
    for row in range(case["B"]):
        lts, lte, uts, ute = (v.astype(np.int64) for v in _bounds(case, row))
        # in these families the upper interval ends at or before the lower one starts
        total += int((case["N"] - np.maximum(lte - lts, 0) - np.maximum(ute - uts, 0)).sum())
    return total


def work(case):
    """Each input read once and each output written once; two matrix products forward, five backward."""
    B, H, Hk, N, d = (case[k] for k in ("B", "H", "Hk", "N", "d"))
    q, kv, lse, mask = 2 * B * H * N * d, 2 * B * Hk * N * d, 4 * B * H * N, 16 * B * N
    flops = 4 * d * H * _unmasked(case)
    moved = 2 * q + 2 * kv + lse + mask                         # q, k, v -> out, lse
    if case["mode"] == "train":
        flops += 10 * d * H * _unmasked(case)
        moved += 4 * q + 4 * kv + lse + mask                    # q, k, v, out, lse, dout -> dq, dk, dv
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    # bf16 results of bf16 products: rounding P and dS to bf16 and the results to bf16 (2^-9 relative each)
    # leaves 0.0025 to 0.003 against float64, whatever the length; two implementations differ by less than the sum
    return {"rel": 1e-2}


def prepare(case, seed):
    B, H, Hk, N, d, mode = (case[k] for k in ("B", "H", "Hk", "N", "d", "mode"))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def tensor(heads):
        shape = (B, N, heads, d) if case["packed"] else (B, heads, N, d)
        x = torch.randn(shape, device="cuda", dtype=torch.bfloat16, generator=gen)
        return x.transpose(1, 2) if case["packed"] else x

    rows = [_bounds(case, row) for row in range(B)]
    state = {"mode": mode, "packed": case["packed"], "scale": 1.0 / math.sqrt(d),
             "q": tensor(H), "k": tensor(Hk), "v": tensor(Hk),
             "mask": tuple(torch.from_numpy(np.stack([r[a] for r in rows])).cuda() for a in range(4))}
    if mode == "train":
        state["dout"] = tensor(H)
    if mode == "noalloc":
        state["out"] = torch.empty((B, H, N, d), device="cuda", dtype=torch.bfloat16)
        state["lse"] = torch.empty((B, H, N), device="cuda", dtype=torch.float32)
    else:   # the scratch a training or serving program keeps for its shape
        passes = (fm.FM_PASS_FWD, fm.FM_PASS_BWD) if mode == "train" else (fm.FM_PASS_FWD,)
        need = max(fm.flashmask_workspace_bytes(p, B, H, N, d) for p in passes)
        state["workspace"] = torch.empty(max(need, 256), device="cuda", dtype=torch.uint8)
    return state


def run(state):
    q, k, v, mask, scale = (state[n] for n in ("q", "k", "v", "mask", "scale"))
    if state["mode"] == "noalloc":
        return fm.flashmask_fwd_noalloc(q, k, v, *mask, scale, state["out"], state["lse"])
    forward, backward = (fm.flashmask_fwd_ex, fm.flashmask_bwd_ex) if state["packed"] else (fm.flashmask_fwd, fm.flashmask_bwd)
    out, lse = forward(q, k, v, *mask, scale, workspace=state["workspace"])
    if state["mode"] == "forward":
        return out, lse
    dq, dk, dv = backward(q, k, v, out, lse, state["dout"], *mask, scale, workspace=state["workspace"])
    return out, lse, dq, dk, dv
