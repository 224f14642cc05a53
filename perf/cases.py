"""What the performance of this library is measured on: the passes that programs built on the head make, from
one query of a serving loop to the training step at the memory limit, over the sizes of the repository's own
workloads (`paper_2603_25011_amd/inputs.py`), tests and sweeps.

A case is the shape of a batch (B sequences of up to S tokens, hidden size D, vocabulary V), the storage type of
H and W, how long the sequences are, how dense the upstream gradient is, and the way the program calls the
library (`path`):

  serve   one forward without the index through lsr_head_forward_static: a serving loop that hands over no workspace
  encode  one forward without the index through lsr_head_forward, workspace and output kept: bulk encoding
  step    lsr_head_forward + lsr_head_backward, float32 gradients, all buffers kept: a training loop of its own
  micro   the same with `micro` micro-batches whose bfloat16 gradients are summed by lsr_head_backward_ex: the
          first overwrites, the others accumulate
  train   the autograd wrapper, forward and backward, gradients in the dtype of the parameters

Inputs follow the repository's recipe: H ~ N(0,1), W ~ N(0, w_std), bias ~ N(0, w_std), lengths uniform in
[len_lo, len_hi], padding at the end (or a scattered mask), dY ~ N(0,1), of which a share `dy_keep` is not zero.
"""
import math

import torch

from paper_2603_25011_amd import binding as lsr
from paper_2603_25011_amd.autograd import lsr_head

DEV = "cuda:0"


def _case(name, path, B, S, D, V, len_lo, len_hi, dtype="bf16", w_std=0.02, dy_keep=1.0, micro=1, scattered=False):
    return {"name": name, "path": path, "B": B, "S": S, "D": D, "V": V, "len_lo": len_lo, "len_hi": len_hi,
            "dtype": dtype, "w_std": w_std, "dy_keep": dy_keep, "micro": micro, "scattered": scattered}


def listed():
    return [
        # one user query against a 30k vocabulary: the smallest call of a serving loop, latency counts
        _case("serve_one_query", "serve", 1, 32, 768, 30522, 4, 32),
        # a handful of passages encoded as they arrive
        _case("serve_few_documents", "serve", 8, 512, 768, 30522, 128, 512),
        # bulk document encoding at the BERT-base shape
        _case("encode_documents", "encode", 32, 256, 768, 30522, 64, 256),
        # the head in float32 at the size people debug and grad-check with
        _case("tiny_float32_step", "step", 2, 16, 64, 1000, 1, 16, dtype="f32", w_std=0.05),
        # a model kept in float32 (the default dtype of a freshly made module) trained on short texts
        _case("train_float32", "train", 64, 32, 768, 30522, 4, 32, dtype="f32"),
        # query tower of a contrastive step: short sequences, large batch, gradients made sparse by a FLOPS regulariser
        _case("step_queries_sparse", "step", 256, 32, 768, 30522, 4, 32, dy_keep=0.05),
        # odd sizes everywhere: D is not a multiple of the kernels' 64, prime-ish V, scattered mask
        _case("train_ragged", "train", 13, 197, 312, 31091, 60, 197, scattered=True),
        # gradient accumulation over micro-batches, gradients summed in the bfloat16 parameters' own buffers
        _case("micro_batches", "micro", 32, 128, 1024, 30522, 16, 128, micro=2),
        # multilingual vocabulary at base size
        _case("train_multilingual", "train", 16, 256, 768, 250002, 32, 256),
        # large batch of full-length sequences, the shape of the paper's batch sweep
        _case("train_large_batch", "train", 256, 512, 768, 30522, 512, 512),
        # long documents, the sequence-length sweep of the paper at its longest
        _case("step_long_documents", "step", 32, 8192, 768, 30522, 4096, 8192),
        # the multilingual training step at the memory-limit shape
        _case("step_large_multilingual", "step", 64, 512, 1024, 250002, 128, 512),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_LARGEST = 2.0 * 64 * 320 * 1024 * 250002        # forward operations of the largest listed case
_LARGEST_F32 = 2.0 * 64 * 18 * 768 * 30522       # ... of the largest in float32


def draw(rng):
    while True:
        path = rng.choice(["serve", "encode", "step", "step", "micro", "train", "train"])
        dtype = "f32" if path in ("step", "train") and rng.random() < 0.25 else "bf16"
        # hidden sizes of transformer encoders, and now and then any multiple of 8
        D = rng.choice([128, 256, 384, 512, 768, 768, 768, 1024, 1024]) if rng.random() < 0.8 else 8 * rng.randint(9, 128)
        V = _log_int(rng, 20000, 250002)
        if path == "serve":
            B, S = _log_int(rng, 1, 8), _log_int(rng, 16, 512)
        elif dtype == "f32":
            B, S = _log_int(rng, 2, 64), _log_int(rng, 16, 128)
            V = _log_int(rng, 1000, 60000)
        elif rng.random() < 0.15:
            B, S = _log_int(rng, 4, 64), _log_int(rng, 1024, 8192)
        else:
            B, S = _log_int(rng, 8, 256), _log_int(rng, 24, 512)
        full = rng.random() < 0.2
        hi = S
        lo = S if full else max(1, int(S * rng.choice([0.125, 0.25, 0.5])))
        c = _case("", path, B, S, D, V, lo, hi, dtype=dtype,
                  dy_keep=rng.choice([1.0, 1.0, 0.05]) if path != "serve" and path != "encode" else 1.0,
                  micro=rng.choice([2, 3, 4]) if path == "micro" else 1,
                  scattered=not full and rng.random() < 0.2)
        ops = c["micro"] * 2.0 * B * _mean_len(c) * D * V
        if ops <= (_LARGEST_F32 if dtype == "f32" else _LARGEST):
            del c["name"]
            return c


def _mean_len(c):
    return 0.5 * (c["len_lo"] + c["len_hi"])


class State:
    """Inputs of one batch and what a program keeps beside them."""


def _batch(c, gen, head):
    B, S, D, V = c["B"], c["S"], c["D"], c["V"]
    s = State()
    s.shape = (B, S, D, V, lsr.LSR_F32 if c["dtype"] == "f32" else lsr.LSR_BF16)
    td = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    s.H = torch.randn((B, S, D), device=DEV, generator=gen).to(td)
    if head is None:
        s.W = torch.empty((V, D), dtype=td, device=DEV)
        for v0 in range(0, V, 65536):
            n = min(65536, V - v0)
            s.W[v0:v0 + n] = torch.randn((n, D), device=DEV, generator=gen).mul_(c["w_std"]).to(td)
        s.bias = torch.randn((V,), device=DEV, generator=gen).mul_(c["w_std"])
    else:
        s.W, s.bias = head.W, head.bias
    lens = torch.randint(c["len_lo"], c["len_hi"] + 1, (B, 1), device=DEV, generator=gen)
    where = torch.arange(S, device=DEV).expand(B, S)
    if c["scattered"]:
        # the same number of valid tokens at random places
        where = torch.rand((B, S), device=DEV, generator=gen).argsort(dim=1).argsort(dim=1)
    s.mask = (where < lens).to(torch.uint8)
    if c["path"] in ("step", "micro", "train"):
        s.dY = torch.randn((B, V), device=DEV, generator=gen)
        if c["dy_keep"] < 1.0:
            s.dY *= torch.rand((B, V), device=DEV, generator=gen) < c["dy_keep"]
    return s


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    s = _batch(case, gen, None)
    s.path = case["path"]
    B, S, D, V, dt = s.shape
    if s.path == "train":
        for t in (s.H, s.W, s.bias):
            t.requires_grad_(True)
        return s
    s.Y = torch.empty((B, V), dtype=torch.float32, device=DEV)
    s.batches = [s] + [_batch(case, gen, s) for _ in range(case["micro"] - 1)]
    if s.path != "serve":
        s.ws = torch.empty(lsr.lsr_head_workspace_bytes(B, S, D, V, dt, False), dtype=torch.uint8, device=DEV)
    if s.path in ("step", "micro"):
        s.gt = lsr.LSR_BF16 if s.path == "micro" else lsr.LSR_F32
        gd = torch.bfloat16 if s.path == "micro" else torch.float32
        s.I = torch.empty((B, V), dtype=torch.int32, device=DEV)
        s.dH = [torch.empty((B, S, D), dtype=gd, device=DEV) for _ in s.batches]
        s.dW = torch.empty((V, D), dtype=gd, device=DEV)
        s.db = torch.empty((V,), dtype=torch.float32, device=DEV)
        # one workspace serves the overwriting and the accumulating call (their needs are the same)
        n = max(lsr.lsr_head_backward_ex_workspace_bytes(B, S, D, V, dt, s.gt, a) for a in (False, True))
        s.ws_bwd = torch.empty(n, dtype=torch.uint8, device=DEV)
    return s


def run(s):
    if s.path == "serve":
        lsr.lsr_head_forward_static(*s.shape, s.H, s.W, s.bias, s.mask, s.Y, None)
        return s.Y
    if s.path == "encode":
        lsr.lsr_head_forward(*s.shape, s.H, s.W, s.bias, s.mask, s.Y, None, s.ws)
        return s.Y
    if s.path == "step":
        lsr.lsr_head_forward(*s.shape, s.H, s.W, s.bias, s.mask, s.Y, s.I, s.ws)
        lsr.lsr_head_backward(*s.shape, s.H, s.W, s.dY, s.Y, s.I, s.dH[0], s.dW, s.db, s.ws_bwd)
        return {"Y": s.Y, "I": s.I, "dH": s.dH[0], "dW": s.dW, "db": s.db}
    if s.path == "micro":
        # every micro-batch has its own hidden states, whose gradient goes on into the encoder: dH is overwritten
        # (accumulated onto zeros), dW and db are summed over the micro-batches
        for k, b in enumerate(s.batches):
            lsr.lsr_head_forward(*s.shape, b.H, s.W, s.bias, b.mask, s.Y, s.I, s.ws)
            if k:
                s.dH[k].zero_()
            lsr.lsr_head_backward_ex(*s.shape, b.H, s.W, b.dY, s.Y, s.I, s.dH[k], s.dW, s.db, s.gt, k > 0, s.ws_bwd)
        return {"Y": s.Y, "I": s.I, "dH": list(s.dH), "dW": s.dW, "db": s.db}
    Y, I = lsr_head(s.H, s.W, s.bias, s.mask)
    dH, dW, db = torch.autograd.grad(Y, (s.H, s.W, s.bias), s.dY)
    return {"Y": Y.detach(), "I": I, "dH": dH, "dW": dW, "db": db}


def work(case):
    """Every input read once (of H the valid rows), every output written once; the multiplications of valid tokens,
    and for the backward one multiply-add per element of dW and of dH and pair with a gradient (a maximum over a
    sequence is nearly always positive, so all pairs count as active where dY is not zero)."""
    B, S, D, V = case["B"], case["S"], case["D"], case["V"]
    e = 4 if case["dtype"] == "f32" else 2
    tokens = B * _mean_len(case)
    bytes_ = tokens * D * e + B * S + 4 * B * V
    flops = 2.0 * tokens * D * V
    once = V * D * e + 4 * V
    if case["path"] in ("step", "micro", "train"):
        ge = 4 if case["path"] == "step" else e
        bytes_ += 4 * B * V + 4 * B * V + B * S * D * ge           # I, dY, dH
        flops += 4.0 * B * V * case["dy_keep"] * D
        once += V * D * ge + 4 * V                                 # dW, db
    return {"bytes": case["micro"] * bytes_ + once, "flops": case["micro"] * flops}


def tolerance(case):
    """Measured against the same pass in float64 (logits in float64, gradients at its own positions), times four.
    Forward alone: Y within rel 1.2e-7 and max 7e-7 (float32 3.1e-7 and 2.2e-6).  With gradients the arg-max
    decides: up to 2e-6 of the positions are near-ties that another order of the sums decides the other way, and
    each of them moves a whole row g * W of dH and replaces one of the few rows that a row of dW is the sum of
    (rel 2.3e-3 there, single elements by more than the root mean square)."""
    if case["path"] in ("serve", "encode"):
        return {"rel": 1.2e-6, "max": 9e-6} if case["dtype"] == "f32" else {"rel": 5e-7, "max": 3e-6}
    if case["dtype"] == "f32":
        return {"rel": 4e-3, "max": 0.99, "differ": 4e-6}
    return {"rel": 1e-2, "max": 0.99, "differ": 8e-6}


def exact(case, seed):
    """Y and db of the same pass in float64.  I and the sums that it routes (dH, dW) have no such value: near-ties,
    which a correct implementation may decide either way, move whole rows of them (see tolerance)."""
    s = prepare(case, seed)
    batches = s.batches if s.path == "micro" else [s]
    with torch.no_grad():
        Ws, db = s.W.detach(), None
        for b in batches:
            Y = torch.empty((case["B"], case["V"]), dtype=torch.float64, device=DEV)
            rows = [b.H[k][b.mask[k] != 0].double() for k in range(case["B"])]
            for v0 in range(0, case["V"], 16384):
                Wc = Ws[v0:v0 + 16384].double().t().contiguous()
                for k, h in enumerate(rows):
                    Y[k, v0:v0 + 16384] = (h @ Wc).amax(dim=0)
            Y = torch.log1p(torch.relu(Y + s.bias.detach().double()))
            if s.path in ("serve", "encode"):
                return Y
            g = torch.where(Y > 0, b.dY.double() * torch.exp(-Y), torch.zeros_like(Y)).sum(dim=0)
            db = g if db is None else db + g
    return {"Y": Y, "I": None, "dH": [None for _ in batches] if s.path == "micro" else None, "dW": None, "db": db}
