"""Parity of the HIP path against the fp64 oracle, element by element, through the C ABI."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2603_25011_amd import binding as lsr
from paper_2603_25011_amd import inputs as wl
from paper_2603_25011_amd.harness import DeviceHead
from tests import parity

pytestmark = pytest.mark.gpu


def run_case(inp, mask=None, want_index=True, check_bwd=True):
    head = DeviceHead(inp, mask=mask, want_index=want_index)
    head.poison_outputs()
    head.forward()
    torch.cuda.synchronize()
    Y = head.Y.cpu().numpy()
    I = head.I.cpu().numpy() if want_index else None
    _, _, _, stats = parity.compare_forward(inp, Y, I, mask=mask)
    m = inp.mask if mask is None else mask
    empty = ~(m != 0).any(axis=1)
    assert np.all(Y[empty] == 0.0)
    assert np.all(Y >= 0.0)
    if want_index:
        assert np.all(I[empty] == 0)
    if check_bwd and head.has_backward and want_index:
        head.backward()
        torch.cuda.synchronize()
        dH, dW, db = head.dH.cpu().numpy(), head.dW.cpu().numpy(), head.db.cpu().numpy()
        stats.update(parity.compare_backward(inp, I, dH, dW, db, mask=mask))
        # positions that cannot be selected receive exactly zero
        assert np.all(dH[m == 0] == 0.0)
        # same call again: owner-computes sums are bit-reproducible
        head.backward()
        torch.cuda.synchronize()
        assert torch.equal(head.dH.cpu(), torch.from_numpy(dH))
        assert torch.equal(head.dW.cpu(), torch.from_numpy(dW))
        assert torch.equal(head.db.cpu(), torch.from_numpy(db))
    return stats


def test_c1_tiny_fp32_forward_backward():
    print(run_case(wl.make_inputs(wl.WORKLOADS["c1_tiny_f32"])))


@pytest.mark.parametrize("B,S,D,V,len_lo", [
    (20, 32, 128, 700, 1),      # one 32-row block per sequence, short last tile, ragged V
    (7, 48, 64, 300, 5),        # one or two blocks per sequence
    (5, 100, 192, 513, 3),      # up to four blocks per sequence
    (3, 300, 256, 1000, 200),   # sequences that straddle tiles
    (2, 129, 200, 260, 1),      # rows that end inside a slab (D not a multiple of 64)
    (4, 1, 64, 257, 1),         # S = 1: a plain linear layer; few tokens, one launch
    (70, 1, 64, 257, 1),        # S = 1 through the packed forward
    (9, 700, 64, 96, 1),        # long sequences, single narrow vocabulary tile, one K slab
    (300, 20, 64, 520, 1),      # more sequences than the planning pass scans at once; several row groups
    (40, 260, 128, 300, 100),   # several row groups of several tiles each
    (1, 8, 8, 1, 1),            # smallest legal D, one vocabulary entry; few tokens
    (17, 4, 8, 1, 1),           # the same through the packed forward
    (2, 16, 128, 70000, 1),     # vocabulary wide enough that the dH gather runs in three vocabulary chunks
    (48, 200, 64, 70000, 1),    # enough workgroups per CU that the row-group cuts are nudged to whole tiles
    (2, 1024, 64, 300, 900),    # longest sequences whose bucket sort still places through LDS
    (2, 1100, 64, 300, 900),    # just beyond: direct placement
    (3, 40, 64, 9000, 1),       # several sort segments per sequence, the last one short
    (260, 256, 64, 4100, 60),   # a batch whose H slice exceeds L2: the dW gather runs in three launches of 87 sequences
    (2, 130, 128, 132000, 40),  # LDS-tile dW kernel: S just above one copy pass, ragged last vocabulary tile; dH slices dealt over XCDs
    (3, 128, 576, 30000, 1),    # LDS-tile dW kernel, one pass; nine column slices: eight owned by XCDs, one shared
    (2, 512, 64, 262200, 300),  # LDS-tile dW kernel at its longest sequence (four passes), one column slice
    (17, 300, 128, 131100, 50), # LDS-tile dW kernel, three passes, S not a multiple of 128; slice-major dH
])
def test_small_bf16_shapes(B, S, D, V, len_lo):
    inp = wl.make_custom(B, S, D, V, seed=B * 1000 + S, len_lo=len_lo)
    print(run_case(inp))


@pytest.mark.parametrize("B,S,D,V", [
    (450, 12, 64, 700),       # more than 384 sequences, D a multiple of 64: whole-row dW kernel beside the sliced dH gather
    (500, 9, 128, 333),
    (3000, 4, 64, 130),       # batches in the thousands (the 48 KiB staging tile of dW is two rows wide)
    (6144, 2, 64, 40),        # the largest batch the backward takes
])
def test_large_batches_whole_row_dw_beside_sliced_dh(B, S, D, V):
    from paper_2603_25011_amd import binding as b
    plan = b.lsr_head_plan(B, S, D, V, b.LSR_BF16)
    assert plan["dw_tile_rows"] == 0 and plan["dh_buckets_per_wave"] > 0
    inp = wl.make_custom(B, S, D, V, seed=B + S, len_lo=1)
    print(run_case(inp))


# up to 64 tokens: the one launch for few tokens; beyond: the packed forward, with 32-row segments at S = 70 and 8-row segments
@pytest.mark.parametrize("B,S,D,V", [(3, 20, 72, 333), (2, 70, 96, 300), (2, 9, 256, 260), (4, 20, 72, 333), (8, 9, 256, 260)])
def test_fp32_logits_are_the_fma_chain_in_ascending_d(B, S, D, V):
    """Near-ties of float32 logits fall as they do for a scalar loop of FMAs: the arg-max is that loop's.  The chain is
    formed in float64 (the product is exact there) and rounded to float32 after every term; the sum is rounded twice,
    which differs from an FMA about once in 2^29 terms (3 * 10^6 are formed here)."""
    inp = wl.make_custom(B, S, D, V, dtype="f32", seed=D, len_lo=S, w_std=0.05)
    head = DeviceHead(inp)
    head.forward()
    H, W = torch.from_numpy(inp.H).double(), torch.from_numpy(inp.W).double()
    acc = torch.zeros((B, S, V), dtype=torch.float64)
    for d in range(D):
        acc = (acc + H[:, :, None, d] * W[None, None, :, d]).float().double()
    top, first = acc.max(dim=1).values, acc.argmax(dim=1)
    assert torch.equal(head.I.cpu().long(), first)
    Y = torch.log1p(torch.relu(top.float() + torch.from_numpy(inp.bias)).double()).float()
    assert torch.allclose(head.Y.cpu(), Y, rtol=2.0 ** -22, atol=0.0)      # log1pf: within two units in the last place


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,S,D,V,dy_keep", [
    (3, 10, 64, 1000, None),       # four waves per bucket, few buckets; lists of one or two 64-entry blocks per wave
    (2, 5, 64, 3000, 0.02),        # ... lists shorter than a block: waves without entries
    (100, 24, 128, 60000, None),   # four waves per bucket, two vocabulary chunks
    (100, 24, 128, 40000, 0.05),
    (40, 30, 256, 9000, None),     # four waves per bucket
    (3300, 10, 64, 2000, None),    # two waves per bucket (33 000 waves at one)
])
def test_dh_lists_shared_by_waves(B, S, D, V, dy_keep, dtype):
    print(run_case(wl.make_custom(B, S, D, V, dtype=dtype, seed=B + S, len_lo=1, dy_keep=dy_keep)))


def dh_in_float64(B, S, V, g, I, W):
    """dH = sum of g W over the entries of each bucket, and the sum of the magnitudes, in float64 (one sequence at a time)."""
    D = W.shape[1]
    out, size = (torch.empty((B, S, D), dtype=torch.float64, device="cuda") for _ in range(2))
    Wd, Wa = W.double(), W.double().abs()
    for b in range(B):
        m = torch.zeros((S, V), dtype=torch.float64, device="cuda")
        m[I[b].long(), torch.arange(V, device="cuda")] = g[b].double()
        out[b] = m @ Wd
        size[b] = m.abs() @ Wa
    return out, size


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,S,D,V,waves", [
    (2, 16, 64, 2500, 4),
    (3, 9, 72, 34000, 4),          # several vocabulary chunks, the last slice partly filled
    (48, 20, 1024, 8000, 4),       # slices in grid order
    (75, 48, 1024, 9500, 2),
])
def test_shared_lists_around_one_block(B, S, D, V, waves, dtype):
    """Lists of 0, 1, 63, 64, 65, 127, ... entries where waves share a bucket: up to 64 entries are the first wave's alone.
    Y is so small that g = dY.  Every addition rounds to 2^-24 of a sum that the magnitudes bound: a lane adds a list in
    chains of at most ceil(n / 4) entries, then joins lanes and waves."""
    dt = lsr.LSR_F32 if dtype == "f32" else lsr.LSR_BF16
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    if dtype == "bf16":
        assert lsr.lsr_head_plan(B, S, D, V, dt)["dh_waves_per_bucket"] == waves
    g = torch.Generator(device="cuda").manual_seed(V)
    sizes = [0, 1, 63, 64, 65, 127, 128, 129, 255, 256, 257]
    I = torch.empty((B, V), dtype=torch.int32, device="cuda")
    for b in range(B):
        n = [sizes[(b + s) % len(sizes)] for s in range(S - 1)]
        lists = torch.repeat_interleave(torch.arange(S, device="cuda"), torch.tensor(n + [V - sum(n)], device="cuda").clamp(min=0))[:V]
        I[b] = lists[torch.randperm(V, device="cuda", generator=g)].int()
    W = torch.randn((V, D), device="cuda", generator=g).mul_(0.05).to(td)
    H = torch.zeros((B, S, D), device="cuda", dtype=td)
    Y = torch.full((B, V), 1e-30, device="cuda")
    for keep in (1.0, 0.3):
        dY = torch.randn((B, V), device="cuda", generator=g) * (torch.rand((B, V), device="cuda", generator=g) < keep)
        want, size = dh_in_float64(B, S, V, dY, I, W)
        for accumulate in (False, True):
            dH0 = torch.randn((B, S, D), device="cuda", generator=g)
            dH = dH0.clone()
            ws = torch.empty(lsr.lsr_head_backward_ex_workspace_bytes(B, S, D, V, dt), dtype=torch.uint8, device="cuda")
            lsr.lsr_head_backward_ex(B, S, D, V, dt, H, W, dY, Y, I, dH, None, None, lsr.LSR_F32, accumulate, ws)
            if accumulate:
                want, size = want + dH0.double(), size + dH0.double().abs()
            n = torch.zeros((B, S), device="cuda", dtype=torch.float64).scatter_add_(1, I.long(), torch.ones((B, V), device="cuda", dtype=torch.float64))
            assert bool(((dH.double() - want).abs() <= (n[:, :, None] / 4 + 16) * 2.0 ** -24 * size).all())


def test_forward_beyond_the_backward_length_limit():
    # S above 8192 is forward-only
    inp = wl.make_custom(2, 9000, 64, 40, seed=31, len_lo=8000, backward=False)
    print(run_case(inp, check_bwd=False))


def test_fp32_small_shapes():
    print(run_case(wl.make_custom(3, 20, 72, 333, dtype="f32", seed=5, w_std=0.05)))
    # D a multiple of 64 and a vocabulary of three dH chunks
    print(run_case(wl.make_custom(3, 20, 64, 40000, dtype="f32", seed=6, w_std=0.05)))
    # two buckets per wave in the dH gather (about 70 entries per bucket expected)
    print(run_case(wl.make_custom(3, 20, 64, 1000, dtype="f32", seed=8, w_std=0.05)))
    # dW in two launches of 100 sequences (the second adds to the first)
    print(run_case(wl.make_custom(200, 128, 64, 2100, dtype="f32", seed=9, w_std=0.05)))
    # a batch above 192: dW from 16-row tiles whose columns are compacted to the non-zero gradients
    print(run_case(wl.make_custom(200, 6, 64, 100, dtype="f32", seed=7, w_std=0.05)))


@pytest.mark.parametrize("B,S,D,V,len_lo", [
    (1, 1, 8, 1, 1),           # smallest legal shape; few tokens, one launch
    (2, 16, 32, 257, 1),       # few tokens, rows of 128 bytes
    (17, 4, 8, 1, 1),          # one short slab
    (5, 16, 32, 257, 1),       # one slab of 32 through the direct loader
    (5, 64, 96, 300, 1),       # odd slab count, short segments
    (70, 33, 64, 600, 1),      # more than 64 sequences: the search for a chunk's first sequence takes two rounds
    (3, 300, 128, 700, 200),   # sequences longer than a tile
    (90, 90, 40, 513, 1),      # D not a multiple of 32, sequences with and without a second segment
])
def test_fp32_matrix_core_forward(B, S, D, V, len_lo):
    """Float32 logits are sums of D products of float32 values: a sum in any order is within D * 2^-24 of the sum of
    the magnitudes, and Y moves by no more than the logit does."""
    inp = wl.make_custom(B, S, D, V, dtype="f32", seed=B * 1000 + S, len_lo=len_lo, w_std=0.05)
    rng = np.random.default_rng(S)
    for mask in (None, wl.scattered_mask(rng, B, S)):
        head = DeviceHead(inp, mask=mask)
        head.poison_outputs()
        head.forward()
        torch.cuda.synchronize()
        Y, I = head.Y.cpu().numpy(), head.I.cpu().numpy()
        Y_ref, _, _, _ = parity.compare_forward(inp, Y, I, mask=mask)
        size = np.abs(inp.H.astype(np.float64)).max(axis=(0, 1)) @ np.abs(inp.W.astype(np.float64)).max(axis=0)
        assert np.abs(Y - Y_ref).max() <= (D + 4) * 2.0 ** -24 * (size + np.abs(Y_ref).max())
    run_case(inp)


@pytest.mark.parametrize("B,S,D,V,dtype", [
    (1, 1, 8, 1, "bf16"),          # one token, half a k-step, one vocabulary entry
    (1, 64, 768, 32768, "bf16"),   # two row blocks at the largest token count; the widest vocabulary of one round
    (1, 64, 768, 32769, "bf16"),   # one entry more: the tile kernel
    (16, 4, 72, 129, "bf16"),      # odd number of 16-byte chunks; a ragged second workgroup; the most sequences
    (3, 11, 264, 640, "bf16"),     # 33 tokens: the second row block holds one; one k-step behind a batch of loads
    (2, 32, 512, 128, "f32"),      # hidden states beyond the LDS: the tile kernel
    (2, 16, 512, 128, "f32"),      # four batches of loads, one workgroup
    (1, 32, 1088, 300, "f32"),     # the longest float32 rows: eight batches and a half
    (1, 64, 448, 260, "f32"),      # two row blocks and three batches and a half
    (5, 7, 20 * 8, 200, "f32"),
    (8, 8, 512, 131100, "bf16"),   # wide vocabulary, too many sequences for rows of 512: the tile kernel
    (8, 8, 520, 131100, "bf16"),   # workgroups that walk several tiles of the vocabulary, the last one ragged
    (1, 9, 1032, 131072, "bf16"),
])
def test_calls_of_few_tokens(B, S, D, V, dtype):
    """The one-launch forward.  Products are exact in float32, so a logit is within D * 2^-24 of the sum of the
    magnitudes, and Y moves by no more than the logit does.  Scattered masks, an empty sequence, and the same result
    without the index."""
    plan = lsr.lsr_head_plan_ex(B, S, D, V, lsr.LSR_F32 if dtype == "f32" else lsr.LSR_BF16)
    assert plan["fwd_few_tokens"] == ((B, S, D, V) not in ((1, 64, 768, 32769), (2, 32, 512, 128), (8, 8, 512, 131100)))
    inp = wl.make_custom(B, S, D, V, dtype=dtype, seed=B * 100 + S, w_std=0.05, backward=False)
    rng = np.random.default_rng(D)
    m2 = wl.scattered_mask(rng, B, S)
    if B > 1:
        m2[1, :] = 0
    size = np.abs(inp.H.astype(np.float64)).max(axis=(0, 1)) @ np.abs(inp.W.astype(np.float64)).max(axis=0)
    for mask in (None, m2):
        ys = []
        for want_index in (True, False):
            head = DeviceHead(inp, mask=mask, want_index=want_index)
            head.poison_outputs()
            head.forward()
            torch.cuda.synchronize()
            ys.append(head.Y.cpu().numpy())
            if want_index:
                I = head.I.cpu().numpy()
        Y_ref, _, _, _ = parity.compare_forward(inp, ys[0], I, mask=mask, v_chunk=16384)
        assert np.array_equal(ys[0], ys[1])
        assert np.abs(ys[0] - Y_ref).max() <= (D + 4) * 2.0 ** -24 * (size + np.abs(Y_ref).max())


def forward_of(inp, mask, H):
    head = DeviceHead(inp, mask=mask)
    head.H.copy_(H)
    head.poison_outputs()
    head.forward()
    return head.Y, head.I


@pytest.mark.parametrize("B,S,D,V,dtype", [
    (1, 1, 8, 1, "bf16"),
    (1, 32, 768, 1000, "bf16"),
    (1, 64, 896, 300, "bf16"),
    (16, 4, 72, 129, "bf16"),      # odd number of 16-byte chunks
    (3, 11, 264, 640, "bf16"),
    (4, 16, 768, 131100, "bf16"),  # workgroups that walk the vocabulary
    (8, 8, 520, 131100, "bf16"),   # ... with an odd number of chunks
    (1, 8, 512, 131100, "bf16"),
    (1, 1, 8, 1, "f32"),
    (5, 7, 160, 333, "f32"),
    (2, 16, 512, 300, "f32"),
    (1, 64, 448, 260, "f32"),
    (1, 32, 1088, 200, "f32"),
])
def test_calls_of_few_tokens_give_the_bits_of_the_packed_forward(B, S, D, V, dtype):
    """The same tokens as they are, and behind them masked positions up to more than 64 tokens.  Masked positions hold NaN in
    the first call and infinities in the second.  All tokens; scattered ones, with an empty sequence; tokens with
    infinite and with NaN hidden states among them, or an infinite one alone (all logits -inf where its weight is
    positive); none."""
    dt, td = (lsr.LSR_F32, torch.float32) if dtype == "f32" else (lsr.LSR_BF16, torch.bfloat16)
    S2 = 64 // B + 1
    assert lsr.lsr_head_plan_ex(B, S, D, V, dt)["fwd_few_tokens"] == 1
    assert lsr.lsr_head_plan_ex(B, S2, D, V, dt)["fwd_few_tokens"] == 0
    inp = wl.make_custom(B, S, D, V, dtype=dtype, seed=D + S, w_std=0.05, backward=False)
    wide = wl.make_custom(B, S2, D, 1, dtype=dtype, backward=False)      # only the shape counts
    wide = replace(wide, workload=replace(wide.workload, V=V), W=inp.W, bias=inp.bias, W_bits=inp.W_bits)
    rng = np.random.default_rng(V)
    some = wl.scattered_mask(rng, B, S)
    some[B - 1] = 0 if B > 1 else some[B - 1]
    H0 = torch.from_numpy(inp.H).to(td).cuda()
    H1 = H0.clone()
    H1[:, 0, 3] = float("inf")
    H1[:, S // 2, 5] = float("-inf")
    H1[:, S - 1, 1] = float("nan")
    full, none = np.ones((B, S), np.uint8), np.zeros((B, S), np.uint8)
    alone = none.copy()
    alone[:, S // 2] = 1
    for mask, H in ((full, H0), (some, H0), (full, H1), (some, H1), (alone, H1), (none, H0)):
        valid = torch.from_numpy(mask).bool().cuda()[:, :, None]
        Y, I = forward_of(inp, mask, torch.where(valid, H, float("nan")))
        mask2 = np.zeros((B, S2), np.uint8)
        mask2[:, :S] = mask
        Hw = torch.full((B, S2, D), float("inf"), device="cuda", dtype=td)
        Hw[:, :S] = torch.where(valid, H, float("inf"))
        Yw, Iw = forward_of(wide, mask2, Hw)
        torch.cuda.synchronize()
        assert torch.equal(Y, Yw) and torch.equal(I, Iw)
        if not mask.any():
            assert not bool(Y.any()) and not bool(I.any())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_exact_ties_in_calls_of_few_tokens(dtype):
    """Each half of a sequence has lanes of its own: equal maxima across the halves and within either."""
    inp = wl.make_custom(3, 20, 64, 500, dtype=dtype, seed=14, len_lo=20)
    for arr in (inp.H,) if dtype == "f32" else (inp.H, inp.H_bits):
        arr[0, 17] = arr[0, 12] = arr[0, 2]      # first half, second half
        arr[1, 9] = arr[1, 0]                    # both in the first half
        arr[2, 19] = arr[2, 11]                  # both in the second half
    assert lsr.lsr_head_plan_ex(3, 20, 64, 500, lsr.LSR_F32 if dtype == "f32" else lsr.LSR_BF16)["fwd_few_tokens"] == 1
    head = DeviceHead(inp)
    head.forward()
    torch.cuda.synchronize()
    I = head.I.cpu().numpy()
    assert np.any(I[0] == 2) and np.any(I[1] == 0) and np.any(I[2] == 11)
    assert not np.any((I[0] == 17) | (I[0] == 12)) and not np.any(I[1] == 9) and not np.any(I[2] == 19)
    parity.compare_forward(inp, head.Y.cpu().numpy(), I)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
# 8-row segments, 32-row segments, several tiles; few tokens, whose sequences have lanes for each half
@pytest.mark.parametrize("B,S,D,V", [(5, 24, 64, 300), (3, 100, 72, 300), (2, 300, 64, 520), (4, 16, 64, 300), (1, 64, 72, 300)])
def test_nan_tokens_are_never_selected(B, S, D, V, dtype):
    """A token whose hidden state holds a NaN has NaN logits; the maximum and its position are those of the other tokens.
    The patterns leave one half-wave of a segment (rows 0..3 of every eight, or 4..7), whole segments, whole tiles or
    whole sequences without a number; a sequence of NaN tokens only gives Y = 0, I = 0."""
    inp = wl.make_custom(B, S, D, V, dtype=dtype, seed=S, len_lo=S, w_std=0.05)
    s = np.arange(S)
    for bad in (s % 8 < 4, s % 8 >= 4, s % 4 != 2, (s // 8) % 2 == 0, s < min(S - 1, 260), s >= 1, s >= 0):
        head = DeviceHead(inp)
        head.H[:, torch.from_numpy(np.nonzero(bad)[0]).cuda(), 3] = float("nan")
        head.poison_outputs()
        head.forward()
        torch.cuda.synchronize()
        Y, I = head.Y.cpu().numpy(), head.I.cpu().numpy()
        keep = np.broadcast_to(~bad, (B, S)).astype(np.uint8)
        parity.compare_forward(inp, Y, I, mask=keep)      # as if the NaN tokens were masked
        if bad.all():
            assert not Y.any() and not I.any()


def test_scattered_mask_and_empty_rows():
    inp = wl.make_custom(6, 150, 128, 600, seed=77)
    rng = np.random.default_rng(3)
    mask = wl.scattered_mask(rng, 6, 150, keep=0.4)
    mask[2, :] = 0
    mask[4, :] = 0
    mask[4, 149] = 1
    print(run_case(inp, mask=mask))
    inp2 = wl.make_custom(40, 30, 64, 300, seed=78)
    mask2 = wl.scattered_mask(rng, 40, 30, keep=0.3)
    mask2[0, :] = 0
    mask2[39, :] = 0
    print(run_case(inp2, mask=mask2))


def test_forced_exact_ties_pick_lowest_position():
    inp = wl.make_custom(2, 40, 64, 500, seed=9, len_lo=40)
    for arr in (inp.H, inp.H_bits):
        arr[0, 33] = arr[0, 2]
        arr[0, 17] = arr[0, 2]
        arr[1, 39] = arr[1, 0]
    head = DeviceHead(inp)
    head.forward()
    torch.cuda.synchronize()
    I = head.I.cpu().numpy()
    assert not np.any((I[0] == 33) | (I[0] == 17)) and not np.any(I[1] == 39)
    parity.compare_forward(inp, head.Y.cpu().numpy(), I)
    inp = wl.make_custom(1, 600, 64, 300, seed=10, len_lo=600)
    for arr in (inp.H, inp.H_bits):
        arr[0, 599] = arr[0, 100]          # twins in different chunks and different waves
        arr[0, 300] = arr[0, 100]
        arr[0, 200] = arr[0, 7]
    head = DeviceHead(inp)
    head.forward()
    torch.cuda.synchronize()
    I = head.I.cpu().numpy()
    assert not np.any((I == 599) | (I == 300) | (I == 200))
    parity.compare_forward(inp, head.Y.cpu().numpy(), I)


def test_forward_without_index_output():
    inp = wl.make_custom(3, 300, 128, 700, seed=12, len_lo=10)
    print(run_case(inp, want_index=False))
    inp = wl.make_custom(12, 32, 128, 700, seed=13)
    print(run_case(inp, want_index=False))


def test_backward_output_subsets():
    inp = wl.make_custom(4, 64, 128, 520, seed=21)
    head = DeviceHead(inp)
    head.forward()
    head.backward()
    torch.cuda.synchronize()
    ref = (head.dH.clone(), head.dW.clone(), head.db.clone())
    from paper_2603_25011_amd import binding as b
    shape = (head.B, head.S, head.D, head.V, head.dt)
    for keep in ((1, 0, 0), (0, 1, 0), (0, 0, 1), (0, 1, 1)):
        head.poison_outputs()
        head.forward()
        b.lsr_head_backward(*shape, head.H, head.W, head.dY, head.Y, head.I,
                            head.dH if keep[0] else None, head.dW if keep[1] else None,
                            head.db if keep[2] else None, head.ws_bwd)
        torch.cuda.synchronize()
        for k, out, r in zip(keep, (head.dH, head.dW, head.db), ref):
            if k:
                assert torch.equal(out, r)
            else:
                assert torch.isnan(out).all()


def test_c2_document_encoding_forward_full():
    inp = wl.make_inputs(wl.WORKLOADS["c2_doc_fwd"])
    print(run_case(inp, check_bwd=False))


def test_c3_query_encoding_forward_backward_full():
    inp = wl.make_inputs(wl.WORKLOADS["c3_query_fwdbwd"])
    print(run_case(inp))


def test_autograd_wrapper_matches_direct_calls():
    from paper_2603_25011_amd.autograd import lsr_head
    inp = wl.make_custom(5, 70, 128, 640, seed=41, len_lo=3)
    head = DeviceHead(inp)
    head.forward()
    head.backward()
    torch.cuda.synchronize()
    H = head.H.clone().requires_grad_(True)
    W = head.W.clone().requires_grad_(True)
    bias = head.bias.clone().requires_grad_(True)
    Y, I = lsr_head(H, W, bias, head.mask)
    assert torch.equal(Y, head.Y) and torch.equal(I, head.I)
    Y.backward(head.dY)
    torch.cuda.synchronize()
    # the wrapper's own outputs against the oracle; dH and dW arrive in the parameters' dtype (bf16), so
    # they are held to the oracle within one bf16 rounding step instead of the fp32 bound
    I_np = I.cpu().numpy()
    print(parity.compare_forward(inp, Y.detach().cpu().numpy(), I_np)[3])
    print(parity.compare_backward(inp, I_np, H.grad.float().cpu().numpy(), W.grad.float().cpu().numpy(),
                                  bias.grad.cpu().numpy(), bf16_grads=True))
    # same kernels, same order of the float32 sums; the library rounds to the parameter dtype as torch does
    assert torch.equal(H.grad, head.dH.to(torch.bfloat16))
    assert torch.equal(W.grad, head.dW.to(torch.bfloat16))
    assert torch.equal(bias.grad, head.db)
    # only the bias needs a gradient: the other outputs are skipped
    H2, W2, b2 = head.H.clone(), head.W.clone(), head.bias.clone().requires_grad_(True)
    Y2, _ = lsr_head(H2, W2, b2, head.mask)
    Y2.backward(head.dY)
    assert torch.equal(b2.grad, head.db)


def test_autograd_wrapper_masks_and_missing_gradients():
    """Masks of one byte per token go to the library as they are: any non-zero byte is a valid token, at any address and
    stride.  An output gradient that autograd leaves out counts as zero.  Calls go to the current stream."""
    from paper_2603_25011_amd.autograd import lsr_head
    inp = wl.make_custom(3, 37, 64, 300, seed=5, len_lo=4)
    head = DeviceHead(inp)
    H, W, bias = head.H, head.W, head.bias
    want = lsr_head(H, W, bias, head.mask)
    odd = torch.zeros((4, 37), dtype=torch.uint8, device="cuda")
    odd[1:] = head.mask * 255                                   # rows begin at odd addresses
    strided = torch.zeros((3, 74), dtype=torch.uint8, device="cuda")
    strided[:, ::2] = head.mask * 7
    for mask in (head.mask != 0, odd[1:], strided[:, ::2], head.mask.long() * 256, head.mask.float()):
        assert all(torch.equal(a, b) for a, b in zip(lsr_head(H, W, bias, mask), want))

    class Dropped(torch.autograd.Function):
        @staticmethod
        def forward(ctx, y):
            return y.clone()

        @staticmethod
        def backward(ctx, _grad):
            return None

    leaves = [t.clone().requires_grad_(True) for t in (H, W, bias)]
    Y, I = lsr_head(*leaves, head.mask)
    assert not I.requires_grad
    Dropped.apply(Y).sum().backward()
    for t in leaves:
        assert t.grad is None or (t.grad.dtype == t.dtype and not t.grad.any())

    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert lsr._stream(None) == side.cuda_stream
    assert lsr._stream(None) == torch.cuda.current_stream().cuda_stream


def test_random_shapes_and_masks():
    """Two dozen seeded random problems: odd sizes, D from the smallest legal value up, masks of any
    density with empty sequences mixed in, both loaders (D a multiple of 64 or not)."""
    rng = np.random.default_rng(20260325)
    for case in range(24):
        B = int(rng.integers(1, 41))
        S = int(rng.integers(1, 301))
        D = int(rng.choice([8, 16, 24, 64, 72, 128, 192, 200, 256]))
        V = int(rng.integers(1, 1501))
        keep = float(rng.choice([0.05, 0.3, 0.7, 1.0]))
        inp = wl.make_custom(B, S, D, V, seed=5000 + case)
        mask = wl.scattered_mask(rng, B, S, keep=keep)
        if B > 2 and case % 3 == 0:
            mask[int(rng.integers(0, B)), :] = 0
        print(f"case {case}: B={B} S={S} D={D} V={V} keep={keep}", flush=True)
        run_case(inp, mask=mask)


def test_random_shapes_batched_long_and_wide():
    """A dozen seeded problems from the corners the first set does not reach: batches of several
    hundred short sequences (16-row dW tiles, compacted), sequences beyond 1024 positions (direct
    bucket placement, eight buckets per wave), vocabularies of tens of thousands (chunked dH)."""
    rng = np.random.default_rng(20260326)
    for case in range(12):
        kind = case % 3
        if kind == 0:
            B, S, V = int(rng.integers(150, 420)), int(rng.integers(1, 40)), int(rng.integers(1, 2500))
        elif kind == 1:
            B, S, V = int(rng.integers(1, 6)), int(rng.integers(300, 1300)), int(rng.integers(1, 1200))
        else:
            B, S, V = int(rng.integers(1, 5)), int(rng.integers(1, 60)), int(rng.integers(33000, 90000))
        D = int(rng.choice([64, 128])) if kind == 2 else int(rng.choice([8, 24, 64, 128, 192, 200, 256, 320]))
        keep = float(rng.choice([0.02, 0.3, 0.7, 1.0]))
        inp = wl.make_custom(B, S, D, V, seed=7000 + case)
        mask = wl.scattered_mask(rng, B, S, keep=keep)
        print(f"case {case}: B={B} S={S} D={D} V={V} keep={keep}", flush=True)
        run_case(inp, mask=mask)


@pytest.mark.parametrize("B,S,D,V", [
    (5, 70, 128, 900),          # sliced gathers
    (3, 200, 128, 131100),      # LDS-tile dW kernel: the tile copy brings masked rows into LDS
    (4, 50, 728, 300),          # whole-row kernels; rows that end inside a slab
    (4, 50, 72, 300),           # the same in slices, the last one partly filled
])
def test_masked_positions_may_hold_anything(B, S, D, V):
    """Hidden states at masked positions are never multiplied, in the forward or in the backward: with
    NaN and infinities written there every output is bit-identical to the run on the clean input."""
    inp = wl.make_custom(B, S, D, V, seed=77 + B, len_lo=3)
    rng = np.random.default_rng(B)
    mask = wl.scattered_mask(rng, B, S, keep=0.6)
    clean = DeviceHead(inp, mask=mask)
    clean.poison_outputs()
    clean.forward()
    clean.backward()
    torch.cuda.synchronize()
    ref = [t.clone() for t in (clean.Y, clean.I, clean.dH, clean.dW, clean.db)]
    dirty = DeviceHead(inp, mask=mask)
    junk = torch.tensor([float("nan"), float("inf"), -float("inf")], device=dirty.dev)
    pick = torch.randint(0, 3, (B, S, D), device=dirty.dev, generator=torch.Generator(device=dirty.dev).manual_seed(3))
    masked = (dirty.mask == 0).view(B, S, 1).expand(B, S, D)
    dirty.H = torch.where(masked, junk[pick].to(dirty.H.dtype), dirty.H).contiguous()
    dirty.poison_outputs()
    dirty.forward()
    dirty.backward()
    torch.cuda.synchronize()
    for name, got, want in zip(("Y", "I", "dH", "dW", "db"), (dirty.Y, dirty.I, dirty.dH, dirty.dW, dirty.db), ref):
        assert torch.equal(got, want), name
    parity.compare_forward(inp, dirty.Y.cpu().numpy(), dirty.I.cpu().numpy(), mask=mask)


def test_random_shapes_lds_tile_dw():
    """Seeded problems in the range of the LDS-tile dW kernel (128 <= S <= 512, at least 256 workgroups of 1024
    vocabulary rows x 64 columns): few sequences against vocabularies wide enough for that, scattered masks
    with empty sequences, gradients from dense to 2 % non-zero (pairs without gradient read the tile's row
    of zeros; all-zero groups are skipped), D from one column slice to sixteen."""
    from paper_2603_25011_amd import binding as b
    rng = np.random.default_rng(20260327)
    for case in range(8):
        D = int(rng.choice([64, 128, 192, 256, 512, 1024]))
        B = int(rng.integers(1, 5))
        S = int(rng.integers(128, 513)) if case else 512
        V = (256 * 1024 * 64) // D - int(rng.integers(0, 1024)) + (1024 if case % 2 else 3000)
        V = max(V, (255 * 1024 * 64) // D + 1025)             # at least 256 vocabulary tiles x slices
        plan = b.lsr_head_plan(B, S, D, V, b.LSR_BF16)
        assert plan["dw_lds_tile_passes"] == (S + 127) // 128, plan
        keep = float(rng.choice([0.3, 0.7, 1.0]))
        density = float(rng.choice([0.02, 0.3, 1.0]))
        inp = wl.make_custom(B, S, D, V, seed=9000 + case)
        inp.dY[...] = inp.dY * (rng.random(inp.dY.shape) < density)
        mask = wl.scattered_mask(rng, B, S, keep=keep)
        if B > 2 and case % 3 == 0:
            mask[int(rng.integers(0, B)), :] = 0
        print(f"case {case}: B={B} S={S} D={D} V={V} keep={keep} gradient density={density}", flush=True)
        run_case(inp, mask=mask)


@pytest.mark.parametrize("B,S,D,V,len_lo,density", [
    (3, 200, 128, 131100, 1, 1.0),       # two copy passes; lengths from one token to the whole row
    (4, 512, 64, 262200, 100, 0.05),     # four passes, one slice
    (5, 129, 128, 131072, 127, 0.0005),  # one row behind a pass, most pairs without a gradient
    (2, 128, 192, 100000, 1, 1.0),       # one pass
])
def test_lds_tile_dw_copies_the_positions_in_use(B, S, D, V, len_lo, density):
    """Behind dH the LDS-tile dW kernel copies the rows up to each sequence's last one with a gradient; beside dH (the plain
    call, from 0.1 GB of gathers on) and without dH it copies all.  The profiled call runs everything on one stream.  Same bits each time;
    one sequence has no valid token, and hidden states behind the others' lengths are NaN."""
    from paper_2603_25011_amd import binding as b
    plan = b.lsr_head_plan(B, S, D, V, b.LSR_BF16)
    assert plan["dw_lds_tile_passes"] == (S + 127) // 128 and plan["dh_chunks"] > 1 and plan["dw_beside_dh"] == 1, plan
    inp = wl.make_custom(B, S, D, V, seed=77 + S, len_lo=len_lo)
    inp.dY[...] = inp.dY * (np.random.default_rng(S).random(inp.dY.shape) < density)
    head = DeviceHead(inp)
    mask = head.mask.clone()
    mask[B // 2] = 0
    head.mask.copy_(mask)
    head.H[mask == 0] = float("nan")
    head.forward()
    head.backward()
    torch.cuda.synchronize()
    ref = [t.clone() for t in (head.dH, head.dW, head.db)]
    assert all(torch.isfinite(t).all() for t in ref)
    for call in (lambda: b.lsr_head_backward_profiled(*head._shape(), head.H, head.W, head.dY, head.Y, head.I, head.dH, head.dW, head.db, head.ws_bwd),
                 lambda: b.lsr_head_backward(*head._shape(), head.H, head.W, head.dY, head.Y, head.I, None, head.dW, head.db, head.ws_bwd)):
        for t in (head.dW, head.db):
            t.fill_(float("nan"))
        call()
        torch.cuda.synchronize()
        for got, want in zip((head.dH, head.dW, head.db), ref):
            assert torch.equal(got, want)


@pytest.mark.parametrize("B,S,D,V,len_lo", [
    (5, 70, 128, 640, 3),          # one launch each
    (2, 16, 128, 70000, 1),        # dH over three vocabulary chunks: float32 partial sums staged in the workspace
    (260, 256, 64, 4100, 60),      # dW over three launches of sequences: staged likewise
    (3, 40, 200, 900, 1),          # D not a multiple of 64: whole-row kernels
    (450, 12, 64, 700, 1),         # whole-row dW beside sliced dH
    (3, 200, 128, 131100, 20),     # LDS-tile dW kernel (dW requested) and the sliced gather (db alone)
])
def test_bf16_gradient_outputs_and_accumulation(B, S, D, V, len_lo):
    """lsr_head_backward_ex: bfloat16 dH / dW (compared with the oracle within one bf16 step), and
    accumulation into the caller's buffers for float32 and bfloat16 outputs."""
    from oracle import lsr_head_oracle as orc
    inp = wl.make_custom(B, S, D, V, seed=900 + B, len_lo=len_lo)
    head = DeviceHead(inp)
    head.forward()
    head.backward()
    torch.cuda.synchronize()
    shape = (head.B, head.S, head.D, head.V, head.dt)
    dev = head.dev
    I = head.I.cpu().numpy()
    parity.compare_forward(inp, head.Y.cpu().numpy(), I)
    dH_ref, dW_ref, db_ref, _, _ = orc.backward(inp.H, inp.W, inp.bias, inp.mask, inp.dY, I_override=I)
    f32 = (head.dH.clone(), head.dW.clone(), head.db.clone())

    def run(grad_dtype, accumulate, dH, dW, db):
        ws = torch.empty(lsr.lsr_head_backward_ex_workspace_bytes(*shape, grad_dtype, accumulate), dtype=torch.uint8, device=dev)
        lsr.lsr_head_backward_ex(*shape, head.H, head.W, head.dY, head.Y, head.I, dH, dW, db, grad_dtype, accumulate, ws)
        torch.cuda.synchronize()

    # float32, overwrite: the same launches as lsr_head_backward
    out = [torch.full_like(t, float("nan")) for t in f32]
    run(lsr.LSR_F32, False, *out)
    for a, b_ in zip(out, f32):
        assert torch.equal(a, b_)
    # bfloat16, overwrite
    dH16 = torch.full((B, S, D), float("nan"), dtype=torch.bfloat16, device=dev)
    dW16 = torch.full((V, D), float("nan"), dtype=torch.bfloat16, device=dev)
    db32 = torch.full((V,), float("nan"), device=dev)
    run(lsr.LSR_BF16, False, dH16, dW16, db32)
    parity.check_close_bf16("dH bf16", dH16.float().cpu().numpy(), dH_ref)
    parity.check_close_bf16("dW bf16", dW16.float().cpu().numpy(), dW_ref)
    assert torch.equal(db32, f32[2])
    # one rounding of the float32 result, exactly
    assert torch.equal(dH16, f32[0].to(torch.bfloat16)) and torch.equal(dW16, f32[1].to(torch.bfloat16))
    # float32, accumulate into buffers that already hold something
    g = torch.Generator(device=dev)
    g.manual_seed(5)
    base = [torch.randn(t.shape, device=dev, generator=g) for t in f32]
    out = [t.clone() for t in base]
    run(lsr.LSR_F32, True, *out)
    for name, a, b0, ref in zip(("dH", "dW", "db"), out, base, (dH_ref, dW_ref, db_ref)):
        parity.check_close(name + " accumulated", a.cpu().numpy(), b0.cpu().numpy().astype(np.float64) + ref)
    # bfloat16, accumulate
    b16 = [base[0].to(torch.bfloat16), base[1].to(torch.bfloat16)]
    dH16, dW16, db32 = b16[0].clone(), b16[1].clone(), base[2].clone()
    run(lsr.LSR_BF16, True, dH16, dW16, db32)
    parity.check_close_bf16("dH bf16 accumulated", dH16.float().cpu().numpy(), b16[0].float().cpu().numpy().astype(np.float64) + dH_ref)
    parity.check_close_bf16("dW bf16 accumulated", dW16.float().cpu().numpy(), b16[1].float().cpu().numpy().astype(np.float64) + dW_ref)
    parity.check_close("db accumulated", db32.cpu().numpy(), base[2].cpu().numpy().astype(np.float64) + db_ref)
    # subsets of outputs
    dW16b = torch.full((V, D), float("nan"), dtype=torch.bfloat16, device=dev)
    run(lsr.LSR_BF16, False, None, dW16b, None)
    assert torch.equal(dW16b, f32[1].to(torch.bfloat16))
    db_only = torch.full((V,), float("nan"), device=dev)
    run(lsr.LSR_F32, False, None, None, db_only)
    assert torch.equal(db_only, f32[2])


@pytest.mark.parametrize("grad_dtype,accumulate", [(lsr.LSR_F32, False), (lsr.LSR_F32, True), (lsr.LSR_BF16, False), (lsr.LSR_BF16, True)])
@pytest.mark.parametrize("B,S,D,V,dtype", [
    (2, 9, 8, 300, "bf16"),        # one slice with a single 16-byte chunk
    (3, 70, 72, 500, "bf16"),      # the last slice holds one chunk
    (5, 40, 568, 700, "bf16"),     # nine slices, the last one short of one chunk; slices owned by XCDs
    (20, 30, 120, 900, "bf16"),    # slices in grid order
    (200, 20, 104, 300, "bf16"),   # 16-row dW tiles
    (400, 6, 104, 200, "bf16"),    # more sequences than the staging tile takes: whole-row dW
    (3, 140, 712, 17000, "bf16"),  # the filled-up problem takes the LDS-tile dW kernel
    (3, 20, 72, 70000, "bf16"),    # several vocabulary chunks
    (30, 64, 200, 70000, "bf16"),  # ... of half the rows (more than the filled-up problem has)
    (4, 20, 40, 600, "f32"),
    (90, 12, 200, 400, "f32"),
    (6, 24, 104, 40000, "f32"),    # several vocabulary chunks
    (4, 60, 728, 500, "bf16"),     # whole rows, 91 of 128 threads
    (3, 12, 1032, 3000, "bf16"),   # whole rows, two chunks per thread
    (70, 80, 200, 2100, "bf16"),   # whole rows for their length
    (3, 66, 40, 700, "f32"),
])
def test_hidden_sizes_that_are_no_multiple_of_64(B, S, D, V, dtype, grad_dtype, accumulate):
    """dH and dW against float64 sums: a sum of n terms in any order is within (n + 16) 2^-24 of the sum of their magnitudes
    (16: the joins of lanes, waves and chunks, and what it is accumulated onto), and a bfloat16 result within half a step of
    its size more.  Nothing behind a row is touched.  Where a problem takes slices, dW and db are, bit for bit, those of the
    same problem with D filled up with zeros to the next multiple of 64 (every sum has the same terms in the same
    order), and so is dH where both are cut into the same vocabulary chunks."""
    if dtype == "f32" and grad_dtype == lsr.LSR_BF16:
        pytest.skip("bfloat16 gradients belong to bfloat16 parameters")
    dt = lsr.LSR_F32 if dtype == "f32" else lsr.LSR_BF16
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gd = torch.bfloat16 if grad_dtype == lsr.LSR_BF16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(B * 1000 + D)
    Dp = (D + 63) // 64 * 64
    H = torch.randn((B, S, D), device="cuda", generator=g).to(td)
    W = torch.randn((V, D), device="cuda", generator=g).mul_(0.05).to(td)
    Y = torch.full((B, V), 1e-30, device="cuda")              # exp(-Y) = 1: the gradient of a pair is dY
    I = torch.randint(0, S, (B, V), device="cuda", generator=g, dtype=torch.int32)
    dY = torch.randn((B, V), device="cuda", generator=g) * (torch.rand((B, V), device="cuda", generator=g) < 0.7)
    dH0 = torch.randn((B, S, D), device="cuda", generator=g).to(gd)
    dW0 = torch.randn((V, D), device="cuda", generator=g).to(gd)
    db0 = torch.randn((V,), device="cuda", generator=g)
    wide = lambda t: torch.nn.functional.pad(t, (0, Dp - D)).contiguous()      # noqa: E731
    got = []
    for d, fill in ((D, lambda t: t.clone()), (Dp, wide)):
        guard = torch.full((4096,), 7.0, dtype=gd, device="cuda")
        bufs = [torch.cat([fill(t).flatten(), guard]) for t in (dH0, dW0)]
        db = db0.clone()
        ws = torch.empty(lsr.lsr_head_backward_ex_workspace_bytes(B, S, d, V, dt, grad_dtype, accumulate), dtype=torch.uint8, device="cuda")
        lsr.lsr_head_backward_ex(B, S, d, V, dt, fill(H), fill(W), dY, Y, I, bufs[0], bufs[1], db, grad_dtype, accumulate, ws)
        torch.cuda.synchronize()
        for b in bufs:
            assert torch.equal(b[-4096:], guard)
        got.append((bufs[0][:-4096].view(B, S, d), bufs[1][:-4096].view(V, d), db))

    dH, size_H = dh_in_float64(B, S, V, dY, I, W)
    dW, size_W = (torch.zeros((V, D), dtype=torch.float64, device="cuda") for _ in range(2))
    n_H = torch.zeros((B, S), device="cuda", dtype=torch.float64)
    n_H.scatter_add_(1, I.long(), (dY != 0).double())
    for b in range(B):
        t = dY[b].double()[:, None] * H[b].double()[I[b].long()]
        dW += t
        size_W += t.abs()
    n_W = (dY != 0).sum(dim=0).double()
    half_step = 2.0 ** -8 if gd == torch.bfloat16 else 0.0      # eight significant bits: steps of 2^-7 between 1 and 2
    for mine, want, size, n, old in ((got[0][0], dH, size_H, n_H[:, :, None], dH0), (got[0][1], dW, size_W, n_W[:, None], dW0)):
        if accumulate:
            want, size = want + old.double(), size + old.double().abs()
        bound = (n + 16) * 2.0 ** -24 * size
        assert bool(((mine.double() - want).abs() <= bound + half_step * (want.abs() + bound)).all())

    plan, plan_p = (lsr.lsr_head_plan(B, S, d, V, dt) for d in (D, Dp))
    if plan["dh_buckets_per_wave"] > 0:
        same_cut = all(plan[k] == plan_p[k] for k in ("dh_chunks", "dh_chunk_len", "dh_buckets_per_wave", "dh_waves_per_bucket"))
        for k, (a, p) in enumerate(zip(got[0][:2], got[1][:2])):
            if k == 1 or same_cut:
                assert torch.equal(a, p[..., :D])
        if plan["dw_sequences_per_launch"] >= B:
            assert torch.equal(got[0][2], got[1][2])


@pytest.mark.parametrize("B,S,D,V,dtype", [
    (6, 40, 64, 500, "bf16"), (6, 40, 72, 500, "bf16"), (6, 40, 728, 500, "bf16"), (6, 70, 72, 500, "f32"), (450, 5, 64, 300, "bf16")])
def test_rows_without_a_gradient_may_hold_nan(B, S, D, V, dtype):
    """Rows of H and W that no gradient points at stay out of every sum (also the first rows, which a gather could
    take to fill up a round): slices, whole rows, and whole-row dW beside sliced dH."""
    dt = lsr.LSR_F32 if dtype == "f32" else lsr.LSR_BF16
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(D)
    H = torch.randn((B, S, D), device="cuda", generator=g).to(td)
    W = torch.randn((V, D), device="cuda", generator=g).to(td)
    Y = torch.rand((B, V), device="cuda", generator=g)
    I = torch.randint(1, S, (B, V), device="cuda", generator=g, dtype=torch.int32)
    dY = torch.randn((B, V), device="cuda", generator=g)
    bad = [0, 7, V - 1]
    dY[:, bad] = 0.0
    H[:, 0] = float("nan")
    W[bad] = float("inf")
    dH, dW, db = torch.empty((B, S, D), device="cuda"), torch.empty((V, D), device="cuda"), torch.empty((V,), device="cuda")
    ws = torch.empty(lsr.lsr_head_workspace_bytes(B, S, D, V, dt, True), dtype=torch.uint8, device="cuda")
    lsr.lsr_head_backward(B, S, D, V, dt, H, W, dY, Y, I, dH, dW, db, ws)
    assert bool(dH.isfinite().all()) and bool(dW.isfinite().all()) and bool(db.isfinite().all())
    assert not dH[:, 0].any() and not dW[bad].any() and not db[bad].any()


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("B,S,D,V,dtype", [
    (13, 40, 72, 300, "bf16"),        # 64-row staging tiles
    (160, 20, 72, 300, "f32"),        # 32-row tiles
    (256, 20, 200, 300, "bf16"),      # 16-row tiles
    (300, 512, 64, 9000, "bf16"),     # several launches, each of which rounds the db it hands on; S above 128 but too few tiles
    (256, 130, 1024, 16400, "bf16"),  # LDS-tile kernel
    (90, 600, 1024, 10000, "f32"),
    (256, 130, 1032, 900, "bf16"),    # whole rows, one launch
    (400, 70, 72, 500, "f32"),
    (500, 9, 128, 333, "bf16"),
])
def test_db_is_rounded_once_per_launch(B, S, D, V, dtype, accumulate):
    """db = sum of dY where Y is tiny (exp(-Y) = 1): every launch rounds its running sum once, to within 2^-24 of its size;
    the float64 sums behind it are off by less (B 2^-47 of the sum of magnitudes).  The whole-row kernel adds every
    64th sequence in a lane and joins the lanes in six steps, each rounded to 2^-24 of a sum that the magnitudes bound.  With
    one gradient in ten too, which the sliced kernel compacts; infinities come out as in a plain sum."""
    dt = lsr.LSR_F32 if dtype == "f32" else lsr.LSR_BF16
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(B + V)
    H = torch.zeros((B, S, D), device="cuda", dtype=td)
    W = torch.zeros((V, D), device="cuda", dtype=td)
    Y = torch.full((B, V), 1e-30, device="cuda")
    I = torch.zeros((B, V), device="cuda", dtype=torch.int32)
    plan = lsr.lsr_head_plan(B, S, D, V, dt)
    sliced = plan["dw_sequences_per_launch"] if plan["dw_tile_rows"] > 0 else B
    per_launch = {True: B if plan["dw_lds_tile_passes"] else sliced, False: sliced}
    db0 = torch.randn((V,), device="cuda", generator=g)
    ws = torch.empty(lsr.lsr_head_backward_ex_workspace_bytes(B, S, D, V, dt), dtype=torch.uint8, device="cuda")
    dW = torch.zeros((V, D), device="cuda")
    for keep in (1.0, 0.1):
        dY = torch.randn((B, V), device="cuda", generator=g) * (torch.rand((B, V), device="cuda", generator=g) < keep)
        start = db0.double() if accumulate else torch.zeros(V, device="cuda", dtype=torch.float64)
        run = torch.cat([start[None], dY.double()]).cumsum(dim=0)
        for want_dw in (True, False):
            per = per_launch[want_dw]
            ends = run[[min(b + per, B) for b in range(0, B, per)]]      # the running sum after each launch
            size = start.abs() + dY.double().abs().sum(dim=0)
            bound = 2.0 ** -24 * ends.abs().sum(dim=0) + B * 2.0 ** -47 * size
            if plan["dw_tile_rows"] == 0:
                bound = ((B + 63) // 64 + 7) * 2.0 ** -24 * size
            db = db0.clone()
            lsr.lsr_head_backward_ex(B, S, D, V, dt, H, W, dY, Y, I, None, dW if want_dw else None, db, lsr.LSR_F32, accumulate, ws)
            assert bool(((db.double() - run[-1]).abs() <= bound).all())
    dY[B // 2, 5] = float("inf")
    dY[B - 1, 6] = float("-inf")
    dY[0, 7], dY[B - 1, 7] = float("inf"), float("-inf")
    db = db0.clone()
    lsr.lsr_head_backward_ex(B, S, D, V, dt, H, W, dY, Y, I, None, None, db, lsr.LSR_F32, accumulate, ws)
    assert db[5] == float("inf") and db[6] == float("-inf") and bool(db[7].isnan()) and bool(db[8:].isfinite().all())
    lsr.lsr_head_backward_ex(B, S, D, V, dt, H, W, dY, Y, I, None, dW, db, lsr.LSR_F32, False, ws)
    assert db[5] == float("inf") and db[6] == float("-inf") and bool(db[7].isnan()) and bool(db[8:].isfinite().all())


def test_two_host_threads_on_two_streams():
    """Two host threads call forward + backward concurrently, each on its own stream, buffers and small
    problem (too small for the library's shared auxiliary stream: the next test's are not).  Every call
    of both threads must match the oracle."""
    import threading
    inps = [wl.make_custom(6, 70, 128, 900, seed=101, len_lo=3), wl.make_custom(9, 33, 64, 1500, seed=102, len_lo=1)]
    errors = []
    results = [[], []]

    def worker(k):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                head = DeviceHead(inps[k])
                for it in range(20):
                    head.poison_outputs()
                    head.forward()
                    head.backward()
                    stream.synchronize()
                    results[k].append(tuple(t.cpu().numpy().copy() for t in (head.Y, head.I, head.dH, head.dW, head.db)))
        except Exception as exc:          # surfaced in the main thread
            errors.append((k, repr(exc)))

    threads = [threading.Thread(target=worker, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k, inp in enumerate(inps):
        assert len(results[k]) == 20
        Y, I, dH, dW, db = results[k][0]
        parity.compare_forward(inp, Y, I)
        parity.compare_backward(inp, I, dH, dW, db)
        for other in results[k][1:]:      # deterministic kernels: every later call is bit-identical to the checked one
            for a, b_ in zip(results[k][0], other):
                assert np.array_equal(a, b_)


def test_two_host_threads_whose_backwards_fork():
    """Problems whose dW gather goes to the library's shared auxiliary stream: calls of two threads on two streams give, bit for
    bit, what each gives alone."""
    import threading
    shapes = ((65, 40, 256, 5000), (200, 20, 64, 2100))
    assert all(lsr.lsr_head_dw_route(*s, lsr.LSR_BF16) == lsr.LSR_DW_ON_AUX_STREAM for s in shapes)
    inps = [wl.make_custom(*s, seed=111 + k, len_lo=3 - 2 * k) for k, s in enumerate(shapes)]
    outs = lambda h: [t.clone() for t in (h.Y, h.I, h.dH, h.dW, h.db)]      # noqa: E731
    heads = [DeviceHead(i) for i in inps]
    alone = []
    for h, inp in zip(heads, inps):
        h.forward()
        h.backward()
        torch.cuda.synchronize()
        alone.append(outs(h))
    torch.cuda.synchronize()
    errors = []

    def worker(k):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for _ in range(20):
                    heads[k].poison_outputs()
                    heads[k].forward()
                    heads[k].backward()
                    stream.synchronize()
                    assert all(torch.equal(a, b) for a, b in zip(outs(heads[k]), alone[k]))
        except BaseException as exc:      # surfaced in the main thread
            errors.append((k, repr(exc)))

    threads = [threading.Thread(target=worker, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_mfma_probe_reports_a_plausible_rate():
    from paper_2603_25011_amd import binding as b
    sink = torch.zeros(1, dtype=torch.float32, device="cuda:0")
    tf = b.lsr_mfma_peak_probe(20000, 2, sink)
    print(f"register-only bf16 MFMA rate: {tf:.0f} TFLOP/s")
    assert 800.0 < tf < 2600.0          # between a third of and just above the nominal 2.5 PFLOP/s
    assert float(sink.item()) == 0.0    # nothing is ever stored


@pytest.mark.parametrize("B,S,D,V,dy_keep", [
    (2, 3, 64, 63, None),          # one step of one wave; the other waves of the placement have nothing
    (3, 257, 64, 4097, None),      # the prefix over the buckets takes two rounds of 256 threads, or one of 1024
    (2, 1024, 64, 9000, 0.3),      # the longest sequences that place through LDS, short last piece
    (2, 1025, 64, 9001, None),     # the first that do not
    (1, 8192, 64, 25000, 0.9),     # the longest of all: four tables of 8192 buckets
    (2, 40, 64, 16384 + 1, None),  # a last segment of few entries
    (1024, 8, 64, 4340, None),     # segments of 17 steps: pieces of five steps and one of two
    (600, 24, 64, 12600, 0.3),     # segments of 33 steps: three pieces of nine, one of six; sparse
])
def test_bucket_sort_pieces(B, S, D, V, dy_keep):
    """Sizes at which the pieces that the waves of the bucket sort take, and its prefix sums, end."""
    print(run_case(wl.make_custom(B, S, D, V, seed=B * 7 + S, len_lo=max(1, S // 2), dy_keep=dy_keep)))


@pytest.mark.parametrize("B,S", [(64, 256), (1, 16384), (31, 513), (17, 512), (64, 2), (128, 64), (65, 33), (129, 5)])
def test_packing_in_one_launch(B, S):
    """The most sequences and mask entries that one workgroup packs, and lengths around its eight entries per lane;
    a scattered mask with an empty first and last sequence."""
    inp = wl.make_custom(B, S, 64, 300 if B * S > 128 else 33000, seed=B + S, backward=False)
    mask = wl.scattered_mask(np.random.default_rng(S), B, S)
    if B > 1:
        mask[0, :] = 0
        mask[B - 1, :] = 0
    for m in (None, mask):
        print(run_case(inp, mask=m, check_bwd=False))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,S,D,V,dy_keep", [
    (1, 1, 64, 1, None), (3, 5, 72, 63, None), (2, 16, 64, 1024, None), (5, 300, 64, 1025, 0.3),      # four and eight steps per wave
    (2, 1024, 8, 2048, None), (3, 40, 128, 2049, None), (4, 700, 64, 4096, 0.05),                      # sixteen
    (96, 7, 64, 640, None), (97, 7, 64, 640, None),                                                    # dW tiles of 64 rows, and of 32
    (3, 40, 64, 4097, None), (2, 1025, 64, 1500, None),                                                # beyond: three launches
])
def test_small_problems_sort_and_dw_in_one_launch(B, S, D, V, dy_keep, dtype):
    """Against the oracle, and bit for bit against the profiled call, which runs the sort and dW apart."""
    inp = wl.make_custom(B, S, D, V, dtype=dtype, seed=3 * B + S + V, len_lo=1, dy_keep=dy_keep)
    run_case(inp)
    assert (lsr.lsr_head_plan(B, S, D, V, lsr.LSR_BF16)["sort_segments"] == 1) == (V <= 4096 and S <= 1024 or V < 2 * max(S, 512))
    head = DeviceHead(inp)
    head.forward()
    head.poison_outputs()
    head.forward()
    head.backward()
    torch.cuda.synchronize()
    ref = [t.clone() for t in (head.dH, head.dW, head.db)]
    head.dH.fill_(float("nan")), head.dW.fill_(float("nan")), head.db.fill_(float("nan"))
    head.backward_profiled()
    torch.cuda.synchronize()
    for got, want in zip((head.dH, head.dW, head.db), ref):
        assert torch.equal(got, want)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,S", [(5, 40), (2, 150)])         # 8-row and 32-row segments
@pytest.mark.parametrize("D", [8, 24, 56, 72, 88, 120, 136, 200])
def test_rows_that_end_inside_a_slab(B, S, D, dtype):
    """A slab is 64 bfloat16 or 32 float32 columns; its chunks behind the end of a row are zeros, whatever follows the row in
    memory: the hidden states behind each valid one are NaN (masked), and every second row of W is infinite."""
    V = 300
    inp = wl.make_custom(B, S, D, V, dtype=dtype, seed=D + S)
    mask = np.zeros((B, S), dtype=np.uint8)
    mask[:, ::2] = 1
    run_case(inp, mask=mask, check_bwd=False)
    head = DeviceHead(inp, mask=mask)
    head.forward()
    torch.cuda.synchronize()
    ref = head.Y.clone(), head.I.clone()
    head.H[head.mask == 0] = float("nan")
    head.W[::2] = float("inf")
    for index in (head.I, None):
        head.Y.fill_(float("nan"))
        lsr.lsr_head_forward(*head._shape(), head.H, head.W, head.bias, head.mask, head.Y, index, head.ws_fwd)
        torch.cuda.synchronize()
        assert torch.equal(head.Y[:, 1::2], ref[0][:, 1::2]) and torch.equal(head.I[:, 1::2], ref[1][:, 1::2])


PLACE, IN_DH = lsr.LSR_DW_IN_PLACEMENT_LAUNCH, lsr.LSR_DW_IN_DH_LAUNCH


@pytest.mark.parametrize("B,S,D,V,dtype,dy_keep,routes,bpw,wpb", [
    (4, 30, 128, 60000, "bf16", None, (IN_DH, PLACE), 1, 4),       # slices owned by XCDs; two windows: float32 gradients in the launch of dH
    (13, 64, 312, 9000, "bf16", 0.05, (IN_DH, IN_DH), 1, 1),       # partly filled last slice
    (20, 40, 256, 6000, "bf16", None, (IN_DH, IN_DH), 1, 4),       # slices in grid order, buckets shared by four waves
    (40, 48, 512, 4500, "bf16", None, (IN_DH, IN_DH), 1, 1),       # the largest dW tile
    (40, 8, 256, 10000, "bf16", 0.3, (IN_DH, IN_DH), 1, 4),        # the same beside the sums of four waves
    (30, 100, 128, 9000, "f32", 0.3, (IN_DH,), 1, 4),
    (2, 20, 512, 34000, "f32", None, (IN_DH,), 1, 4),              # windows in float32
    (12, 300, 64, 33000, "bf16", None, (IN_DH, PLACE), 2, 4),      # two windows, four waves per bucket
    (22, 230, 128, 12400, "bf16", 0.05, (IN_DH, IN_DH), 2, 1),     # two buckets per wave
    (12, 120, 256, 9000, "f32", None, (IN_DH,), 2, 1),
    (13, 300, 128, 5000, "bf16", None, (IN_DH, IN_DH), 4, 1),      # four
    (13, 300, 128, 5000, "f32", 0.3, (IN_DH,), 4, 1),
    (3, 700, 72, 5000, "bf16", None, (IN_DH, IN_DH), 8, 1),        # eight, and a partly filled last slice
    (70, 9, 64, 5000, "f32", 0.05, (PLACE,), 1, 4),                # too large a dW tile for the launch of dH
])
def test_dw_in_the_launch_of_dh_or_of_the_placement(B, S, D, V, dtype, dy_keep, routes, bpw, wpb):
    """Against the oracle, and bit for bit against the profiled call, which launches dW apart; overwriting and accumulating,
    in float32 and, for bfloat16 parameters, in bfloat16 (their routes, buckets per wave and waves per bucket are what the rows say)."""
    inp = wl.make_custom(B, S, D, V, dtype=dtype, seed=B + S + V, len_lo=1, dy_keep=dy_keep)
    dt = lsr.LSR_BF16 if dtype == "bf16" else lsr.LSR_F32
    plan = lsr.lsr_head_plan(B, S, D, V, dt)
    assert (plan["dh_buckets_per_wave"], plan["dh_waves_per_bucket"]) == (bpw, wpb)
    for grad_dtype, route in zip((lsr.LSR_F32, lsr.LSR_BF16), routes):
        assert lsr.lsr_head_dw_route(B, S, D, V, dt, grad_dtype) == route
    run_case(inp)
    head = DeviceHead(inp)
    head.forward()
    for t in (head.dH, head.dW, head.db):
        t.fill_(float("nan"))
    head.backward_profiled()
    torch.cuda.synchronize()
    ref = [t.clone() for t in (head.dH, head.dW, head.db)]
    head.backward()
    torch.cuda.synchronize()
    for got, want in zip((head.dH, head.dW, head.db), ref):
        assert torch.equal(got, want)
    for gt in ((lsr.LSR_F32, lsr.LSR_BF16) if dtype == "bf16" else (lsr.LSR_F32,)):
        td = torch.bfloat16 if gt == lsr.LSR_BF16 else torch.float32
        ws = torch.empty(lsr.lsr_head_backward_ex_workspace_bytes(B, S, D, V, dt, gt, True), dtype=torch.uint8, device="cuda")
        for accumulate in (False, True):
            dH, dW = (torch.ones_like(t, dtype=td) for t in (head.dH, head.dW))
            db = torch.ones_like(head.db)
            lsr.lsr_head_backward_ex(*head._shape(), head.H, head.W, head.dY, head.Y, head.I, dH, dW, db, gt, accumulate, ws)
            torch.cuda.synchronize()
            one = 1.0 if accumulate else 0.0
            for got, want in ((dH, ref[0]), (dW, ref[1])):
                # one rounding to the output type (a result that windows add up is rounded once per window in float32)
                scale = (want.abs() + one).double()
                tol = 2.0 ** -8 * scale if gt == lsr.LSR_BF16 else 2.0 ** -21 * scale
                assert bool(((got.double() - (want.double() + one)).abs() <= tol + 1e-6).all())
            assert torch.allclose(db, ref[2] + one, rtol=1e-6, atol=1e-6)


def test_two_host_threads_share_the_auxiliary_stream():
    """dW beside dH from LDS and from L2, in two threads on two streams: bit for bit what each call gives alone."""
    import threading
    heads = [DeviceHead(wl.make_custom(*shape, seed=113, len_lo=1)) for shape in ((3, 128, 128, 131100), (65, 40, 256, 14000))]
    alone, errors = [], []
    for h in heads:
        assert lsr.lsr_head_plan(*h._shape())["dw_beside_dh"] == 1
        h.forward()
        h.backward()
        torch.cuda.synchronize()
        alone.append([t.clone() for t in (h.dH, h.dW, h.db)])

    def worker(h, want):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for _ in range(20):
                    for t in (h.dH, h.dW, h.db):
                        t.fill_(float("nan"))
                    h.backward()
                    stream.synchronize()
                    assert all(torch.equal(a, b) for a, b in zip((h.dH, h.dW, h.db), want))
        except BaseException as exc:      # surfaced in the main thread
            errors.append(repr(exc))

    threads = [threading.Thread(target=worker, args=a) for a in zip(heads, alone)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


@pytest.mark.parametrize("B,S,D,V,dtype", [(19, 64, 896, 11500, "bf16"), (19, 64, 896, 5801, "f32")])
def test_buckets_of_two_waves_leave_dw_a_launch_of_its_own(B, S, D, V, dtype):
    """dW in workgroups of two waves would take up to 1.7 times as long, and sum db in another order: against the profiled call, which runs dW apart, where
    float64 terms of 2^60 cancel in one order of the sums and not in another."""
    dt = lsr.LSR_BF16 if dtype == "bf16" else lsr.LSR_F32
    assert lsr.lsr_head_plan(B, S, D, V, dt)["dh_waves_per_bucket"] == 2
    assert lsr.lsr_head_dw_route(B, S, D, V, dt) == lsr.LSR_DW_ON_AUX_STREAM
    head = DeviceHead(wl.make_custom(B, S, D, V, dtype=dtype, seed=5))
    head.forward()
    head.Y.fill_(1e-12)                     # exp(-Y) = 1
    head.dY[0], head.dY[2] = 2.0 ** 60, -2.0 ** 60
    head.dY[1].fill_(1.0)
    head.backward_profiled()
    torch.cuda.synchronize()
    apart = [t.clone() for t in (head.dH, head.dW, head.db)]
    for t in (head.dH, head.dW, head.db):
        t.fill_(float("nan"))
    head.backward()
    torch.cuda.synchronize()
    for got, want in zip((head.dH, head.dW, head.db), apart):
        assert torch.equal(got, want)


def test_sort_of_one_segment_beside_a_dw_of_many_sequences():
    """More than 384 sequences with dW on the auxiliary stream: one segment, counted, scanned and placed in three launches; the profiled
    call sorts in one."""
    B, S, D, V = 450, 12, 128, 700
    assert lsr.lsr_head_dw_route(B, S, D, V, lsr.LSR_BF16) == lsr.LSR_DW_ON_AUX_STREAM
    assert lsr.lsr_head_plan(B, S, D, V, lsr.LSR_BF16)["sort_segments"] == 1
    inp = wl.make_custom(B, S, D, V, seed=9, len_lo=1)
    run_case(inp)
    head = DeviceHead(inp)
    head.forward()
    head.backward()
    torch.cuda.synchronize()
    ref = [t.clone() for t in (head.dH, head.dW, head.db)]
    for t in (head.dH, head.dW, head.db):
        t.fill_(float("nan"))
    head.backward_profiled()
    torch.cuda.synchronize()
    for got, want in zip((head.dH, head.dW, head.db), ref):
        assert torch.equal(got, want)


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 72), ("f32", 32), ("f32", 40)])      # whole slabs, and a partly filled last one
@pytest.mark.parametrize("B,S", [(5, 70), (12, 60)])                                            # 32-row and 8-row segments
def test_forward_beyond_4_gib_of_w(B, S, dtype, D):
    """W of 4 GiB goes through the register-staged loader with 64-bit addresses.  Its rows repeat those of a small W, whose result
    (direct loads to LDS, held to the oracle) has to come back bit for bit in every period."""
    P = 8209                                # not a multiple of a tile
    inp = wl.make_custom(B, S, D, P, dtype=dtype, seed=D + S, len_lo=1)
    run_case(inp, check_bwd=False)
    head = DeviceHead(inp)
    head.forward()
    n = (1 << 32) // (P * D * head.W.element_size()) + 1
    W, bias = head.W.repeat(n, 1), head.bias.repeat(n)
    assert W.numel() * W.element_size() >= 1 << 32
    ws = torch.empty(lsr.lsr_head_workspace_bytes(B, S, D, n * P, head.dt, False), dtype=torch.uint8, device="cuda")
    Y = torch.full((B, n * P), float("nan"), device="cuda")
    I = torch.full((B, n * P), -7, dtype=torch.int32, device="cuda")
    for index in (I, None):
        Y.fill_(float("nan"))
        lsr.lsr_head_forward(B, S, D, n * P, head.dt, head.H, W, bias, head.mask, Y, index, ws)
        torch.cuda.synchronize()
        assert torch.equal(Y.view(B, n, P), head.Y[:, None].expand(B, n, P))
    assert torch.equal(I.view(B, n, P), head.I[:, None].expand(B, n, P))


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 72), ("f32", 40)])
def test_forward_beyond_4_gib_of_hidden_states(dtype, D):
    """The same for the hidden states: the sequences repeat those of a small batch."""
    S, V, P = 8000, 300, 3
    inp = wl.make_custom(P, S, D, V, dtype=dtype, seed=D, len_lo=S // 2)
    run_case(inp, check_bwd=False)
    head = DeviceHead(inp)
    head.forward()
    n = (1 << 32) // (head.H.numel() * head.H.element_size()) + 1
    H, mask = head.H.repeat(n, 1, 1), head.mask.repeat(n, 1)
    assert H.numel() * H.element_size() >= 1 << 32
    ws = torch.empty(lsr.lsr_head_workspace_bytes(n * P, S, D, V, head.dt, False), dtype=torch.uint8, device="cuda")
    Y = torch.full((n * P, V), float("nan"), device="cuda")
    I = torch.full((n * P, V), -7, dtype=torch.int32, device="cuda")
    lsr.lsr_head_forward(n * P, S, D, V, head.dt, H, head.W, head.bias, mask, Y, I, ws)
    torch.cuda.synchronize()
    assert torch.equal(Y.view(n, P, V), head.Y.expand(n, P, V)) and torch.equal(I.view(n, P, V), head.I.expand(n, P, V))
