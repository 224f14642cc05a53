"""The launch plan the host derives from a shape (lsr_head_plan): documented values for the benchmark
shapes and the invariants the kernels rely on, over a few thousand random shapes.  No GPU needed."""
import ctypes

import numpy as np
import pytest

import paper_2603_25011_amd as lsr
from paper_2603_25011_amd import binding


@pytest.fixture(scope="module", autouse=True)
def lib():
    import os
    if not os.path.exists(lsr.library_path()):
        from paper_2603_25011_amd import build
        build.build()
    return lsr.load_library()


def test_plans_of_the_benchmark_shapes():
    p = lsr.lsr_head_plan(64, 512, 1024, 250002, lsr.LSR_BF16)          # C5
    assert p == {"fwd_tiles_per_chunk": 4, "fwd_chunks": 32, "fwd_segment_rows": 32, "fwd_resident_workgroups": 0,
                 "sort_segments": 64, "sort_segment_len": 3968, "sort_places_through_lds": 1,
                 "dh_chunks": 8, "dh_chunk_len": 31251, "dh_buckets_per_wave": 2, "dw_tile_rows": 64,
                 "dw_sequences_per_launch": 64, "dh_slices_owned_by_xcd": 0, "dw_lds_tile_passes": 4,
                 "dh_waves_per_bucket": 1, "fwd_window_segments": 0, "dw_beside_dh": 0}
    p = lsr.lsr_head_plan(16, 256, 768, 250002, lsr.LSR_BF16)           # C4: longer buckets, one per wave
    assert (p["dh_chunks"], p["dh_buckets_per_wave"], p["dw_tile_rows"]) == (8, 1, 64)
    # a small batch: dH slices owned by XCDs; S = 256: the LDS-tile dW kernel with two copy passes per tile
    assert (p["dh_slices_owned_by_xcd"], p["dw_lds_tile_passes"]) == (1, 2)
    p = lsr.lsr_head_plan(256, 32, 768, 30522, lsr.LSR_BF16)            # C3: one pass over a 30k vocabulary, 16-row dW tiles
    assert (p["dh_chunks"], p["dh_buckets_per_wave"], p["dw_tile_rows"]) == (1, 1, 16)
    # short sequences: 8-row segments; a shallow grid: resident workgroups over one-tile units
    assert (p["fwd_tiles_per_chunk"], p["fwd_chunks"], p["fwd_segment_rows"], p["fwd_resident_workgroups"]) == (1, 32, 8, 1)
    assert (p["dh_slices_owned_by_xcd"], p["dw_lds_tile_passes"]) == (0, 0)      # S below the LDS-tile kernel's range
    p = lsr.lsr_head_plan(128, 8192, 768, 30522, lsr.LSR_BF16)          # long sequences: short buckets, direct placement
    assert (p["dh_buckets_per_wave"], p["sort_places_through_lds"], p["dh_chunks"]) == (8, 0, 1)
    assert p["dw_lds_tile_passes"] == 0                                 # a sequence's slice does not fit an LDS tile
    # the LDS-tile dW kernel needs a workgroup per CU: 1024 vocabulary rows x 64 columns each
    assert lsr.lsr_head_plan(32, 256, 128, 30522, lsr.LSR_BF16)["dw_lds_tile_passes"] == 0      # 30 x 2 workgroups
    assert lsr.lsr_head_plan(32, 256, 768, 30522, lsr.LSR_BF16)["dw_lds_tile_passes"] == 2      # 30 x 12
    assert lsr.lsr_head_plan(32, 256, 768, 30522, lsr.LSR_F32)["dw_lds_tile_passes"] == 0       # bfloat16 only
    assert lsr.lsr_head_plan(32, 513, 768, 30522, lsr.LSR_BF16)["dw_lds_tile_passes"] == 0
    assert lsr.lsr_head_plan(32, 127, 768, 30522, lsr.LSR_BF16)["dw_lds_tile_passes"] == 0
    assert lsr.lsr_head_plan(17, 128, 768, 30522, lsr.LSR_BF16)["dh_slices_owned_by_xcd"] == 0
    p = lsr.lsr_head_plan(256, 512, 768, 250002, lsr.LSR_BF16)          # a batch whose H slice is 4x L2: four dW launches
    assert (p["dw_sequences_per_launch"], p["dw_tile_rows"]) == (64, 64)
    # D not a multiple of 64: sliced kernels for short sequences and small problems ...
    p = lsr.lsr_head_plan(3, 40, 200, 900, lsr.LSR_BF16)
    assert (p["dh_buckets_per_wave"], p["dw_tile_rows"], p["dh_chunks"], p["fwd_resident_workgroups"]) == (4, 64, 1, 0)      # 32 entries per bucket: four buckets per wave
    p = lsr.lsr_head_plan(100, 40, 552, 150000, lsr.LSR_BF16)           # windows of half the rows: row pieces straddle cache lines
    assert (p["dh_chunks"], p["dh_chunk_len"], p["dw_tile_rows"], p["dw_lds_tile_passes"], p["dw_beside_dh"]) == (10, 15000, 32, 0, 1)
    p = lsr.lsr_head_plan(13, 197, 312, 31091, lsr.LSR_BF16)
    assert (p["dh_chunks"], p["dh_buckets_per_wave"], p["dw_tile_rows"], p["dw_lds_tile_passes"]) == (1, 1, 64, 0)
    # ... and whole rows elsewhere: slices cost sparse gradients too much there
    for shape in ((40, 200, 712, 60000), (64, 64, 776, 60000), (30, 3000, 312, 60000), (16, 250, 904, 200000)):
        p = lsr.lsr_head_plan(*shape, lsr.LSR_BF16)
        assert (p["dh_chunks"], p["dh_buckets_per_wave"], p["dh_waves_per_bucket"], p["dw_tile_rows"], p["dw_lds_tile_passes"]) == (1, 0, 1, 0, 0)
    assert lsr.lsr_head_plan(5, 100, 72, 900, lsr.LSR_F32)["dh_buckets_per_wave"] == 0
    # dW beside dH: from 0.1 GB of gathers on; beyond 16 GB for small slices of H, or from LDS beside a single dH window
    beside = {(64, 512, 1024, 250002): 0, (256, 512, 768, 30522): 1, (128, 512, 1024, 30522): 1, (60, 128, 1024, 80000): 0, (256, 32, 768, 30522): 1,
              (128, 64, 768, 60000): 1, (200, 64, 768, 40000): 0, (256, 40, 768, 30522): 1, (256, 46, 768, 30522): 0, (128, 100, 936, 100000): 0, (16, 256, 768, 250002): 1, (1, 32, 768, 1000): 0}
    for shape, yes in beside.items():
        assert lsr.lsr_head_plan(*shape, lsr.LSR_BF16)["dw_beside_dh"] == yes, shape
    # waves that share a list: surplus waves cost sparse gradients a few per cent at most
    waves = {(64, 32, 768, 30522): 4, (100, 24, 384, 60000): 4, (4, 64, 768, 30522): 4, (32, 128, 1024, 30522): 2, (128, 40, 768, 30522): 2,
             (60, 40, 768, 200000): 2, (64, 100, 768, 50000): 1, (256, 32, 768, 30522): 1, (250, 60, 1024, 100000): 1}
    for shape, n in waves.items():
        assert lsr.lsr_head_plan(*shape, lsr.LSR_BF16)["dh_waves_per_bucket"] == n, shape
    assert lsr.lsr_head_plan(64, 32, 768, 30522, lsr.LSR_F32)["dh_waves_per_bucket"] == 4
    # float32: windows of whole sequences; a single query runs without the auxiliary stream
    p = lsr.lsr_head_plan(64, 32, 768, 30522, lsr.LSR_F32)
    assert (p["fwd_window_segments"], p["fwd_chunks"], p["fwd_segment_rows"]) == (96, 3, 8)
    assert lsr.lsr_head_plan(2, 16, 64, 1000, lsr.LSR_F32)["dw_beside_dh"] == 0


def test_plan_invariants_on_random_shapes():
    rng = np.random.default_rng(11)
    for _ in range(3000):
        B = int(rng.choice([1, 2, 7, 16, 64, 192, 193, 256, 384, 385, 1000, 6144]))
        S = int(rng.choice([1, 5, 32, 33, 512, 1024, 1025, 4096, 8192]))
        D = int(rng.choice([8, 64, 72, 128, 712, 728, 768, 1024, 4096]))
        V = int(rng.choice([1, 63, 512, 4097, 30522, 32769, 65536, 250002, 1000003]))
        if B * V >= 2 ** 31 or B * S >= 2 ** 31:
            continue
        for dt, esize in ((lsr.LSR_BF16, 2), (lsr.LSR_F32, 4)):
            p = lsr.lsr_head_plan(B, S, D, V, dt)
            n_seg, seg_len = p["sort_segments"], p["sort_segment_len"]
            assert n_seg >= 1 and seg_len % 64 == 0 and n_seg * seg_len >= V and (n_seg - 1) * seg_len < V
            assert n_seg == 1 or n_seg * S <= V + S              # count table stays within about B*V ints
            if S <= 1024:
                assert seg_len <= 4096 and p["sort_places_through_lds"] == 1
            else:
                assert p["sort_places_through_lds"] == 0
            c, clen = p["dh_chunks"], p["dh_chunk_len"]
            assert 1 <= c <= 64 and c * clen >= V and (c - 1) * clen < V
            ragged = D % 64 != 0
            rows, nb = p["dw_tile_rows"], p["dw_sequences_per_launch"]
            assert 1 <= nb <= B and (B + nb - 1) // nb <= 16
            # several launches only where rows of H are reused often, and few enough that re-reading dW stays small
            assert nb == B or (V >= 16 * S and (B + nb - 1) // nb <= min(16, 1 + B * esize // 32))
            assert p["dh_waves_per_bucket"] in (1, 2, 4)
            whole_rows = p["dh_buckets_per_wave"] == 0
            if whole_rows:
                assert ragged and (S > 64 or D > 720) and c == 1 and rows == 0 and p["dh_waves_per_bucket"] == 1
                assert p["dh_slices_owned_by_xcd"] == 0 and p["dw_lds_tile_passes"] == 0
            else:
                assert p["dh_buckets_per_wave"] in ((1, 2, 4) if dt == lsr.LSR_F32 else (1, 2, 4, 8))
                assert c == 1 or c <= V * esize // (32 * S)      # re-reading dH stays below a quarter of the gathers
                if ragged:
                    # the chunk bounds (c + 1 per bucket) take the place of the counts, which the placement read last
                    assert c == 1 or B * S * (c + 1) <= B * n_seg * S
                assert c == 1 or clen * 64 * esize <= (4 << 20) or c == 64 or c == V * esize // (32 * S) or (ragged and c == n_seg - 1)
                assert rows in (0, 16, 32, 64) and nb * rows * 8 <= 48 * 1024
                assert (rows == 0) == (nb * 16 * 8 > 48 * 1024)
            seg = p["fwd_segment_rows"]
            assert seg == (8 if S <= 64 else 32)
            segs = B * ((S + seg - 1) // seg)
            tiles_max = (segs * seg + 255) // 256
            assert p["fwd_tiles_per_chunk"] >= 1 and p["fwd_chunks"] <= B
            if dt == lsr.LSR_BF16:
                assert (p["fwd_chunks"] - 1) * p["fwd_tiles_per_chunk"] < tiles_max <= p["fwd_chunks"] * p["fwd_tiles_per_chunk"]
            else:
                # windows cover the longest list; the last sequence that begins in one may run on behind it
                win, per_seq = p["fwd_window_segments"], (S + seg - 1) // seg
                assert (p["fwd_chunks"] - 1) * win < segs <= p["fwd_chunks"] * win and win >= per_seq
                assert p["fwd_tiles_per_chunk"] * 256 >= min(segs, win + per_seq - 1) * seg
            # forward workspace: O(B*S) tables, plus one (max, position) slot per chunk and vocabulary entry
            # where a chunk boundary can fall inside a sequence (bf16 path, S above one block)
            fw = lsr.lsr_head_workspace_bytes(B, S, D, V, dt, False)
            tables = 4 * B + 4 * B * S + 4 * (B + 1) + 4 * segs + 8 * seg * segs
            parts = 8 * p["fwd_chunks"] * V if (dt == lsr.LSR_BF16 and S > seg and p["fwd_chunks"] > 1) else 0
            assert tables + parts <= fw <= tables + parts + 8 * 256
            # the backward workspace holds what the plan implies
            # (the sorted (v, g) lists are followed by 256 entries of slack that the dH gather may read, never write)
            need = 8 * (B * V + 256) + 4 * B * n_seg * S + 4 * B * (S + 1) + (4 * B * S * (c + 1) if c > 1 and not ragged else 0)
            if S <= 8192 and B <= 6144:
                ws = lsr.lsr_head_workspace_bytes(B, S, D, V, dt, True)
                assert need <= ws <= need + 4 * 256


def test_plan_argument_errors(lib):
    out = (ctypes.c_int32 * 16)()
    d = binding._desc(2, 16, 64, 1000, lsr.LSR_BF16)
    assert lib.lsr_head_plan(ctypes.byref(d), None) == 1
    bad = binding._desc(2, 16, 60, 1000, lsr.LSR_BF16)
    assert lib.lsr_head_plan(ctypes.byref(bad), out) == 2
    assert lib.lsr_head_plan(None, out) == 1
    assert lib.lsr_head_plan_ex(ctypes.byref(d), out, 0) == 2
    out[14] = out[15] = -5
    assert lib.lsr_head_plan(ctypes.byref(d), out) == 0 and out[13] >= 0      # the first 14 values and nothing behind them
    assert list(out)[14:] == [-5, -5]


def test_float32_forward_grids_stay_launchable():
    """A launch holds fewer than 2^32 threads: 512 per (chunk, tile of 256 vocabulary entries), in groups of four tiles.
    With two sequences and half of the largest B * |V| each window would otherwise be one sequence: 2^23 workgroups."""
    for B in (1, 2, 3, 5, 8, 16, 100, 1000, 65535):
        for S in (1, 8, 64, 65, 512, 4096, 32768):
            for V in ((2 ** 31 - 1) // B, 2 ** 30 // B, 2 ** 26 // B + 1, 256):
                V = min(V, 2 ** 31 - 4097)
                if B * S >= 2 ** 31 or V < 1:
                    continue
                p = lsr.lsr_head_plan(B, S, 8, V, lsr.LSR_F32)
                tiles = ((V + 255) // 256 + 3) // 4 * 4
                assert (tiles * p["fwd_chunks"] + 7) // 8 * 8 * 512 < 2 ** 32, (B, S, V)


def test_bfloat16_gradients_are_staged_only_where_several_launches_add_up():
    """Beside the float32 workspace: B*S*D floats where dH takes several vocabulary chunks, |V|*D floats where the sliced
    dW gather takes several launches; none for the LDS-tile dW kernel, which takes one."""
    for B, S, D, V in ((256, 512, 1000, 100000), (256, 512, 768, 250002), (64, 512, 1024, 250002), (300, 100, 768, 30522),
                       (260, 1024, 72, 30522), (16, 64, 128, 30522), (256, 512, 1000, 30522)):
        p = lsr.lsr_head_plan(B, S, D, V, lsr.LSR_BF16)
        extra = (lsr.lsr_head_backward_ex_workspace_bytes(B, S, D, V, lsr.LSR_BF16, lsr.LSR_BF16)
                 - lsr.lsr_head_workspace_bytes(B, S, D, V, lsr.LSR_BF16, True))
        want = 4 * B * S * D if p["dh_chunks"] > 1 else 0
        if p["dw_tile_rows"] > 0 and p["dw_sequences_per_launch"] < B and p["dw_lds_tile_passes"] == 0:
            want += 4 * V * D
        assert want <= extra <= want + 2 * 256, (B, S, D, V)


def test_every_value_of_the_plan_has_a_name():
    import os
    import re
    header = open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "include", "lsr_head_measure.h")).read()
    assert len(binding.LSR_PLAN_EX_FIELDS) == int(re.search(r"#define LSR_PLAN_EX_SLOTS (\d+)", header).group(1))
    for shape in ((64, 512, 1024, 250002), (1, 32, 768, 30522)):
        p = lsr.lsr_head_plan_ex(*shape, lsr.LSR_BF16)
        assert list(p)[:-1] == list(binding.LSR_PLAN_FIELDS)
        assert {k: p[k] for k in binding.LSR_PLAN_FIELDS} == lsr.lsr_head_plan(*shape, lsr.LSR_BF16)


def test_which_forwards_are_calls_of_few_tokens():
    """Both sides of each line: 64 tokens, the hidden states (in 32-row blocks) and logits in 156 KiB of LDS, 16 sequences
    up to 32768 vocabulary entries; bfloat16 and rows of 512 from 131072 entries on, nothing between.  There the sequences are
    few enough to hide behind the loads.  Odd numbers of rounds of 32768 entries: four (five with at most 32 tokens), from
    D = 768 on six (eight), from D = 1024 on eight.  Even numbers: one more than the row has batches of 256 columns (from D = 768 on
    two more with at most 32 tokens), eight from D = 1280 on; with a part of a batch two, and three, six, seven and eight from
    D = 768, 1024, 1280 and 1600 on; two in rows of 4 KiB.  Eight where the tile kernel could not load directly to LDS."""
    bf, f32 = lsr.LSR_BF16, lsr.LSR_F32
    lines = [
        ((1, 64, 768, 30522, bf), (1, 65, 768, 30522, bf)), ((8, 8, 64, 1000, f32), (5, 13, 64, 1000, f32)),
        ((1, 32, 2176, 30522, bf), (1, 32, 2184, 30522, bf)), ((1, 64, 896, 30522, bf), (1, 64, 904, 30522, bf)),
        ((1, 32, 2176, 30522, bf), (1, 33, 2176, 30522, bf)), ((1, 32, 1088, 300, f32), (1, 32, 1096, 300, f32)),
        ((2, 32, 448, 128, f32), (2, 32, 456, 128, f32)), ((2, 16, 512, 128, f32), (2, 32, 512, 128, f32)),
        ((16, 4, 768, 30522, bf), (17, 3, 768, 30522, bf)), ((16, 1, 8, 1, f32), (17, 1, 8, 1, f32)),
        ((1, 32, 768, 32768, bf), (1, 32, 768, 32769, bf)), ((1, 32, 768, 32768, f32), (1, 32, 768, 32769, f32)),
        ((1, 32, 768, 131072, bf), (1, 32, 768, 131071, bf)), ((1, 32, 512, 250002, bf), (1, 32, 504, 250002, bf)),
        ((1, 16, 512, 250002, bf), (1, 16, 512, 250002, f32)), ((8, 8, 520, 131100, bf), (9, 7, 520, 131100, bf)),
        ((3, 20, 512, 131072, bf), (4, 16, 512, 131072, bf)), ((4, 16, 768, 131072, bf), (5, 12, 768, 131072, bf)),
        ((6, 5, 1024, 250002, bf), (7, 4, 1024, 250002, bf)), ((2, 32, 640, 131072, bf), (3, 20, 640, 131072, bf)),
        ((5, 6, 768, 131072, bf), (5, 7, 768, 131072, bf)), ((3, 10, 512, 131072, bf), (4, 8, 512, 131072, bf)),
        ((8, 4, 1280, 131072, bf), (8, 4, 1344, 131072, bf)), ((8, 4, 1600, 131072, bf), (8, 4, 1472, 131072, bf)),
        ((7, 4, 1344, 131072, bf), (7, 4, 1216, 131072, bf)), ((6, 5, 1088, 131072, bf), (6, 5, 960, 131072, bf)),
        ((3, 20, 832, 131072, bf), (3, 20, 704, 131072, bf)),
        ((2, 16, 2048, 131072, bf), (3, 10, 2048, 131072, bf)), ((4, 16, 640, 131100, bf), (5, 12, 640, 131100, bf)),
        ((5, 6, 640, 131100, bf), (6, 5, 640, 131100, bf)), ((6, 10, 768, 163840, bf), (7, 9, 768, 163840, bf)),
        ((8, 4, 768, 163840, bf), (8, 5, 768, 163840, bf)), ((8, 4, 1024, 131073, bf), (8, 4, 1024, 163841, bf)),
        ((6, 10, 896, 131073, bf), (6, 10, 896, 131072, bf)),
        ((8, 4, 2048, 131073, bf), (8, 4, 2048, 131072, bf)), ((8, 8, 520, 131072, bf), (8, 8, 512, 131072, bf)),
    ]
    for yes, no in lines:
        assert lsr.lsr_head_plan_ex(*yes)["fwd_few_tokens"] == 1, yes
        assert lsr.lsr_head_plan_ex(*no)["fwd_few_tokens"] == 0, no


def test_where_dw_runs():
    """dW/db in a launch of the dH chain, on the auxiliary stream beside it or behind it.  With several vocabulary windows of dH
    bfloat16 gradients are staged and keep a launch of their own; the plan's dw_beside_dh is the answer for float32 ones."""
    bf, f32 = lsr.LSR_BF16, lsr.LSR_F32
    behind, aux, placement, dh = lsr.LSR_DW_BEHIND_DH, lsr.LSR_DW_ON_AUX_STREAM, lsr.LSR_DW_IN_PLACEMENT_LAUNCH, lsr.LSR_DW_IN_DH_LAUNCH
    for shape, dt, as_f32, as_bf16 in (
            ((8, 30, 128, 100000), bf, dh, aux), ((12, 40, 64, 100000), bf, dh, aux), ((4, 30, 128, 100000), bf, dh, placement),
            ((13, 64, 312, 9000), bf, dh, dh), ((65, 40, 256, 14000), bf, aux, aux), ((64, 512, 1024, 250002), bf, behind, behind),
            ((3, 128, 128, 131100), bf, aux, aux), ((6, 70, 128, 900), bf, placement, placement),
            # up to three sequences with several windows: by the size of dW
            ((1, 69, 1024, 46510), bf, aux, aux), ((1, 14, 600, 90968), bf, aux, aux), ((3, 737, 1024, 17089), f32, dh, None), ((3, 737, 1024, 17090), f32, aux, None),
            ((4, 15, 512, 55539), bf, dh, aux), ((2, 51, 600, 20036), f32, dh, None), ((1, 30, 600, 32769), bf, dh, placement),
            ((20, 64, 832, 12160), bf, aux, aux), ((5, 143, 1536, 14121), f32, aux, None), ((13, 109, 768, 21410), bf, aux, aux),      # two waves per bucket
            ((8, 30, 128, 50000), f32, dh, None), ((2, 16, 64, 1000), f32, placement, None)):
        assert lsr.lsr_head_dw_route(*shape, dt) == as_f32, (shape, dt)
        assert lsr.lsr_head_plan(*shape, dt)["dw_beside_dh"] == (as_f32 == aux)
        if as_bf16 is not None:
            assert lsr.lsr_head_dw_route(*shape, dt, lsr.LSR_BF16) == as_bf16, shape
    for bad, status in (((2, 16, 60, 1000, bf, f32), 2), ((2, 16, 64, 1000, f32, bf), 3), ((2, 16, 64, 1000, bf, 9), 3),
                        ((2, 8193, 64, 1000, bf, f32), 2), ((6145, 2, 64, 1000, bf, f32), 2)):
        with pytest.raises(lsr.LsrError) as e:
            lsr.lsr_head_dw_route(*bad)
        assert e.value.status == status, bad
    route = ctypes.c_int32(-5)
    d = binding._desc(2, 16, 64, 1000, bf)
    assert binding.load_library().lsr_head_dw_route(ctypes.byref(d), None, None) == 1
    assert binding.load_library().lsr_head_dw_route(None, None, ctypes.byref(route)) == 1 and route.value == -5
    assert binding.load_library().lsr_head_dw_route(ctypes.byref(d), None, ctypes.byref(route)) == 0 and route.value == placement
