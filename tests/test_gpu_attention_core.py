"""The attention sub-layer at the sizes where the split of a head's work can go wrong: query
rows that do not fill a tile or span query heads, windows around a multiple of 32 positions,
windows kept whole (up to 256 positions, and up to 512 in large batches), cut into 2, 4 and 8
parts (a part may be empty) with one and several query tiles per workgroup, or scored twice,
one and many workgroups per head, head widths that are no multiple of 16 or 32.  Every token
against the CPU oracle; the projections' tiles with them.  Also: scores beyond the range of
fp32, and that a sequence's result does not depend on the size of its batch."""
import numpy as np
import pytest
import torch

from oracle import des_oracle as O
from paper_2602_00879_amd import binding as B
from paper_2602_00879_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

# (sequences, tokens, hidden, query heads, key/value heads, head width, cached positions)
CASES = {
    "one_row_one_key": (1, 1, 128, 16, 16, 8, 0),
    "rows_15": (1, 5, 128, 24, 8, 16, 11),
    "rows_17": (1, 17, 128, 8, 8, 16, 14),
    "window_31": (1, 3, 128, 8, 2, 64, 28),
    "window_32": (1, 4, 128, 8, 2, 64, 28),
    "window_33": (1, 5, 128, 8, 2, 64, 28),
    "window_96_three_steps": (1, 16, 256, 4, 2, 128, 80),
    "window_160_five_steps": (1, 16, 256, 4, 1, 128, 144),
    "window_193": (1, 16, 256, 4, 1, 128, 177),
    "window_255": (1, 16, 256, 4, 2, 128, 239),
    "window_256": (2, 9, 256, 4, 2, 128, 247),
    "window_257_four_parts_the_last_empty": (2, 9, 256, 2, 1, 128, 248),
    "window_at_the_limit_eight_parts": (1, 28, 128, 1, 1, 128, 572),
    "narrow_heads_eight_parts": (1, 20, 128, 16, 4, 24, 700),
    "two_parts_two_tiles": (40, 25, 128, 16, 16, 64, 245),
    "two_parts_four_tiles": (64, 25, 128, 16, 4, 32, 235),
    "four_parts_two_tiles": (8, 32, 256, 32, 4, 128, 464),
    "four_parts_two_tiles_ragged": (8, 31, 256, 32, 4, 120, 466),
    "wide_257": (33, 31, 128, 32, 8, 16, 226),
    "wide_512": (32, 32, 128, 32, 8, 40, 480),
    "twice_large_batch": (32, 32, 128, 32, 8, 96, 500),
    "twice_narrow": (1, 20, 128, 16, 4, 16, 2100),
    "many_rows": (4, 128, 128, 32, 4, 40, 30),
    "batch": (64, 32, 256, 16, 2, 64, 32),
    "long_block": (1, 300, 128, 4, 4, 32, 7),
    # the projections' forms: tiles with the reduction whole or cut, rows and columns that do
    # not fill a tile, a reduction of whole 64-element chunks and of one chunk more or less,
    # large and wide matrices (test_gpu_projection_tiles.py has an entry per tile)
    "tile_33_rows": (1, 33, 128, 4, 2, 32, 3),
    "tile_cut_65_rows": (1, 65, 1024, 8, 2, 64, 3),
    "tile_whole_65_rows": (5, 13, 1152, 8, 2, 48, 0),
    "tile_large": (10, 103, 1152, 72, 8, 128, 0),
    "tile_50_rows_wide": (1, 50, 8192, 64, 1, 128, 0),
    "tile_64_rows_odd_length": (2, 32, 8192, 65, 1, 128, 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_attention_core(name):
    Bn, N, D, Hq, G, dh, P = CASES[name]
    print(f"attention core {name}", flush=True)
    cfg = W.AttnConfig(name, Bn, N, D, Hq, G, dh, P, 0, 91)
    t = W.make_attention(cfg)
    dev = {k: H.dev_tensor(v) for k, v in t.items()}
    shape = B.make_shape(Bn, N, D, 16, 128, 2, 4, "vanilla", "bf16")
    attn = B.make_attn_shape(Hq, G, dh, P, 0)
    y = B.des_block_attention(shape, attn, dev["x"], dev["wq"], dev["wk"], dev["wv"], dev["wo"],
                              dev["k_cache"] if P else None, dev["v_cache"] if P else None)
    torch.cuda.synchronize()
    f = {k: W.to_f64(v) for k, v in t.items()}
    ref = O.block_attention(f["x"], f["wq"], f["wk"], f["wv"], f["wo"], f["k_cache"], f["v_cache"], Hq, G)
    d = y.float().cpu().numpy().astype(np.float64) - ref
    rel = np.sqrt((d ** 2).sum() / (ref ** 2).sum())
    # q, k, v, the weights, the heads' outputs and y are each rounded to bf16 once (2^-9 relative at
    # most): 1e-2 relative in all.  A single element: the errors spread like the outputs, with a
    # standard deviation of rel x rms; eight of them leave out nobody among 10^7 elements even where
    # outputs (and with them the last rounding's errors) differ in size several times over
    rms = np.sqrt((ref ** 2).mean())
    print(f"  max {np.abs(d).max():.2e} rms {rms:.2e} rel {rel:.2e}", flush=True)
    bound = 8 * rel * rms
    assert np.abs(d).max() <= bound and rel <= H.BF16_REL_L2, (name, np.abs(d).max(), rel)


# A form of the attention core per entry: (sequences, tokens, query heads, key/value heads, head
# width, cached positions) and the cached positions to push out of range.
OUT_OF_RANGE = {
    "whole": ((1, 16, 2, 1, 128, 180), [(0, 64), (64, 180)]),
    "parts_first_steps": ((1, 16, 2, 1, 128, 470), [(0, 64)]),
    "parts_a_whole_part": ((1, 16, 2, 1, 128, 470), [(0, 130), (250, 330)]),
    "parts_all_cached": ((8, 16, 8, 1, 128, 470), [(0, 470)]),
    "wide": ((128, 8, 32, 2, 64, 400), [(0, 100), (300, 400)]),
    "twice": ((1, 16, 8, 2, 16, 2200), [(0, 300), (1000, 2100)]),
}


@pytest.mark.parametrize("name", list(OUT_OF_RANGE))
def test_scores_of_minus_infinity_weigh_nothing(name):
    """Finite keys whose scores overflow fp32 to -inf: those positions have weight zero, as in
    exact arithmetic, wherever in the window they lie."""
    (Bn, N, Hq, G, dh, P), ranges = OUT_OF_RANGE[name]
    print(f"out of range {name}", flush=True)
    cfg = W.AttnConfig(name, Bn, N, 128, Hq, G, dh, P, 0, 93)
    t = W.make_attention(cfg)
    dev = {k: H.dev_tensor(v) for k, v in t.items()}
    dev["x"], dev["wq"] = dev["x"].abs(), dev["wq"].abs()       # every query coordinate positive
    for lo, hi in ranges:
        dev["k_cache"][:, :, lo:hi] = -3.0e38                   # (the largest bf16 is 3.39e38)
    shape = B.make_shape(Bn, N, 128, 16, 128, 2, 4, "vanilla", "bf16")
    y = B.des_block_attention(shape, B.make_attn_shape(Hq, G, dh, P, 0), dev["x"], dev["wq"], dev["wk"], dev["wv"],
                              dev["wo"], dev["k_cache"], dev["v_cache"])
    torch.cuda.synchronize()
    assert bool(torch.isfinite(y).all()), name
    f = {k: v.double().cpu().numpy() for k, v in dev.items()}
    ref = O.block_attention(f["x"], f["wq"], f["wk"], f["wv"], f["wo"], f["k_cache"], f["v_cache"], Hq, G)
    d = y.double().cpu().numpy() - ref
    assert np.sqrt((d ** 2).sum() / (ref ** 2).sum()) <= H.BF16_REL_L2, name


@pytest.mark.parametrize("G", [1, 9])
def test_a_sequence_does_not_depend_on_its_batch(G):
    """A window of 300 positions under 1, 24 and 100 sequences of 40 tokens takes different cuts and
    forms; a sequence's result is the same bits.  (More than 32 rows and widths that are no multiple
    of 512, so that the projections add in one order at every size.)"""
    Bn, N, D, Hq, dh, P = 100, 40, 384, 9, 128, 260
    t = W.make_attention(W.AttnConfig("batch", Bn, N, D, Hq, G, dh, P, 0, 95))
    dev = {k: H.dev_tensor(v) for k, v in t.items()}
    attn = B.make_attn_shape(Hq, G, dh, P, 0)

    def run(lo, hi):
        print(f"batch of {hi - lo}, {G} key/value heads", flush=True)
        shape = B.make_shape(hi - lo, N, D, 16, 128, 2, 4, "vanilla", "bf16")
        y = B.des_block_attention(shape, attn, dev["x"][lo:hi].contiguous(), dev["wq"], dev["wk"], dev["wv"], dev["wo"],
                                  dev["k_cache"][lo:hi].contiguous(), dev["v_cache"][lo:hi].contiguous())
        torch.cuda.synchronize()
        return y

    whole = run(0, Bn)
    assert torch.equal(run(30, 54), whole[30:54])
    for b in (0, 57, 99):
        assert torch.equal(run(b, b + 1)[0], whole[b]), b
