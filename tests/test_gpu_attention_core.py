"""The attention sub-layer at the sizes where the split of a head's work can go wrong: query
rows that do not fill a tile or span query heads, windows around a multiple of 32 positions,
windows cut into 1 to 8 parts (a part may be empty), one and many workgroups per head, head
widths that are no multiple of 16 or 32.  Every token against the CPU oracle; the projections' tiles with them."""
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
    "window_257_nine_steps_eight_parts": (2, 9, 256, 2, 1, 128, 248),
    "window_at_the_limit": (1, 28, 128, 1, 1, 128, 572),
    "narrow_heads_long_window": (1, 20, 128, 16, 4, 24, 700),
    "many_rows": (4, 128, 128, 32, 4, 40, 30),
    "batch": (64, 32, 256, 16, 2, 64, 32),
    "long_block": (1, 300, 128, 4, 4, 32, 7),
    # the projections' forms: tiles with the reduction whole or cut, rows and columns that do
    # not fill a tile, a reduction of whole 64-element chunks and of one chunk more or less,
    # the large tile, the streamed one
    "tile_33_rows": (1, 33, 128, 4, 2, 32, 3),
    "tile_cut_65_rows": (1, 65, 1024, 8, 2, 64, 3),
    "tile_whole_65_rows": (5, 13, 1152, 8, 2, 48, 0),
    "tile_large": (10, 103, 1152, 72, 8, 128, 0),
    "streamed_50_rows": (1, 50, 8192, 64, 1, 128, 0),
    "streamed_64_rows_odd_length": (2, 32, 8192, 65, 1, 128, 0),
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
    # q, k, v, the weights and the heads' outputs are each rounded to bf16 once (2^-9 relative):
    # 1e-2 relative in all.  A single element: the benchmark's absolute bound holds for outputs
    # of order one; wide layers have larger ones (weights N(0, 0.02): rms 0.02 sqrt(width) times
    # the heads'), where errors of standard deviation at most 1e-2 rms stay below six of them
    # over 10^6 elements
    bound = max(H.BF16_MAX_ABS, 6 * H.BF16_REL_L2 * np.sqrt((ref ** 2).mean()))
    assert np.abs(d).max() <= bound and rel <= H.BF16_REL_L2, (name, np.abs(d).max(), rel)
