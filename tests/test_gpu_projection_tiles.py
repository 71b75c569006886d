"""Every tile that the attention projections of more than 32 rows choose from (64 x 64 down to 32 x 32
rows and up to 128 x 128, the reduction whole or in two halves; the largest straight into LDS and through
registers), with rows and columns that do not fill it and the shortest reduction.  Every token against the
CPU oracle, as for the attention core.  test_launch_plans.py holds each entry to the tiles it names."""
import numpy as np
import pytest
import torch

from oracle import des_oracle as O
from paper_2602_00879_amd import binding as B
from paper_2602_00879_amd import workloads as W
from tests import helpers as H
from tests import test_gpu_attention_core as core

pytestmark = pytest.mark.gpu

# (sequences, tokens, hidden, query heads, key/value heads, head width, cached positions), then the tiles
# of q/k/v and output: units of 32 rows (weights, tokens), parts of the reduction, 1 = through registers
TILES = {
    "two_chunks": ((1, 33, 128, 4, 2, 32, 0), (1, 1, 1, 0), (1, 1, 1, 0)),
    "cut_small": ((1, 45, 512, 8, 2, 64, 5), (1, 1, 2, 0), (1, 1, 2, 0)),
    "cut_64_x_32": ((6, 77, 512, 8, 2, 64, 0), (2, 1, 2, 0), (1, 1, 2, 0)),
    "64_x_32": ((3, 50, 1152, 40, 4, 128, 0), (2, 1, 1, 0), (1, 1, 2, 0)),
    "cut_64_x_64": ((8, 90, 512, 8, 2, 64, 0), (2, 2, 2, 0), (2, 1, 2, 0)),
    "64_x_64": ((10, 103, 256, 8, 2, 32, 0), (2, 2, 1, 0), (1, 1, 1, 0)),
    "cut_128_x_64": ((10, 103, 512, 8, 2, 64, 3), (4, 2, 2, 0), (2, 2, 2, 0)),
    "128_x_64": ((2, 65, 1152, 72, 8, 128, 0), (4, 2, 1, 0), (1, 1, 2, 0)),
    "128_x_128": ((6, 77, 1152, 72, 8, 128, 0), (4, 4, 1, 0), (2, 2, 2, 0)),
    "two_per_unit": ((8, 125, 128, 62, 1, 128, 3), (4, 4, 1, 0), (1, 1, 1, 0)),
    "registers_three_per_unit": ((32, 33, 128, 88, 1, 96, 5), (4, 4, 1, 1), (1, 1, 1, 0)),
}


@pytest.mark.parametrize("name", list(TILES))
def test_projection_tiles(name, monkeypatch):
    monkeypatch.setitem(core.CASES, name, TILES[name][0])
    core.test_attention_core(name)


# The output projection in the register tile, one per compute unit, the last column of tiles not full.
REGISTERS_OUT = ((8, 125, 4096, 16, 2, 128, 0), (4, 2, 1, 0), (4, 4, 1, 1))


def test_register_tile_adds_the_residual():
    Bn, N, D, Hq, G, dh, P = REGISTERS_OUT[0]
    print("register tile, output with residual", flush=True)
    t = W.make_attention(W.AttnConfig("registers_out", Bn, N, D, Hq, G, dh, P, 0, 97))
    dev = {k: H.dev_tensor(v) for k, v in t.items()}
    shape = B.make_shape(Bn, N, D, 16, 128, 2, 4, "vanilla", "bf16", residual=1)
    y = B.des_block_attention(shape, B.make_attn_shape(Hq, G, dh, P, 0), dev["x"], dev["wq"], dev["wk"], dev["wv"],
                              dev["wo"], None, None)
    torch.cuda.synchronize()
    f = {k: W.to_f64(v) for k, v in t.items()}
    out = O.block_attention(f["x"], f["wq"], f["wk"], f["wv"], f["wo"], f["k_cache"], f["v_cache"], Hq, G)
    d = y.double().cpu().numpy() - (f["x"] + out)
    # the projection's error, as in test_attention_core, and the rounding of the sum, 2^-9 of it at most
    rms = np.sqrt((out ** 2).mean())
    rel = np.sqrt((d ** 2).mean()) / rms
    bound = H.BF16_REL_L2 + 2.0 ** -9 * np.sqrt(((f["x"] + out) ** 2).mean()) / rms
    print(f"  rel {rel:.2e} bound {bound:.2e}", flush=True)
    assert rel <= bound
    # no element is out of line: the sum's rounding is at most 2^-8 of the element (half an ulp at the low
    # end of a binade is 2^-9), the rest spreads as in test_attention_core
    assert (np.abs(d) <= 2.0 ** -8 * np.abs(f["x"] + out) + 8 * H.BF16_REL_L2 * rms).all()
