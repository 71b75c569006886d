"""The streamed expert kernels with four weight tiles per wavefront (packed weights, many pairs per
expert), at the edges of their sizes: the shortest reduction, row tiles that do not fill a workgroup,
units of one expert side by side (up to sixteen, more than one block of eight), a shared expert of
another width.  Every token against the CPU oracle, and bit for bit against the tile kernels on the
same weights row-major, which add up in the same order."""
import pytest
import torch

from paper_2602_00879_amd import binding as B
from paper_2602_00879_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

# (sequences, tokens of each, D, M, F, Fs, K, C)
WIDE = {
    "gate_two_chunks": (3, 501, 128, 8, 896, 0, 2, 8),
    "gate_ragged_rows": (3, 499, 256, 8, 1120, 0, 2, 8),
    "down_two_chunks_ragged": (12, 125, 1888, 8, 128, 0, 2, 8),
    "shared": (16, 125, 1152, 16, 640, 256, 2, 12),
    "sixteen_units": (2, 1030, 640, 6, 1152, 0, 2, 3),
}


@pytest.mark.parametrize("name", list(WIDE))
def test_wide_streams(name):
    Bn, N, D, M, F, Fs, K, C = WIDE[name]
    print(f"wide {name}", flush=True)
    cfg = W.LayerConfig(name, "bf16", Bn, N, D, M, F, Fs, K, C, 1.1, 83)
    layer = W.make_layer(cfg)
    dev = H.layer_to_device(layer)
    sh = None if dev["shared"] is None else tuple(B.des_pack_expert_weights(m) for m in dev["shared"])
    packed = (*(B.des_pack_expert_weights(dev[k]) for k in ("w_gate", "w_up", "w_down")), sh)
    out = H.run_gpu(cfg, dev, "vote", layout=B.DES_LAYOUT_PACKED, packed_weights=packed)
    H.check_against_oracle(cfg, layer, out, "vote", label=name)
    assert torch.equal(out.y, H.run_gpu(cfg, dev, "vote").y)
