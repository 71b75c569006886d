"""GPU parity of batches of many sequences: the routing runs as launches of its own there,
the permutation over several workgroups, and an expert may have hundreds of pairs.  Every
token against the CPU oracle; integers exact."""
import pytest
import torch

from paper_2602_00879_amd import binding as B
from paper_2602_00879_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu


# (sequences, tokens of each, D, M, F, Fs, K, C): pairs below, at and beyond what one
# permutation workgroup takes (2048), token counts that are no multiple of 32, the most
# tokens the library accepts, M * ceil(T / 32) at its limit, more pairs per expert than a
# unit's rows times the units of an expert
BATCHES = {
    "pairs_2049": (3, 683, 64, 24, 32, 0, 1, 6),
    "pairs_2048": (32, 32, 64, 24, 32, 0, 2, 6),
    "ragged": (37, 29, 160, 40, 96, 96, 3, 9),
    "aligned": (64, 32, 256, 128, 128, 0, 8, 32),
    "most_tokens": (32, 128, 128, 64, 128, 128, 4, 8),
    "few_experts": (20, 100, 128, 8, 256, 0, 2, 3),
    # the tiles of the expert kernels: units of at most 64 rows, reductions of whole chunks of
    # 64 and half a chunk more (one chunk at most, too), row tiles that do not fill a workgroup,
    # a shared expert of another width, unrolled and other packed sizes on both
    # sides of 32 pairs per expert
    "tiles_small": (5, 10, 224, 16, 160, 160, 2, 4),
    "tiles_33_tokens": (3, 11, 32, 16, 32, 0, 3, 5),
    "tiles_96_rows": (1, 97, 288, 8, 224, 64, 4, 4),
    "streamed_31_pairs": (5, 33, 256, 16, 384, 128, 3, 6),
    "tiles_32_pairs": (5, 35, 256, 16, 384, 128, 3, 6),
    "unrolled_256_tokens": (8, 32, 2048, 8, 512, 512, 2, 4),
    # ... enough workgroups for four row tiles per wavefront, and fewer (two, one chunk ahead),
    # in units of 64 and of 128 rows, row tiles that do not fill a workgroup
    "tiles_four_60_tokens": (2, 30, 160, 256, 96, 32, 4, 256),
    "tiles_four_150_tokens": (3, 50, 416, 128, 224, 96, 7, 128),
    "tiles_two_60_tokens": (2, 30, 96, 128, 96, 0, 3, 128),
    "tiles_two_150_tokens": (1, 150, 96, 64, 288, 0, 4, 64),
}


@pytest.mark.parametrize("name", list(BATCHES))
@pytest.mark.parametrize("mode", ["vote", "vanilla"])
def test_batches(name, mode):
    Bn, N, D, M, F, Fs, K, C = BATCHES[name]
    print(f"batch {name} {mode}", flush=True)
    cfg = W.LayerConfig(name, "bf16", Bn, N, D, M, F, Fs, K, C, 1.1, 71)
    layer = W.make_layer(cfg)
    dev = H.layer_to_device(layer)
    out = H.run_gpu(cfg, dev, mode)
    H.check_against_oracle(cfg, layer, out, mode, label=f"{name} {mode}")
    sh = None if dev["shared"] is None else tuple(B.des_pack_expert_weights(m) for m in dev["shared"])
    packed = (*(B.des_pack_expert_weights(dev[k]) for k in ("w_gate", "w_up", "w_down")), sh)
    out_p = H.run_gpu(cfg, dev, mode, layout=B.DES_LAYOUT_PACKED, packed_weights=packed)
    assert torch.equal(out.y, out_p.y) and torch.equal(out.topk_idx, out_p.topk_idx)
