"""Blocks of at most 32 tokens: x is copied into operand order beside the election, or read in rows.  Token
counts that are no multiple of four or 16 and at both sides of the least, several short sequences, one router
tile and many, hidden sizes of one k-step, of fewer pieces than a copying workgroup has threads and of more
than all of them have, with a shared expert.  Every token against the CPU oracle; both weight layouts bit for
bit.  (test_launch_plans.py holds the sizes to the copy.)"""
import pytest
import torch

from paper_2602_00879_amd import binding as B
from paper_2602_00879_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

# (sequences, tokens of each, D, M, F, Fs, K, C)
SHORT = [(1, 1, 32, 16, 32, 32, 1, 2), (3, 5, 96, 24, 64, 0, 3, 6), (31, 1, 64, 40, 32, 96, 2, 5),
         (1, 17, 2080, 16, 32, 32, 2, 4), (4, 8, 4640, 17, 32, 0, 2, 3), (1, 32, 4128, 64, 96, 64, 4, 12)]
# ... whose x is copied, in these modes
COPIED = {(1, 17, 2080, 16, 32, 32, 2, 4): ("vote",), (1, 32, 4128, 64, 96, 64, 4, 12): ("vote",),
          (1, 6, 1024, 16, 32, 0, 1, 3): ("vote",), (1, 7, 1056, 24, 64, 32, 2, 5): ("vote",),
          (1, 31, 1248, 20, 32, 0, 3, 8): ("vote", "vanilla"), (5, 6, 1056, 24, 64, 32, 2, 5): ("vote", "vanilla")}
SHORT += [c for c in COPIED if c not in SHORT] + [(1, 5, 1056, 24, 64, 32, 2, 5), (19, 1, 1024, 16, 32, 0, 1, 3)]


@pytest.mark.parametrize("case", SHORT, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("mode", ["vote", "vanilla"])
def test_x_in_operand_order(case, mode):
    Bn, N, D, M, F, Fs, K, C = case
    cfg = W.LayerConfig("operand_order", "bf16", Bn, N, D, M, F, Fs, K, C, 1.1, 67)
    layer = W.make_layer(cfg)
    dev = H.layer_to_device(layer)
    out = H.run_gpu(cfg, dev, mode, residual=1)
    H.check_against_oracle(cfg, layer, out, mode, residual=True, label=f"{case} {mode}")
    sh = None if dev["shared"] is None else tuple(B.des_pack_expert_weights(m) for m in dev["shared"])
    packed = (*(B.des_pack_expert_weights(dev[k]) for k in ("w_gate", "w_up", "w_down")), sh)
    out_p = H.run_gpu(cfg, dev, mode, layout=B.DES_LAYOUT_PACKED, residual=1, packed_weights=packed)
    assert torch.equal(out.y, out_p.y) and torch.equal(out.topk_idx, out_p.topk_idx)
