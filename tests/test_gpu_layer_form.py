"""A layer call asks once how many compute units there are and decides from that how its routing is launched; what
the expert FFN then reads is what those launches leave.  One failed question (the call takes three routing launches)
gives the bits of the single launch, with scratch that holds nothing of an earlier call."""
import pytest
import torch

from paper_2602_00879_amd import binding as B
from paper_2602_00879_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

KEYS = ("y", "logits", "topk_idx", "topk_w", "expert_counts", "n_unique", "coreset_idx", "coreset_size")


@pytest.mark.parametrize("Bn,N", [(1, 20), (3, 9), (1, 40)])
@pytest.mark.parametrize("mode", ["vanilla", "vote"])
def test_one_answer_decides_for_the_whole_layer(mode, Bn, N):
    cfg = W.LayerConfig("layer_form", "bf16", Bn, N, 256, 40, 64, 32, 4, 10, 1.1, 31)
    layer = W.make_layer(cfg)
    dev = H.layer_to_device(layer)
    shape = H.shape_of(cfg, mode, residual=1)
    args = (shape, dev["x"], dev["w_router"], dev["bias"], dev["w_gate"], dev["w_up"], dev["w_down"])
    ref = B.des_moe_forward(*args, shared=dev["shared"])
    torch.cuda.synchronize()
    H.check_against_oracle(cfg, layer, ref, mode, residual=True, label=f"{mode} {Bn}x{N}")
    for answer in (0, 4):  # none, and too few for the single launch
        bufs = B.MoeBuffers(shape, "cuda", torch.bfloat16)
        bufs.workspace.fill_(0xFF)
        print(f"{mode} {Bn}x{N}: told of {answer} compute units", flush=True)
        B.des_test_compute_units(answer)
        B.des_moe_forward(*args, shared=dev["shared"], buffers=bufs)
        torch.cuda.synchronize()
        for k in KEYS:
            assert torch.equal(getattr(bufs, k), getattr(ref, k)), (k, answer)
        B.des_moe_forward(*args, shared=dev["shared"], buffers=bufs)  # asks the device again
        torch.cuda.synchronize()
        assert torch.equal(bufs.y, ref.y)
