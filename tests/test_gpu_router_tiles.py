"""The router as a launch of its own: four tiles per workgroup (large batches) against one, on the same
tokens in smaller calls, bit for bit, and against float64.  Expert and token tiles that do not fill a
workgroup, reductions shorter than a workgroup's wavefronts and with a remainder.  (test_launch_plans.py
holds the sizes to those two forms.)"""
import numpy as np
import pytest
import torch

from paper_2602_00879_amd import binding as B
from paper_2602_00879_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu


# (experts, width, tokens, tokens of a smaller call)
ROUTER = [(136, 96, 1073, 100), (256, 2048, 530, 131), (24, 3104, 2200, 550), (24, 32, 4096, 1000)]


@pytest.mark.parametrize("M,D,T,part", ROUTER)
def test_router_tiles(M, D, T, part):
    print(f"router {M} {D} {T}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.randn((1, T, D), generator=g, device="cuda").bfloat16()
    w = (torch.randn((M, D), generator=g, device="cuda") * 0.02).bfloat16()
    bias = torch.randn(M, generator=g, device="cuda")

    def route(rows):
        shape = B.make_shape(1, rows.shape[1], D, M, 32, 1, M, "vanilla", "bf16")
        return B.des_route(shape, rows.contiguous(), w, bias)

    logits, probs = route(x)
    for t in range(0, T, part):
        l, p = route(x[:, t:t + part])
        assert torch.equal(l, logits[:, t:t + part]) and torch.equal(p, probs[:, t:t + part])
    ref = x[0].double().cpu().numpy() @ w.double().cpu().numpy().T + bias.double().cpu().numpy()
    assert np.abs(logits[0].cpu().numpy() - ref).max() <= H.LOGIT_ATOL


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N", [(3, 1), (16, 16), (16, 17), (17, 16)])
@pytest.mark.parametrize("mode", ["vote", "seq", "vanilla"])
def test_one_tile_and_its_neighbours(dtype, M, N, mode):
    """A single router tile is computed by the selector's workgroup, two by workgroups of their own."""
    cfg = W.LayerConfig("one_tile", dtype, 1, N, 64, M, 32, 0, 2, 3, 1.1, 41)
    layer = W.make_layer(cfg)
    out = H.run_gpu(cfg, H.layer_to_device(layer), mode)
    H.check_against_oracle(cfg, layer, out, mode, label=f"{dtype} {M} {N} {mode}")
