"""GPU parity of the short-block expert kernels where their pipelines and row groups end: row
groups that do not fill (the hidden width is no multiple of 64), one to nine stages with and
without left-over k-steps, one and two token tiles, with and without a shared expert, under
DES (dense handling) and vanilla, both weight layouts.  Every token against the CPU oracle."""
import pytest
import torch

from paper_2602_00879_amd import binding as B
from paper_2602_00879_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

# (sequences, tokens, D, M, F, Fs, K, C)
BLOCKS = {
    "ragged_7_stages": (7, 1, 928, 24, 448, 448, 1, 18),
    "ragged_3_stages_two_tiles": (1, 20, 224, 16, 192, 0, 4, 6),
    "ragged_5_stages_and_a_step": (2, 9, 160, 16, 352, 32, 3, 6),
    "ragged_1_stage": (1, 5, 96, 8, 64, 0, 2, 4),
    "one_step": (1, 32, 32, 8, 32, 0, 2, 4),
    "fine_stages": (1, 17, 544, 40, 800, 0, 4, 5),
    "nine_stages": (1, 31, 576, 32, 576, 64, 8, 8),
}


@pytest.mark.parametrize("name", list(BLOCKS))
@pytest.mark.parametrize("mode", ["vote", "vanilla"])
def test_short_blocks(name, mode):
    Bn, N, D, M, F, Fs, K, C = BLOCKS[name]
    print(f"short block {name} {mode}", flush=True)
    cfg = W.LayerConfig(name, "bf16", Bn, N, D, M, F, Fs, K, C, 1.1, 73)
    layer = W.make_layer(cfg)
    dev = H.layer_to_device(layer)
    out = H.run_gpu(cfg, dev, mode)
    H.check_against_oracle(cfg, layer, out, mode, label=f"{name} {mode}")
    sh = None if dev["shared"] is None else tuple(B.des_pack_expert_weights(m) for m in dev["shared"])
    packed = (*(B.des_pack_expert_weights(dev[k]) for k in ("w_gate", "w_up", "w_down")), sh)
    out_p = H.run_gpu(cfg, dev, mode, layout=B.DES_LAYOUT_PACKED, packed_weights=packed)
    assert torch.equal(out.y, out_p.y) and torch.equal(out.topk_idx, out_p.topk_idx)


@pytest.mark.parametrize("D", [4, 68, 1024])
def test_fp32_router_scores_do_not_depend_on_the_number_of_tokens(D):
    """Tokens are scored in groups of eight, four, two and one: the same bits for a token in any
    of them.  Against float64: a score is rounded D / 64 + 8 times on its way (a lane's products, six
    steps over the lanes, the bias), each time by at most 2^-24 of a number below 6 sqrt(D)."""
    M, T = 19, 35
    g = torch.Generator().manual_seed(5)
    x, w, b = (torch.randn(*s, generator=g) for s in ((1, T, D), (M, D), (M,)))
    xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
    print(f"fp32 router, width {D}", flush=True)
    ref = x.double()[0] @ w.double().T + b.double()
    want = None
    for n in range(T, 0, -1):
        shape = B.make_shape(1, n, D, M, 4, 2, 4, "vote", "f32")
        logits, _ = B.des_route(shape, xd[:, :n].contiguous(), wd, bd)
        torch.cuda.synchronize()
        if want is None:
            want = logits[0]
            assert (want.cpu().double() - ref).abs().max().item() <= (D / 64 + 8) * 2.0 ** -24 * 6 * D ** 0.5
        assert torch.equal(logits[0], want[:n]), n
