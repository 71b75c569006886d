"""The selection reads a token's logits four at a time where rows are whole, aligned fours, else one by one:
the same logits at addresses that are 16-byte aligned and at others elect the same coreset from the same
votes, bit for bit, and the votes are those of float64.  Expert counts that are multiples of eight, four, two and one."""
import numpy as np
import pytest
import torch

from paper_2602_00879_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [5, 60, 100, 128, 130, 252, 512])
@pytest.mark.parametrize("mode", ["vote", "seq"])
def test_logits_at_any_address(M, mode):
    Bn, N, K, C = 3, 37, min(5, M), max(5, M // 4)
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    logits = torch.randn((Bn, N, M), generator=g, device="cuda")
    shape = B.make_shape(Bn, N, 32, M, 32, K, C, mode, "bf16")
    ref = B.des_select_coreset(shape, logits)
    for shift in (1, 2, 3):
        buf = torch.empty(logits.numel() + 8, device="cuda")
        moved = buf[shift:shift + logits.numel()].view(Bn, N, M)
        moved.copy_(logits)
        assert moved.data_ptr() % 16 == 4 * shift
        out = B.des_select_coreset(shape, moved)
        for k in ref:
            assert torch.equal(out[k], ref[k]), (k, shift)
    if mode == "vote":  # softmax weights of each token's K best experts, summed over the tokens
        l = logits.double().cpu().numpy()
        p = np.exp(l - l.max(-1, keepdims=True))
        p /= p.sum(-1, keepdims=True)
        keep = np.zeros_like(p, dtype=bool)
        np.put_along_axis(keep, np.argsort(-l, axis=-1, kind="stable")[..., :K], True, -1)
        # (fp32: the exponential and its sum to a few 2^-24 each, up to 37 votes added)
        np.testing.assert_allclose(ref["votes"].cpu().numpy(), (p * keep).sum(1), rtol=4e-6, atol=1e-7)
