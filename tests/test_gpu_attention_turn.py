"""The attention core of 128-wide heads under a cut window loads queries and keys along their rows where many
wavefronts share the compute units, in operand order where few do: the same sequences in a batch and alone,
bit for bit, and against the oracle.  Query rows and windows that do not fill their tiles; windows in two, four
and eight parts, in eight the turned keys need more LDS than what the parts exchange.  (test_launch_plans.py holds
the shapes to those forms.)"""
import numpy as np
import pytest
import torch

from oracle import des_oracle as O
from paper_2602_00879_amd import binding as B
from paper_2602_00879_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu


# (sequences, tokens, key/value heads of nine query heads, cached positions): parts, tiles of a workgroup
TURNED = {(12, 40, 3, 417): (4, 1), (15, 37, 1, 220): (4, 1), (22, 40, 3, 417): (4, 2), (52, 33, 3, 267): (2, 4),
          (7, 33, 1, 452): (8, 1)}


@pytest.mark.parametrize("Bn,N,G,P", list(TURNED))
def test_loads_along_rows(Bn, N, G, P):
    D, Hq, dh = 384, 9, 128  # (the projections add in one order at every size)
    t = W.make_attention(W.AttnConfig("turn", Bn, N, D, Hq, G, dh, P, 0, 97))
    dev = {k: H.dev_tensor(v) for k, v in t.items()}
    attn = B.make_attn_shape(Hq, G, dh, P, 0)

    def run(lo, hi):
        print(f"{hi - lo} sequences of {N}, {G} key/value heads, {P} cached", flush=True)
        shape = B.make_shape(hi - lo, N, D, 16, 128, 2, 4, "vanilla", "bf16")
        y = B.des_block_attention(shape, attn, dev["x"][lo:hi].contiguous(), dev["wq"], dev["wk"], dev["wv"], dev["wo"],
                                  dev["k_cache"][lo:hi].contiguous(), dev["v_cache"][lo:hi].contiguous())
        torch.cuda.synchronize()
        return y

    y = run(0, Bn)
    for b in (0, Bn - 1):
        assert torch.equal(run(b, b + 1)[0], y[b]), b
    f = {k: W.to_f64(v) for k, v in t.items()}
    ref = O.block_attention(f["x"][:2], f["wq"], f["wk"], f["wv"], f["wo"], f["k_cache"][:2], f["v_cache"][:2], Hq, G)
    d = y[:2].float().cpu().numpy().astype(np.float64) - ref
    assert np.sqrt((d ** 2).sum() / (ref ** 2).sum()) <= H.BF16_REL_L2
