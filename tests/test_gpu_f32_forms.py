"""The fp32 layer's two launches at their edges: choices in fours with a remainder, widths around the 256
elements that a wavefront takes at once, a shared expert of another width, unused choices (skipping),
one token and several sequences.  Every token against the CPU oracle."""
import pytest

from paper_2602_00879_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

# (sequences, tokens of each, D, M, F, Fs, K, C)
F32 = [(1, 1, 4, 3, 4, 0, 1, 2), (1, 7, 260, 12, 252, 8, 5, 9), (3, 11, 64, 9, 260, 516, 4, 6),
       (2, 40, 36, 40, 20, 0, 9, 24), (1, 32, 256, 16, 1028, 4, 3, 5)]


@pytest.mark.parametrize("case", F32, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("mode,skip", [("vote", 0.0), ("vanilla", 0.2)])
def test_f32_layer(case, mode, skip):
    Bn, N, D, M, F, Fs, K, C = case
    cfg = W.LayerConfig("f32_forms", "f32", Bn, N, D, M, F, Fs, K, C, 1.1, 83)
    layer = W.make_layer(cfg)
    dev = H.layer_to_device(layer)
    for residual in (0, 1):
        out = H.run_gpu(cfg, dev, mode, residual=residual, skip_beta=skip)
        H.check_against_oracle(cfg, layer, out, mode, residual=bool(residual), skip_beta=skip, label=f"{case} {mode}")
