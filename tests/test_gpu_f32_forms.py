"""The fp32 layer's two launches at their edges: choices in fours with a remainder, widths around the 256
elements that a wavefront takes at once, a shared expert of another width, unused choices (skipping),
one token and several sequences; large experts at both sides of the number of pairs from which gate/up takes
them in the order of the experts, one choice per token and more outputs than down has wavefronts.  Every token
against the CPU oracle.  (test_launch_plans.py holds the sizes to those forms.)"""
import pytest

from paper_2602_00879_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

# (sequences, tokens of each, D, M, F, Fs, K, C)
F32 = [(1, 1, 4, 3, 4, 0, 1, 2), (1, 7, 260, 12, 252, 8, 5, 9), (3, 11, 64, 9, 260, 516, 4, 6),
       (2, 40, 36, 40, 20, 0, 9, 24), (1, 32, 256, 16, 1028, 4, 3, 5)]
# ... and {mode: pairs in the order of the experts, choices at once, workgroups of down per token}
FORMS = {(1, 87, 1024, 8, 1024, 0, 3, 3): {"vote": (0, 1, 256), "vanilla": (1, 1, 256)},
         (1, 43, 1028, 4, 4084, 64, 3, 3): {"vote": (1, 1, 257), "vanilla": (1, 1, 257)},
         (1, 42, 1028, 4, 4084, 64, 3, 3): {"vote": (0, 4, 257), "vanilla": (0, 4, 257)},
         (1, 3, 4100, 4, 8, 0, 2, 3): {"vote": (0, 4, 1024), "vanilla": (0, 4, 1024)},
         (1, 70, 4100, 4, 8, 4, 1, 3): {"vote": (0, 1, 64), "vanilla": (0, 1, 64)}}
F32 += list(FORMS)


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
