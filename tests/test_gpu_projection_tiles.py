"""Every tile that the attention projections of more than 32 rows choose from (64 x 64 down to 32 x 32
rows and up to 128 x 128, the reduction whole or in two halves), with rows and columns that do not fill
it and the shortest reduction.  Every token against the CPU oracle, as for the attention core."""
import pytest

from tests import test_gpu_attention_core as core

pytestmark = pytest.mark.gpu

# (sequences, tokens, hidden, query heads, key/value heads, head width, cached positions); in
# brackets the tiles of q/k/v and output in units of 32 rows (weights, tokens), * = in halves
TILES = {
    "two_chunks": (1, 33, 128, 4, 2, 32, 0),             # (1, 1), (1, 1)
    "cut_small": (1, 45, 512, 8, 2, 64, 5),              # (1, 1)*, (1, 1)*
    "cut_64_x_32": (6, 77, 512, 8, 2, 64, 0),            # (2, 1)*, (2, 1)*
    "64_x_32": (3, 50, 1152, 40, 4, 128, 0),             # (2, 1), (1, 1)*
    "cut_64_x_64": (8, 90, 512, 8, 2, 64, 0),            # (2, 2)*
    "64_x_64": (10, 103, 256, 8, 2, 32, 0),              # (2, 2)
    "cut_128_x_64": (10, 103, 512, 8, 2, 64, 3),         # (4, 2)*, (2, 2)*
    "128_x_64": (2, 65, 1152, 72, 8, 128, 0),            # (4, 2)
    "128_x_128": (6, 77, 1152, 72, 8, 128, 0),           # (4, 4)
}


@pytest.mark.parametrize("name", list(TILES))
def test_projection_tiles(name, monkeypatch):
    monkeypatch.setitem(core.CASES, name, TILES[name])
    core.test_attention_core(name)
