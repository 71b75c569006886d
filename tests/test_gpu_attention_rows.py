"""The attention core with its values as rows in LDS (heads of 64 and 128): every form of it, windows that
end inside a step of 32 positions and that fill it, block and cache rows in one direct load.  Every token
against the CPU oracle, as for the other forms."""
import pytest

from tests import test_gpu_attention_core as core

pytestmark = pytest.mark.gpu

# (sequences, tokens, hidden, query heads, key/value heads, head width, cached positions)
ROWS = {
    "one_step_64": (1, 7, 128, 8, 2, 64, 3),
    "one_step_128": (1, 3, 128, 4, 2, 128, 29),
    "whole_97_full_workgroups": (64, 32, 128, 16, 4, 64, 65),
    "parts_of_one_step_more": (2, 9, 256, 4, 2, 64, 280),
    "wide_257_64": (33, 31, 128, 32, 8, 64, 226),
    "wide_512_128": (32, 32, 128, 32, 8, 128, 480),
    "twice_532_128": (32, 32, 128, 32, 8, 128, 500),
    "twice_1100_64": (1, 20, 128, 4, 1, 64, 1080),
}


@pytest.mark.parametrize("name", list(ROWS))
def test_values_as_rows(name, monkeypatch):
    monkeypatch.setitem(core.CASES, name, ROWS[name])
    core.test_attention_core(name)
