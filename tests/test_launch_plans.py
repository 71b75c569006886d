"""The rules that choose a launch's form, asked on the host (no GPU): the tile of the attention projections
at the sizes where its rule changes, and that the shapes of the GPU tests reach the forms they are there for."""
import pytest

from paper_2602_00879_amd import binding as B
from tests import test_gpu_attention_turn as turn
from tests import test_gpu_f32_forms as f32
from tests import test_gpu_operand_order as order
from tests import test_gpu_projection_tiles as tiles
from tests import test_gpu_router_tiles as router


def _plans(case, residual=0):
    Bn, N, D, Hq, G, dh, P = case
    shape = B.make_shape(Bn, N, D, 16, 128, 2, 4, "vanilla", "bf16", residual=residual)
    attn = B.make_attn_shape(Hq, G, dh, P, 0)
    return B.des_test_plan(shape, attn, 0), B.des_test_plan(shape, attn, 1)


@pytest.mark.parametrize("name", list(tiles.TILES))
def test_projection_tests_reach_their_tiles(name):
    case, qkv, out = tiles.TILES[name]
    assert _plans(case) == (qkv, out)


def test_residual_test_reaches_the_register_tile():
    case, qkv, out = tiles.REGISTERS_OUT
    assert _plans(case, 1) == (qkv, out)


def test_every_tile_has_a_test():
    """All that launch_linear can choose: five tiles, whole or cut (not the largest), and the register tile."""
    reached = {p for case, qkv, out in tiles.TILES.values() for p in (qkv, out)}
    sizes = [(4, 4), (4, 2), (2, 2), (2, 1), (1, 1)]
    assert reached == {(m, n, kw, 0) for m, n in sizes for kw in (1, 2) if (m, n, kw) != (4, 4, 2)} | {(4, 4, 1, 1)}


# (rows, hidden, query heads, key/value heads, head width, launch): tile.  Compute units filled by 128 x 128
# tiles: one, two, three, four and nine per unit, one whose last round is not full, and the longest reduction.
RULE = [
    ((1024, 4096, 32, 8, 128, 1), (4, 4, 1, 1)),     # one per unit
    ((2048, 2048, 32, 8, 128, 1), (4, 4, 1, 1)),
    ((3072, 2048, 32, 4, 128, 1), (4, 4, 1, 0)),     # two
    ((1760, 2048, 16, 16, 128, 0), (4, 4, 1, 1)),    # three
    ((2048, 5120, 40, 8, 128, 0), (4, 4, 1, 0)),     # four
    ((2048, 2048, 128, 8, 128, 0), (4, 4, 1, 1)),    # nine
    ((1280, 5120, 40, 8, 128, 0), (4, 4, 1, 1)),     # three again
    ((4096, 2048, 128, 8, 128, 1), (4, 4, 1, 1)),    # two, reduction of 16384
    ((2304, 512, 8, 1, 64, 1), (2, 1, 2, 0)),        # two groups of 64 x 64 would take turns on a unit
    ((32, 2048, 32, 4, 128, 0), (0, 0, 0, 0)),       # a kernel of its own
]


@pytest.mark.parametrize("case,tile", RULE)
def test_rule_of_the_projection_tile(case, tile):
    T, D, Hq, G, dh, launch = case
    n = next(n for n in (32, 1) if T % n == 0)
    assert _plans((T // n, n, D, Hq, G, dh, 0))[launch] == tile


def test_plan_is_refused_where_the_call_is():
    shape = B.make_shape(1, 33, 100, 16, 128, 2, 4, "vanilla", "bf16")
    with pytest.raises(B.DesError):
        B.des_test_plan(shape, B.make_attn_shape(4, 2, 32, 0, 0), 0)
    with pytest.raises(B.DesError):
        B.des_test_plan(B.make_shape(1, 33, 128, 16, 128, 2, 4, "vanilla", "bf16"), None, 0)


@pytest.mark.parametrize("M,D,T,part", router.ROUTER)
def test_router_test_compares_four_tiles_with_one(M, D, T, part):
    def form(n):
        return B.des_test_plan(B.make_shape(1, n, D, M, 32, 1, M, "vanilla", "bf16"), None, 2)
    assert form(T) == (2, 2, 0, 0)
    assert {form(min(part, T - t)) for t in range(0, T, part)} == {(1, 1, 0, 0)}


# (experts, width): the fewest tokens of the launch with four tiles per workgroup
@pytest.mark.parametrize("M,D,least", [(128, 1024, 513), (256, 768, 257), (128, 2048, 577), (64, 1280, 1153),
                                       (256, 2048, 513), (192, 2048, 561), (128, 3072, 513), (24, 4096, 2049),
                                       (256, 3072, 513), (320, 1536, 401), (128, 256, 513), (128, 224, 1009)])
def test_rule_of_the_router_tiles(M, D, least):
    def form(n):
        return B.des_test_plan(B.make_shape(1, n, D, M, 32, 1, M, "vanilla", "bf16"), None, 2)
    assert form(least - 1) == (1, 1, 0, 0) and form(least) == (2, 2, 0, 0)


def _core(Bn, N, D, Hq, G, dh, P):
    """(parts, tiles, workgroups per head, turned), (LDS bytes, of the values among them) of the attention core."""
    shape, attn = B.make_shape(Bn, N, D, 16, 128, 2, 4, "vanilla", "bf16"), B.make_attn_shape(Hq, G, dh, P, 0)
    return B.des_test_plan(shape, attn, 3), B.des_test_plan(shape, attn, 4)[:2]


@pytest.mark.parametrize("Bn,N,G,P", list(turn.TURNED))
def test_turn_test_compares_both_orders(Bn, N, G, P):
    (parts, tiles, _, turned), (lds, values) = _core(Bn, N, 384, 9, G, 128, P)
    assert (parts, tiles) == turn.TURNED[Bn, N, G, P] and turned == 1
    assert _core(1, N, 384, 9, G, 128, P)[0][3] == 0
    ring = 512 + 256 * tiles + 2048 * tiles * -(-((P + N + 31) // 32) // parts)
    assert lds - values == max(ring, 512 + 256 * tiles + 1024 * max(4, parts * tiles))
    assert (lds - values > ring) == (parts == 8)


@pytest.mark.parametrize("dh", [32, 64, 96, 104, 120])
def test_only_heads_of_128_are_turned(dh):
    """Others reserve no LDS for it: 160 tokens, heads of 64 over 570 positions, two workgroups per compute unit."""
    for Bn, N, P in ((10, 16, 554), (8, 32, 464), (16, 32, 368), (1, 128, 440)):
        (parts, tiles, _, turned), (lds, values) = _core(Bn, N, 2048, 32, 4, dh, P)
        assert parts > 1 and turned == 0
        assert lds - values == 512 + 256 * tiles + 2048 * tiles * -(-((P + N + 31) // 32) // parts)
        if (dh, Bn) == (64, 10):
            assert parts == 8 and 2 * lds <= 160 * 1024


@pytest.fixture
def routing_form():
    """Form of a layer's routing as on a device with so many compute units."""
    def form(case, mode, units=256, dtype="bf16"):
        Bn, N, D, M, F, Fs, K, C = case
        B.des_test_compute_units(units)
        return B.des_test_plan(B.make_shape(Bn, N, D, M, F, K, C, mode, dtype, ffn_shared=Fs), None, 5)
    return form


def test_operand_order_test_has_blocks_that_are_copied(routing_form):
    for case in order.SHORT:
        for mode in ("vote", "vanilla"):
            assert routing_form(case, mode)[2] == (mode in order.COPIED.get(case, ())), (case, mode)


def test_routing_form_follows_the_number_of_compute_units(routing_form):
    """Two expert tiles of 17 tokens make four workgroups, the election one more."""
    case = (1, 17, 2080, 20, 32, 32, 2, 4)
    assert routing_form(case, "vote") == (1, 1, 1, 1)
    assert routing_form(case, "seq", 5) == (1, 1, 1, 1)
    assert routing_form(case, "vote", 4) == routing_form(case, "vote", 0) == (0, 0, 0, 1)
    assert routing_form(case, "vanilla") == (1, 0, 0, 1)
    assert routing_form((3, 9, 2048, 20, 32, 0, 2, 4), "vote") == (1, 0, 1, 1)
    assert routing_form((3, 9, 2080, 20, 32, 0, 2, 4), "vote") == (1, 0, 0, 1)
    assert routing_form((3, 9, 992, 20, 32, 0, 2, 4), "vote") == (1, 0, 0, 1)
    assert routing_form((1, 4, 1024, 20, 32, 0, 2, 4), "vote") == (1, 1, 0, 1)
    assert routing_form((1, 17, 1024, 20, 32, 0, 2, 4), "vote", dtype="f32") == (1, 0, 0, 1)


def _f32(case, mode, dtype="f32"):
    Bn, N, D, M, F, Fs, K, C = case
    return B.des_test_plan(B.make_shape(Bn, N, D, M, F, K, C, mode, dtype, ffn_shared=Fs), None, 6)


def test_f32_test_reaches_its_forms():
    for case, forms in f32.FORMS.items():
        for mode, form in forms.items():
            assert _f32(case, mode) == (*form, 0), (case, mode)


@pytest.mark.parametrize("D,F,M,C,K,least", [(2048, 768, 128, 32, 8, 128), (2048, 768, 64, 40, 8, 32),
                                             (4096, 1024, 16, 4, 4, 32), (1024, 512, 64, 64, 8, 4097)])
def test_rule_of_the_f32_pairs_order(D, F, M, C, K, least):
    """Fewest tokens whose pairs gate/up takes in the order of the experts (none of a small expert's)."""
    assert _f32((1, least - 1, D, M, F, 0, K, C), "vote")[0] == 0
    assert least > 4096 or _f32((1, least, D, M, F, 0, K, C), "vote")[0] == 1


def test_f32_down_fills_the_chip_with_one_token():
    assert _f32((1, 1, 2048, 128, 768, 0, 8, 32), "vote")[1:3] == (4, 512)
    assert _f32((1, 1, 2048, 128, 768, 0, 8, 32), "vote", "bf16") == (0, 0, 0, 0)
