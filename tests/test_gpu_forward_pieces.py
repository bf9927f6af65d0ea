"""The stored layer applied to many tokens: the two float16 pieces of a token's rotated input, its power of two, and what the
launches share out, at the sizes where these change; against the dequantized product in float64."""
import pytest
import torch

import paper_2601_19675_amd as ptq
from test_gpu_forward_tiles import _apply, _check, _codes, _random_layer, _reference

pytestmark = pytest.mark.gpu


# tokens of very different sizes, one of zeros, one with an entry 2^20 times the others, which meets a zero weight in some rows,
# one of equal entries, which a rotation makes sqrt(b_H) times as large (b_H of even and odd powers)
ANY_SIZE = [(4, 40, 70, 544, torch.float32), (2, 7, 300, 4096, torch.bfloat16), (8, 65, 33, 96, torch.float64), (3, 6, 33, 1152, torch.bfloat16)]


def _layer_of_any_size(bits, tokens, m, n, dtype):
    layer = list(_random_layer(bits + n, bits, tokens, m, n, 32, 0, dtype))
    X = layer[4]
    for t in range(tokens):
        X[t] *= 2.0 ** ((t * 11) % 120 - 60)
    X[2] = 0.0
    X[3, 5] = X[3].abs().amax() * 2.0 ** 20
    X[4] = 255 / 128
    return layer


@pytest.mark.parametrize("bits,tokens,m,n,dtype", ANY_SIZE)
def test_tokens_of_any_size(bits, tokens, m, n, dtype):
    layer = _layer_of_any_size(bits, tokens, m, n, dtype)
    _check(_apply(layer, bits, 32), layer, bits, 32)


def _put_code(packed, bits, column, rows, code):
    """Sets the code of a column (position in the rotated basis, its bits in one word) in some rows."""
    word, shift = divmod(column % 32 * bits, 32)
    assert shift + bits <= 32
    w = packed[column // 32, rows, word].long() & 0xFFFFFFFF
    w = (w & ~(((1 << bits) - 1) << shift)) | (code.long() << shift)
    packed[column // 32, rows, word] = torch.where(w >= 2**31, w - 2**32, w).to(torch.int32)


def _zero_weight(layer, bits, group, column, rows):
    _put_code(layer[0], bits, column, rows, layer[2][column // group, rows])


def _rows_off(got, layer, bits, group, rows):
    """Largest error of a token's outputs in these rows, relative to the norm that they would have with random signs."""
    want, _, size = _reference(layer, bits, group)
    return float(((got - want)[:, rows].norm(dim=1) / size[:, rows].norm(dim=1)).max())


def _norm(rows):
    """Bound for the above: 1.5e-7 is the largest measured over many rows where all entries are of a size (2e-7 here); a few rows
    alone may be off by four standard deviations."""
    return 2e-7 * (1 + 4 / rows.numel() ** 0.5)


# an entry 2^20 times the others that meets a zero weight in every other row: there the others keep all their bits
@pytest.mark.parametrize("bits,tokens,m,n,dtype", [(4, 40, 70, 544, torch.float32), (2, 7, 300, 2048, torch.float32), (3, 70, 90, 1024, torch.float64),
                                                   (8, 65, 33, 96, torch.float64)])
def test_a_massive_entry_beside_a_zero_weight(bits, tokens, m, n, dtype):
    layer = list(_random_layer(3 * bits + n, bits, tokens, m, n, 32, 0, dtype))
    perm, X = layer[3:5]
    column, rows = 37, torch.arange(0, m, 2)
    _zero_weight(layer, bits, 32, column, rows)
    X[:, perm[column]] = X[:, perm[column]].sign() * 2.0 ** 20
    assert _rows_off(_apply(layer, bits, 32), layer, bits, 32, rows) <= _norm(rows)


# the same with an entry 2^34 times the others, or an ordinary one over entries 2^-34 times it: past what two pieces hold.  Tokens
# of one tile of either kind; columns in one part, two halves and several splits; a row that leaves no room in LDS behind it;
# several narrow tokens to a workgroup; a last run of tokens; every third token all ordinary
@pytest.mark.parametrize("bits,tokens,m,n,group,dtype", [
    (4, 40, 70, 544, 32, torch.float32), (2, 7, 300, 2048, 128, torch.bfloat16), (3, 70, 600, 1024, 1024, torch.float64), (8, 65, 33, 96, 96, torch.float32),
    (4, 3, 9, 20448, 32, torch.float64), (8, 1027, 40, 352, 32, torch.float32), (3, 4096, 20, 256, 64, torch.bfloat16), (2, 585, 2, 4096, 64, torch.float32)])
def test_tokens_past_the_pieces(bits, tokens, m, n, group, dtype):
    layer = list(_random_layer(5 * bits + n, bits, tokens, m, n, group, 0, dtype))
    perm, X = layer[3:5]
    columns, rows = (20, n - 7), torch.arange(0, m, 2)
    kind = torch.arange(tokens) % 3
    for column in columns:
        _zero_weight(layer, bits, group, column, rows)
        X[kind == 1, perm[column]] = X[kind == 1, perm[column]].sign() * 2.0 ** 34
    X[kind == 2] *= 2.0 ** -34
    X[kind == 2, perm[columns[0]]] = 1.0
    got = _apply(layer, bits, group)
    assert _rows_off(got, layer, bits, group, rows) <= _norm(rows)
    assert _rows_off(got, layer, bits, group, torch.arange(m)) <= _norm(torch.arange(m))


# some entries of a row 2^-40 times the others are left to the pieces
@pytest.mark.parametrize("every", [300, 5])
def test_some_small_entries(every):
    layer = list(_random_layer(77, 4, 40, 70, 2048, 32, 0, torch.float32))
    layer[4][:, ::every] *= 2.0 ** -40
    assert _rows_off(_apply(layer, 4, 32), layer, 4, 32, torch.arange(70)) <= _norm(torch.arange(70))


# tokens of numbers below float32's normal range
@pytest.mark.parametrize("bits,tokens,dtype", [(4, 40, torch.float32), (3, 70, torch.bfloat16), (2, 6, torch.float64)])
def test_subnormal_tokens(bits, tokens, dtype):
    layer = list(_random_layer(13, bits, tokens, 70, 544, 32, 0, torch.float32))
    layer[4] = (layer[4].double() * 2.0 ** (-131 if dtype != torch.float64 else -140)).to(dtype)
    layer[1] *= 2.0 ** 60
    if dtype == torch.float64:
        layer[4][1::2] *= 2.0 ** 200
    assert _rows_off(_apply(layer, bits, 32), layer, bits, 32, torch.arange(70)) <= _norm(torch.arange(70))


# group scales far from those of a grid, with tokens whose size brings the outputs back: some rows, or some groups of all
@pytest.mark.parametrize("power", [120, 90, -90, -140])
@pytest.mark.parametrize("bits,tokens,m,n,group,dtype", [(4, 40, 70, 544, 32, torch.float32), (2, 7, 300, 2048, 128, torch.bfloat16),
                                                         (3, 70, 600, 1024, 1024, torch.float64), (8, 193, 260, 96, 32, torch.float32)])
def test_extreme_scales(bits, tokens, m, n, group, dtype, power):
    layer = list(_random_layer(7 * bits + n, bits, tokens, m, n, group, 0, dtype))
    scales, zeros, perm, X = layer[1:5]
    X *= 2.0 ** (-power * 0.6)
    scales[:, ::3] *= 2.0 ** power
    if n // group > 3:
        scales[1::2] *= 2.0 ** power if power < 0 else 1.0
    X[1::5, perm[20]] *= 2.0 ** 30   # tokens of either kind
    rows = torch.arange(0, m, 3)
    assert _rows_off(_apply(layer, bits, group), layer, bits, group, rows) <= _norm(rows)


# scales of zero are ordinary
def test_scales_of_zero():
    layer = list(_random_layer(3, 4, 40, 70, 544, 32, 0, torch.float32))
    layer[1][::2, ::2] = 0.0
    layer[1][:, 5] = 0.0
    got = _apply(layer, 4, 32)
    assert (got[:, 5] == 0).all()
    rows = torch.arange(70)[torch.arange(70) != 5]
    assert _rows_off(got, layer, 4, 32, rows) <= _norm(rows)


# an infinity or a NaN stays in its own token
def test_tokens_that_are_not_finite():
    layer = list(_random_layer(9, 4, 37, 130, 320, 64, 3, torch.float32))
    X = layer[4]
    X[4, 17], X[20, 300] = float("inf"), float("nan")
    got = _apply(layer, 4, 64)
    assert torch.isnan(got[4]).all() and torch.isnan(got[20]).all()
    X[4, 17] = X[20, 300] = 0.0
    got[[4, 20]] = _apply(layer, 4, 64)[[4, 20]]
    _check(got, layer, 4, 64)


# a row that leaves no room in LDS behind it; tokens whose exponents the workspace of a tiny layer cannot hold at once (two whole
# runs and one token); coefficients by several workgroups, with ranks and tokens past their tiles, and without room for that;
# two, four and eight narrow tokens to a workgroup, the last run of them whole or not; parts of 1, 2 and 3 chunks past a multiple of
# four
EDGES = [
    (4, 2, 9, 20448, 32, 0, torch.float64), (3, 193, 1, 32, 32, 2, torch.float32), (4, 200, 300, 2048, 128, 17, torch.bfloat16),
    (2, 223, 64, 4096, 64, 16, torch.float32), (8, 192, 8, 4096, 4096, 40, torch.bfloat16), (4, 1027, 40, 352, 32, 5, torch.float32),
    (8, 70, 20, 1120, 32, 0, torch.bfloat16), (3, 5, 257, 864, 96, 16, torch.bfloat16), (2, 33, 4100, 1184, 32, 1, torch.float32),
    (4, 2050, 33, 288, 32, 3, torch.float32), (2, 4090, 20, 256, 64, 16, torch.bfloat16), (8, 4096, 9, 96, 32, 0, torch.float64)]


@pytest.mark.parametrize("bits,tokens,m,n,group,r,dtype", EDGES)
def test_edges_of_what_the_launches_share_out(bits, tokens, m, n, group, r, dtype):
    layer = _random_layer(7 * bits + tokens, bits, tokens, m, n, group, r, dtype)
    _check(_apply(layer, bits, group), layer, bits, group)


# tokens in runs, the last of which splits its columns over several workgroups
LAST_RUNS = [(4, 133, 1, 512, 0), (3, 585, 1, 4096, 16), (8, 395, 3, 544, 2)]


@pytest.mark.parametrize("bits,tokens,m,n,r", LAST_RUNS)
def test_a_last_run_that_splits(bits, tokens, m, n, r):
    layer = _random_layer(11 * bits + tokens, bits, tokens, m, n, 32, r, torch.float32)
    _check(_apply(layer, bits, 32), layer, bits, 32)


# quotients x / s whose reciprocal alone would not do: s beyond 2^500 and below 2^-500, beside ordinary ones
def test_coefficients_of_extreme_scales():
    layer = list(_random_layer(5, 4, 200, 64, 1024, 64, 16, torch.float32))
    s = layer[8]
    s[7], s[8], s[9] = 1e-310, 2.0 ** 600, 2.0 ** -600
    layer[4][:, 7] = layer[4][:, 9] = 0.0
    _check(_apply(layer, 4, 64), layer, 4, 64)
