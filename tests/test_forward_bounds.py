"""The bounds of the stored layer's GPU tests notice a product that has lost the second float16 piece of its input, at every size
that these tests list; and pass one that has both (on the CPU)."""
import pytest
import torch

import test_gpu_forward_pieces as pieces
import test_gpu_forward_tiles as tiles

F32 = torch.float32


def _layers():
    for bits, tokens, m, n, group, r, dtype in tiles.TILES:
        yield bits, group, lambda a=(1000 * bits + tokens, bits, tokens, m, n, group, r, dtype): tiles._random_layer(*a)
    for tokens, n, r, dtype in tiles.COEFFICIENTS:
        if tokens > 4:   # fewer go row by row here, in float32
            yield 4, 32, lambda a=(tokens + n, 4, tokens, 70, n, 32, r, dtype): tiles._random_layer(*a)
    for bits, tokens, m, n, dtype in pieces.ANY_SIZE:
        yield bits, 32, lambda a=(bits, tokens, m, n, dtype): pieces._layer_of_any_size(*a)
    for bits, tokens, m, n, group, r, dtype in pieces.EDGES:
        yield bits, group, lambda a=(7 * bits + tokens, bits, tokens, m, n, group, r, dtype): tiles._random_layer(*a)
    for bits, tokens, m, n, r in pieces.LAST_RUNS:
        yield bits, 32, lambda a=(11 * bits + tokens, bits, tokens, m, n, 32, r, F32): tiles._random_layer(*a)


def _first_piece(Xt):
    unit = torch.exp2(14 - torch.floor(torch.log2(Xt.abs().amax(1, keepdim=True).clamp_min(1e-300))))
    return (Xt * unit).half().double() / unit


def _both_pieces(Xt):
    first = _first_piece(Xt)
    return first + _first_piece(Xt - first)


@pytest.mark.parametrize("bits,group,make", _layers())
def test_bounds_notice_a_lost_piece(bits, group, make):
    layer = make()
    tiles._check(tiles._reference(layer, bits, group, _both_pieces)[0], layer, bits, group)
    with pytest.raises(AssertionError):
        tiles._check(tiles._reference(layer, bits, group, _first_piece)[0], layer, bits, group)
