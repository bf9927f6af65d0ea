"""The stored layer applied to tokens (the float16 matrix-core product of two pieces per activation, and row by row for a few) at
the edges of its tiles, against the dequantized product in float64."""
import pytest
import torch

import paper_2601_19675_amd as ptq

pytestmark = pytest.mark.gpu


def _codes(packed, n, bits):
    words = packed.cpu().long() & 0xFFFFFFFF          # n / 32 x m x bits
    out = torch.empty((n, packed.shape[1]), dtype=torch.float64)
    for j in range(32):
        w, sh = (j * bits) // 32, (j * bits) % 32
        v = words[:, :, w] >> sh
        if sh + bits > 32:
            v = v | (words[:, :, w + 1] << (32 - sh))
        out[j::32] = (v & ((1 << bits) - 1)).double()
    return out


def _random_layer(seed, bits, tokens, m, n, group, r, dtype):
    g = torch.Generator().manual_seed(seed)
    packed = torch.randint(-2**31, 2**31, (n // 32, m, bits), generator=g, dtype=torch.int64).to(torch.int32)
    scales = 0.002 + 0.05 * torch.rand((n // group, m), generator=g)
    zeros = torch.randint(0, 2**bits, (n // group, m), generator=g).to(torch.uint8)
    perm = torch.randperm(n, generator=g).to(torch.int32)
    X = torch.randn((tokens, n), generator=g).to(dtype)
    U = torch.randint(0, 0x7f, (r, m), generator=g).to(torch.uint8) ^ (torch.randint(0, 2, (r, m), generator=g) * 128).to(torch.uint8)
    V = torch.randint(0, 0x40, (r, n), generator=g).to(torch.uint8)
    sigma = (torch.rand(r, generator=g) * 0.1).to(torch.float16)
    s = torch.exp(torch.randn(n, generator=g, dtype=torch.float64))
    return packed, scales, zeros, perm, X, U, V, sigma, s


def _basis(n, dtype):
    """b_I and b_H: bfloat16 activations are rotated, as they would fit one float16 piece; the others are not."""
    if dtype != torch.bfloat16:
        return n, 16
    b_H = min(256, n & -n)
    return (b_H if n > b_H else 0), b_H


def _turned(Xt, b_I, b_H):
    h = torch.ones((1, 1), dtype=torch.float64)
    while h.shape[0] < b_H:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    tail = Xt[:, b_I:]
    return torch.cat([Xt[:, :b_I], (tail.reshape(-1, b_H) @ h / b_H ** 0.5).reshape(tail.shape)], 1)


def _apply(layer, bits, group):
    packed, scales, zeros, perm, X, U, V, sigma, s = layer
    n, r, m = X.shape[1], U.shape[0], scales.shape[1]
    d = lambda t: t.cuda()  # noqa: E731
    low = (d(U), d(V), d(sigma), d(s)) if r else (None,) * 4
    wide = torch.full((X.shape[0], m + 3), float("nan"), device="cuda")   # an output with a leading dimension of its own
    ptq.ptq_lopro_linear_forward(d(X), d(packed), bits, d(scales), d(zeros), group, d(perm), *_basis(n, X.dtype), *low, wide[:, :m])
    torch.cuda.synchronize()
    assert torch.isnan(wide[:, m:]).all()
    return wide[:, :m].cpu().double()


def _reference(layer, bits, group, pieces=lambda Xt: Xt):
    """The dequantized product in float64 and, entry by entry, the sum of the terms' magnitudes and the root of the sum of their
    squares (the size that the entry would have with random signs).  `pieces`: what is made of X~ before it is multiplied."""
    packed, scales, zeros, perm, X, U, V, sigma, s = layer
    n, r = X.shape[1], U.shape[0]
    rep = lambda g: g.double().repeat_interleave(group, 0)  # noqa: E731
    X64, codes = X.double(), _codes(packed, n, bits)
    Wt = rep(scales) * (codes - rep(zeros))
    Xt = _turned(X64[:, perm.long()], *_basis(n, X.dtype))
    want, mag, square = pieces(Xt) @ Wt, Xt.abs() @ Wt.abs(), Xt.square() @ Wt.square()
    if X.shape[0] <= 4:   # the few-token product sums code x and zero x separately
        both = [rep(scales) * codes, rep(scales) * rep(zeros)]
        mag, square = Xt.abs() @ (both[0] + both[1]), Xt.square() @ (both[0].square() + both[1].square())
    if r:
        u, v, sg = U.view(torch.float8_e4m3fn).double(), V.view(torch.float8_e4m3fn).double(), sigma.double()
        want = want + (((X64 / s) @ v.T) * sg) @ u
        mag = mag + (((X64 / s).abs() @ v.abs().T) * sg) @ u.abs()
        square = square + (((X64 / s).square() @ v.square().T) * sg.square()) @ u.square()
    return want, mag, square.sqrt()


def _check(got, layer, bits, group):
    """Against the dequantized product in float64."""
    X, r = layer[4], layer[5].shape[0]
    n = X.shape[1]
    want, mag, size = _reference(layer, bits, group)
    err = (got - want).abs()
    # X~ is off by 2^-23 of an entry (2^-47 of the token's largest is far less here); every sum of float32 rounds once: two
    # products a column, three a rank, one per group and per split, one after the other at worst
    bound = (2 * n + 3 * r + 2 * (n // group) + n // 256 + 10) * 2.0 ** -24
    assert (err <= bound * mag + 1e-30).all(), float((err / (bound * mag + 1e-30)).max())
    # and as the roundings fall at random: 1.5e-7 is the largest measured over many entries (2e-7 here), a few entries alone may
    # be off by four standard deviations.  One float16 piece without the other is off by 1e-4.
    off = (err / size)[size > 0]
    assert float(off.square().mean().sqrt()) <= 2e-7 * (1 + 4 / off.numel() ** 0.5), float(off.square().mean().sqrt())


# one chunk of 32 columns, an odd number of them, more than a split holds; groups of one chunk and of all; the
# last row / token alone in its tile; ranks over one round of 32; few rows (the columns are split) and many
TILES = [
    (4, 8, 1, 32, 32, 0, torch.float32), (2, 32, 255, 96, 96, 5, torch.bfloat16), (3, 33, 257, 608, 32, 16, torch.float32),
    (8, 64, 300, 1056, 352, 33, torch.bfloat16), (4, 65, 129, 2048, 128, 16, torch.float64), (3, 130, 513, 4128, 4128, 2, torch.float32),
    (8, 1025, 70, 288, 32, 1, torch.bfloat16), (3, 5, 300, 4096, 128, 4, torch.float32)]


@pytest.mark.parametrize("bits,tokens,m,n,group,r,dtype", TILES)
def test_forward_tiles_match_the_dequantized_product(bits, tokens, m, n, group, r, dtype):
    layer = _random_layer(1000 * bits + tokens, bits, tokens, m, n, group, r, dtype)
    _check(_apply(layer, bits, group), layer, bits, group)


def _misaligned(t):
    """The same values on the GPU, one element past an aligned address and with a leading dimension of their own."""
    if t.dim() == 1:
        out = torch.empty(t.shape[0] + 1, dtype=t.dtype, device="cuda")[1:]
    else:
        out = torch.empty((t.shape[0], t.shape[1] + 3), dtype=t.dtype, device="cuda")[:, 1:1 + t.shape[1]]
    return out.copy_(t)


# rows staged by one workgroup and by several, ranks around the 4 and 16 of a workgroup, tokens around the coefficients' change of
# form at 192, each storage type in either form with wide loads and element by element
COEFFICIENTS = [(1, 4128, 1, torch.bfloat16), (2, 32, 5, torch.float32), (7, 2080, 4, torch.float64), (31, 544, 17, torch.bfloat16),
                (33, 2048, 16, torch.float32), (64, 96, 19, torch.float64), (191, 1056, 16, torch.bfloat16), (193, 2080, 17, torch.float32),
                (192, 544, 16, torch.float64), (200, 2112, 33, torch.bfloat16)]


@pytest.mark.parametrize("tokens,n,r,dtype", COEFFICIENTS)
@pytest.mark.parametrize("aligned", [True, False])
def test_activations_and_coefficients_at_the_edges_of_their_forms(tokens, n, r, dtype, aligned):
    m, bits, group = 70, 4, 32
    layer = _random_layer(tokens + n, bits, tokens, m, n, group, r, dtype)
    packed, scales, zeros, perm, X, U, V, sigma, s = layer
    d = lambda t: t.cuda()  # noqa: E731
    Xd, Vd, sd = d(X), d(V), d(s)
    if not aligned:
        Xd, sd = _misaligned(X), _misaligned(s)
        Vd = torch.empty(r * n + 1, dtype=torch.uint8, device="cuda")[1:].view(r, n).copy_(V)
    O = torch.full((tokens, m), float("nan"), device="cuda")
    ptq.ptq_lopro_linear_forward(Xd, d(packed), bits, d(scales), d(zeros), group, d(perm), *_basis(n, dtype), d(U), Vd, d(sigma), sd, O)
    torch.cuda.synchronize()
    _check(O.cpu().double(), layer, bits, group)


# row by row: the last row alone, eight and sixteen rows a workgroup, one chunk, a second batch of a lane's chunks, columns
# staged in two pieces (two tokens beyond 18432 columns), more ranks than slices, and the token counts around the change of form
@pytest.mark.parametrize("bits,tokens,m,n,group,r", [(2, 1, 1, 32, 32, 0), (3, 1, 2049, 1056, 96, 16), (4, 2, 4100, 320, 64, 3),
                                                     (8, 3, 17, 5440, 32, 40), (4, 4, 33, 4096, 4096, 5), (3, 4, 33, 4128, 32, 5),
                                                     (8, 2, 9, 18496, 32, 1)])
def test_forward_rows_match_the_dequantized_product(bits, tokens, m, n, group, r):
    layer = _random_layer(77 * bits + tokens, bits, tokens, m, n, group, r, torch.float32)
    _check(_apply(layer, bits, group), layer, bits, group)


# a coefficient beyond float32: its products with U are infinite (NaN with a zero of U), whatever form the product takes
@pytest.mark.parametrize("bits,tokens,m,n,r", [(4, 1, 40, 96, 2), (4, 4, 40, 4096, 3), (3, 5, 300, 608, 1), (8, 33, 70, 288, 35), (2, 64, 4100, 512, 2),
                                               (4, 1100, 4352, 64, 33)])
def test_an_infinite_coefficient_stays_infinite(bits, tokens, m, n, r):
    layer = list(_random_layer(31 * bits + tokens, bits, tokens, m, n, 32, r, torch.float32))
    packed, scales, zeros, perm, X, U, V, sigma, s = layer
    U[:, ::7], U[:, 1::7] = 0, 0x80                       # zeros of either sign
    s.clamp_(min=0.1)
    s[3], X[:, 3] = 1e-20, 0.0
    hit = torch.arange(tokens) % 3 == 0
    X[hit, 3] = torch.where(torch.arange(tokens)[hit] % 2 == 0, 1e30, -1e30)
    last = torch.arange(r) == r - 1
    V[:, 3] = torch.where(last, 0x38, 0).to(torch.uint8)   # 1 or 0: the other coefficients stay finite
    sigma.fill_(1.0)
    d = lambda t: t.cuda()  # noqa: E731
    O = torch.full((tokens, m), float("nan"), device="cuda")
    ptq.ptq_lopro_linear_forward(d(X), d(packed), bits, d(scales), d(zeros), 32, d(perm), n, 16, d(U), d(V), d(sigma), d(s), O)
    torch.cuda.synchronize()
    got = O.cpu()
    u, v = U.view(torch.float8_e4m3fn).float(), V.view(torch.float8_e4m3fn).double()
    y = ((X.double() / s) @ v.T).float()
    assert torch.equal(torch.isinf(y), hit[:, None] & last[None, :])
    low = (y[:, :, None] * u[None]).sum(1)                # infinite or NaN where it is decided by infinite coefficients
    assert torch.equal(torch.isnan(got), torch.isnan(low)) and torch.isnan(low).any()
    assert torch.equal(torch.isinf(got), torch.isinf(low)) and torch.isinf(low).any()
    assert torch.equal(got[torch.isinf(low)], low[torch.isinf(low)]) and torch.isfinite(got[~hit]).all()


# x / s, not x times a rounded 1 / s: a scale whose reciprocal is past the float64 range, under an activation of zero and
# under one of its own size
@pytest.mark.parametrize("tokens,r", [(1, 3), (33, 16), (200, 16)])
def test_the_smallest_scales_divide(tokens, r):
    m, n, bits = 40, 96, 4
    layer = list(_random_layer(5 + tokens, bits, tokens, m, n, 32, r, torch.float64))
    packed, scales, zeros, perm, X, U, V, sigma, s = layer
    s[3], X[:, 3] = 1e-310, 0.0
    s[40], X[:, 40] = 2e-309, 4e-309
    V[:, 40] = 0x38                                       # 1: the quotient counts
    d = lambda t: t.cuda()  # noqa: E731
    O = torch.full((tokens, m), float("nan"), device="cuda")
    ptq.ptq_lopro_linear_forward(d(X), d(packed), bits, d(scales), d(zeros), 32, d(perm), n, 16, d(U), d(V), d(sigma), d(s), O)
    torch.cuda.synchronize()
    _check(O.cpu().double(), layer, bits, 32)
