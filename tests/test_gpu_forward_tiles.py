"""The stored layer applied to many tokens (the bfloat16 matrix-core product of three exact pieces per activation)
at the edges of its tiles, against the dequantized product in float64."""
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


# one chunk of 32 columns, an odd number of them, more than a split holds; groups of one chunk and of all; the
# last row / token alone in its tile; ranks over one round of 32; few rows (the columns are split) and many
@pytest.mark.parametrize("bits,tokens,m,n,group,r,dtype", [
    (4, 8, 1, 32, 32, 0, torch.float32), (2, 32, 255, 96, 96, 5, torch.bfloat16), (3, 33, 257, 608, 32, 16, torch.float32),
    (8, 64, 300, 1056, 352, 33, torch.bfloat16), (4, 65, 129, 2048, 128, 16, torch.float64), (3, 130, 513, 4128, 4128, 2, torch.float32),
    (8, 1025, 70, 288, 32, 1, torch.bfloat16)])
def test_forward_tiles_match_the_dequantized_product(bits, tokens, m, n, group, r, dtype):
    g = torch.Generator().manual_seed(1000 * bits + tokens)
    packed = torch.randint(-2**31, 2**31, (n // 32, m, bits), generator=g, dtype=torch.int64).to(torch.int32)
    scales = 0.002 + 0.05 * torch.rand((n // group, m), generator=g)
    zeros = torch.randint(0, 2**bits, (n // group, m), generator=g).to(torch.uint8)
    perm = torch.randperm(n, generator=g).to(torch.int32)
    X = torch.randn((tokens, n), generator=g).to(dtype)
    U = torch.randint(0, 0x7f, (r, m), generator=g).to(torch.uint8) ^ (torch.randint(0, 2, (r, m), generator=g) * 128).to(torch.uint8)
    V = torch.randint(0, 0x40, (r, n), generator=g).to(torch.uint8)
    sigma = (torch.rand(r, generator=g) * 0.1).to(torch.float16)
    s = torch.exp(torch.randn(n, generator=g, dtype=torch.float64))
    d = lambda t: t.cuda()  # noqa: E731
    low = (d(U), d(V), d(sigma), d(s)) if r else (None,) * 4
    wide = torch.full((tokens, m + 3), float("nan"), device="cuda")   # an output with a leading dimension of its own
    ptq.ptq_lopro_linear_forward(d(X), d(packed), bits, d(scales), d(zeros), group, d(perm), n, 16, *low, wide[:, :m])
    torch.cuda.synchronize()
    assert torch.isnan(wide[:, m:]).all()
    got = wide[:, :m].cpu().double()

    X64 = X.double()
    Wt = scales.double().repeat_interleave(group, 0) * (_codes(packed, n, bits) - zeros.double().repeat_interleave(group, 0))
    Xt = X64[:, perm.long()]
    want, mag = Xt @ Wt, Xt.abs() @ Wt.abs()
    if r:
        u, v = U.view(torch.float8_e4m3fn).double(), V.view(torch.float8_e4m3fn).double()
        y, y_mag = ((X64 / s) @ v.T) * sigma.double(), ((X64 / s).abs() @ v.abs().T) * sigma.double()
        want, mag = want + y @ u, mag + y_mag @ u.abs()
    # float32: X~, the coefficients and every product's pieces are exact or rounded once; the three products of a
    # column and the columns are added one after the other at worst, then a rounding per group and per split
    bound = (3 * (n + r) + 2 * (n // group) + n // 256 + 8) * 2.0 ** -24
    err = (got - want).abs()
    assert (err <= bound * mag + 1e-30).all(), float((err / (bound * mag + 1e-30)).max())
    # and as the roundings fall at random: their square root
    assert float(err.norm() / mag.norm()) <= 4 * bound ** 0.5 * 2.0 ** -12
