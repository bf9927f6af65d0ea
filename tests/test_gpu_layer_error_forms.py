"""The layer error in tiles of 256 x 128, at sizes that are no multiples of them, against both traces in float64."""
import pytest
import torch

import paper_2601_19675_amd as ptq

pytestmark = pytest.mark.gpu


# just enough tiles for the form, in each type and number of rows, a last row of tiles that is half there, rows of tiles past two
# groups of sixteen, columns past the last tile; just too few tiles, and seven rows of them
@pytest.mark.parametrize("m,n,dtype", [(3100, 3900, torch.bfloat16), (1409, 4100, torch.float32), (6144, 2050, torch.bfloat16),
                                       (11000, 1155, torch.bfloat16), (2048, 3072, torch.float32), (3072, 3968, torch.bfloat16),
                                       (2200, 6399, torch.bfloat16), (2304, 6200, torch.bfloat16), (600, 8190, torch.float32),
                                       (1700, 4100, torch.float32)])
def test_traces_of_the_wide_form(m, n, dtype):
    g = torch.Generator(device="cuda").manual_seed(m)
    W = (0.02 * torch.randn((m, n), generator=g, device="cuda")).to(dtype)
    Wq = torch.round(W.double() / 0.017) * 0.017
    scale = torch.exp(0.8 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64))
    X = torch.randn((n + 64, n), generator=g, device="cuda", dtype=torch.float64) * scale
    H = X.T @ X
    stored = torch.triu(H) + torch.tril(torch.full_like(H, float("nan")), -1)   # only the upper triangle is read
    out = torch.empty(3, dtype=torch.float64, device="cuda")
    ptq.ptq_layer_error(W, Wq, stored, out)
    torch.cuda.synchronize()
    D = W.double() - Wq
    num, den = float(((D @ H) * D).sum()), float(((W.double() @ H) * W.double()).sum())
    # every term is off by up to 2^-16 of itself, at random: a few 1e-7 of a trace of 1e7 terms (the other form's tests allow 4e-6)
    assert abs(float(out[1]) - num) <= 4e-6 * num and abs(float(out[2]) - den) <= 4e-6 * den
    assert abs(float(out[0]) - (num / den) ** 0.5) <= 1e-6 * (num / den) ** 0.5
