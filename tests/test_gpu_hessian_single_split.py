"""Hessian calls whose tokens stay in one split: tiles (whole or in halves) are added to H without partial tiles."""
import pytest
import torch

import paper_2601_19675_amd as ptq

pytestmark = pytest.mark.gpu


# halves of tiles with the smallest width, a last tile of 8 and of 136 channels, an odd and an even number of tiles, tokens
# around the 32 of a stage and the ring of four; whole tiles (5640 = 22 tiles + 8 channels); three calls in a row
@pytest.mark.parametrize("n,chunks", [(2048, (1,)), (2056, (31, 33)), (2184, (129, 96, 1)), (2304, (700,)), (4096, (64, 160)),
                                      (5640, (65, 32)), (6144, (130,))])
def test_single_split_adds_the_gram_matrix_to_the_upper_triangle(n, chunks):
    g = torch.Generator().manual_seed(n)
    t = sum(chunks)
    X = (torch.randn((t, n), generator=g) * torch.exp(torch.randn(n, generator=g))).to(torch.bfloat16)
    wide = torch.full((n, n + 3), 0.5, dtype=torch.float64, device="cuda")   # a leading dimension of its own
    H = wide[:, :n]
    Xd, a = X.cuda(), 0
    for c in chunks:
        ptq.ptq_hessian_accumulate(H, Xd[a:a + c])
        a += c
    torch.cuda.synchronize()
    x = X.double()
    want, mag = x.T @ x, x.abs().T @ x.abs()
    got = wide.cpu()
    assert (got[:, n:] == 0.5).all() and (torch.tril(got[:, :n], -1) == torch.tril(torch.full((n, n), 0.5), -1)).all()
    # float32 sums of exact products, at worst one after the other
    err = (torch.triu(got[:, :n] - 0.5) - torch.triu(want)).abs()
    bound = t * 2.0 ** -24 * mag + 1e-12 * mag.max()
    assert (err <= bound).all(), float((err / bound).max())
