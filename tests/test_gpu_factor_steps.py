"""The factor of up to a few thousand columns goes 128 columns at a time: a leaf beside the update with the block column
before it, the panel, the next leaf's block.  Sizes at the edges of the leaf, of the panel's strips of 32 and of the
update's tiles, one to many block columns, an output with a longer row; a width just past the largest block, whose
halves go this way under one recursion; and rows too long for the steps."""
import numpy as np
import pytest
import torch

import paper_2601_19675_amd as ptq
from paper_2601_19675_amd import binding
from oracle import ptq_oracle as orc

pytestmark = pytest.mark.gpu
DAMP = 0.01


def _case(n, seed):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n + 32, n)) * np.exp(0.5 * rng.standard_normal(n))
    X += 0.5 * rng.standard_normal((n + 32, 1))   # correlated channels
    return X.T @ X


def _gpu(H, extra, fill):
    n = H.shape[0]
    Hd = torch.from_numpy(np.triu(H)).cuda()
    U = torch.full((n, n + extra), float("nan"), dtype=torch.float64, device="cuda")[:, :n]
    dead = torch.zeros(n, dtype=torch.uint8, device="cuda")
    info = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    ws = torch.empty(ptq.ptq_workspace_bytes(binding.OP_CHOLESKY_INV, 0, n), dtype=torch.uint8, device="cuda").fill_(fill)
    ptq.ptq_damped_cholesky_inv(Hd, DAMP, U, dead, info, ws)
    torch.cuda.synchronize()
    return U, info.cpu().tolist()


def _check(n, extra):
    H = _case(n, n)
    Hd, _ = orc.damp(H, DAMP)
    U, info = _gpu(H, extra, 0xFF)   # (an all-ones workspace reads as NaN)
    assert info == [0, 0]
    U = U.cpu().numpy()
    assert np.all(np.tril(U, -1) == 0.0)
    # Every step is a product or a subtraction of at most n terms in float64: to first order the computed L and X = L^-1 satisfy
    # |LL^T - G| <= (n + 1) u |L||L^T| and |XL - I| <= (n + 1) u |X||L| (u = 2^-53), so |U H_d U^T - I| is at most
    # 3 (n + 1) u |U||R||R^T||U^T| with H_d = R R^T; doubled for the products that this check itself makes.
    R = np.linalg.inv(orc.inverse_cholesky_upper(Hd))
    B = np.abs(U) @ np.abs(R)
    assert np.all(np.abs(U @ Hd @ U.T - np.eye(n)) <= 6 * (n + 1) * 2.0**-53 * (B @ B.T))


@pytest.mark.parametrize("n,extra", [(1, 0), (127, 0), (128, 0), (129, 0), (160, 1), (161, 0), (256, 0), (257, 3), (383, 0), (449, 0),
                                     (640, 0), (1000, 1), (1601, 0)])
def test_factor_in_steps(n, extra):
    _check(n, extra)


@pytest.mark.parametrize("n", [129, 300, 700])
def test_factor_of_long_rows(n):
    """Rows of U past 2^20 entries: the recursion down to 128 columns, nodes of 1 to 316 rows, ragged ones among them."""
    _check(n, (1 << 20) + 1 - n)


@pytest.mark.parametrize("n,ldu", [(140, (1 << 25) + 1), (4400, (1 << 20) + 1)])
def test_factor_of_rows_past_31_bits(n, ldu):
    """U of 37 GB: offsets across a tile's rows, and down the columns of a node, that 31 bits do not hold."""
    _check(n, ldu - n)


def test_factor_of_halves_in_steps():
    n = 5150
    H = _case(n, 5)
    Hd, _ = orc.damp(H, DAMP)
    U, info = _gpu(H, 2, 0)
    assert info == [0, 0]
    g = torch.Generator(device="cuda").manual_seed(3)
    V = torch.randn((n, 8), dtype=torch.float64, device="cuda", generator=g)
    back = U.T @ (U @ (torch.from_numpy(Hd).cuda() @ V))   # H_d^-1 H_d V
    # error of a solve through the factor: n u cond(H_d) at most (no eigenvalue is below the damping or above the norm)
    cond = float(np.linalg.norm(Hd)) / (DAMP * float(np.mean(np.diag(H))))
    assert float((back - V).norm() / V.norm()) <= n * 2.0**-53 * cond


def test_factor_in_steps_reports_the_first_bad_pivot():
    # the factor walks the reversed matrix: the first bad pivot is the largest index that fails
    n, bad = 700, 300
    H = np.eye(n) * 2.0
    H[bad, bad] = -5.0
    Hd = torch.from_numpy(H).cuda()
    U = torch.empty((n, n), dtype=torch.float64, device="cuda")
    dead = torch.zeros(n, dtype=torch.uint8, device="cuda")
    info = torch.zeros(2, dtype=torch.int32, device="cuda")
    ptq.ptq_damped_cholesky_inv(Hd, 0.0, U, dead, info)
    torch.cuda.synchronize()
    assert info.cpu().tolist()[1] == bad and info.cpu().tolist()[0] != 0
