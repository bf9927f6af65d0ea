"""The column walk shares its block between waves: one walks, each of the others pushes errors onto one tile, sooner or later
by whether the tile is walked next or a group's grid is about to be taken.  Blocks of one tile to more tiles than
waves, a last block that is narrower, groups of one tile to the whole block, heights of one, two and three row tiles
per workgroup with ragged ends; every decision against the oracle, values, errors and row sums against what they imply."""
import numpy as np
import pytest
import torch

import paper_2601_19675_amd as ptq
from oracle import ptq_oracle as orc
from parity import compare_quantization

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,bits,group,block", [
    (5, 48, 4, 16, 16), (17, 80, 3, 16, 48), (16, 96, 2, 48, 48), (33, 208, 4, 16, 128), (31, 320, 3, 64, 128), (48, 256, 2, 128, 128),
    (20, 160, 8, 32, 64), (40, 320, 4, 64, 256), (24, 288, 3, 16, 144), (4700, 176, 4, 16, 128), (4610, 192, 2, 64, 128),
    (9300, 160, 3, 32, 128), (9217, 160, 4, 16, 160)])
def test_walk(m, n, bits, group, block):
    rng = np.random.default_rng(1000 * n + m)
    W = (0.02 * rng.standard_normal((m, n))).astype(np.float32)
    X = rng.standard_normal((3 * n, n)) @ (np.eye(n) + 0.8 / np.sqrt(n) * rng.standard_normal((n, n)))
    U = orc.inverse_cholesky_upper(orc.damp(X.T @ X, 0.01)[0])
    dead = np.zeros(n, dtype=bool)
    dead[[1, n - 2]] = True
    Wg, Ug = torch.from_numpy(W).cuda(), torch.from_numpy(np.ascontiguousarray(U)).cuda()
    codes = torch.full((m, n), 255, dtype=torch.uint8, device="cuda")
    scales = torch.full((m, n // group), -1.0, dtype=torch.float32, device="cuda")
    zeros = torch.full((m, n // group), 255, dtype=torch.uint8, device="cuda")
    Wq = torch.full((m, n), float("nan"), dtype=torch.float64, device="cuda")
    err2 = torch.full((m,), float("nan"), dtype=torch.float64, device="cuda")
    ptq.ptq_quantize_layer(Wg, Ug, torch.from_numpy(dead.astype(np.uint8)).cuda(), bits, group, block, codes, scales, zeros, Wq, err2)
    torch.cuda.synchronize()
    codes, scales, zeros, Wq, err2 = (x.cpu().numpy() for x in (codes, scales, zeros, Wq, err2))
    # rows are independent: the first and last ones and some between
    rows = np.unique(np.r_[0:min(m, 20), max(0, m - 20):m, rng.integers(0, m, 10)])
    W64 = W[rows].astype(np.float64)
    rep = compare_quantization(W64, U, bits, group, dead, codes[rows], scales[rows], zeros[rows])
    assert rep["unflagged"] == 0, rep["details"][:3]
    # the values are scale (code - zero), exact in float64 (24-bit by 9-bit)
    rep_g = np.repeat(scales.astype(np.float64), group, 1) * (codes.astype(np.float64) - np.repeat(zeros.astype(np.float64), group, 1))
    assert np.array_equal(Wq, rep_g)
    # (W - Wq) = E U: the row sums are those of the errors that the values imply.  The errors come back through U^-1; what
    # that rounds is at most n u of |D||U^-1|, taken twice for the sum of squares
    W0 = W64.copy()
    W0[:, dead] = 0.0
    D, inv = W0 - Wq[rows], np.linalg.inv(U)
    E = D @ inv
    slack = 4 * n * 2.0**-53 * (np.abs(D) @ (np.abs(inv) @ np.abs(U) @ np.abs(inv)))
    assert np.all(np.abs(err2[rows] - (E * E).sum(1)) <= (2 * np.abs(E) * slack + slack**2).sum(1) + 1e-300)
