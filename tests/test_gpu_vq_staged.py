"""The vector walk of codebooks of more than 64 entries of 4 weights: the form that has its block of U in LDS (blocks of three to
eight tiles), the one for one or two tiles, the one for more than eight; last blocks that are narrower, ragged rows, dead columns."""
import numpy as np
import pytest
import torch

import paper_2601_19675_amd as ptq
from parity import compare_vq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,block,entries", [(3, 16, 16, 65), (17, 112, 48, 100), (16, 240, 112, 256), (33, 208, 128, 200),
                                               (20, 384, 128, 256), (18, 160, 256, 256),
                                               (19, 96, 32, 256), (35, 160, 128, 90), (9, 176, 96, 256)])
def test_staged_walk(m, n, block, entries):
    rng = np.random.default_rng(10 * n + entries)
    W = rng.normal(0, 0.02, (m, n))
    U = np.triu(rng.normal(0, 0.05, (n, n)), 1) + np.diag(np.exp(rng.normal(0, 0.5, n)))
    C = rng.normal(0, 0.02, (entries, 4)).astype(np.float32)
    dead = np.zeros(n, dtype=bool)
    dead[[0, n - 1]] = True
    idx = torch.empty((m, n // 4), dtype=torch.uint8, device="cuda")
    Wq, err = torch.empty((m, n), dtype=torch.float64, device="cuda"), torch.empty(m, dtype=torch.float64, device="cuda")
    Up = torch.full((n, n + 3), float("nan"), dtype=torch.float64, device="cuda")
    Up[:, :n] = torch.from_numpy(U).cuda()
    ptq.ptq_quantize_layer_vq(torch.from_numpy(W).cuda(), Up[:, :n], torch.from_numpy(dead.astype(np.uint8)).cuda(),
                              torch.from_numpy(C).cuda(), block, idx, Wq, err)
    torch.cuda.synchronize()
    got = idx.cpu().numpy()
    rep = compare_vq(W, U, C, dead, got)
    assert rep["unflagged"] == 0 and rep["flagged"] == 0, rep["details"][:3]
    assert np.array_equal(Wq.cpu().numpy(), C.astype(np.float64)[got].reshape(m, n))
    # n / 4 groups of float64 chains of some ten operations each, compared as the other forms' tests do
    assert np.allclose(err.cpu().numpy(), rep["oracle"]["row_err2"], rtol=1e-9, atol=0)
