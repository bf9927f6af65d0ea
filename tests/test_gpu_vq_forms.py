"""The vector-quantized walk at the edges of its two codebook forms (up to 64 entries, up to 256) against its oracle."""
import numpy as np
import pytest
import torch

import paper_2601_19675_amd as ptq
from oracle import vq_oracle as vo
from parity import compare_vq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entries,dim", [(1, 1), (31, 2), (33, 4), (64, 1), (65, 2), (255, 4), (256, 1)])
@pytest.mark.parametrize("block", [16, 128, 256])
def test_entries_around_the_lanes_and_the_forms(entries, dim, block):
    rng = np.random.default_rng(100 * entries + dim)
    m, n = 21, 272   # a last block narrower than the others
    W = rng.normal(0, 0.02, (m, n))
    W[:, 5] = 0.0
    U = np.triu(rng.normal(0, 0.05, (n, n)), 1) + np.diag(np.exp(rng.normal(0, 0.5, n)))
    C = rng.normal(0, 0.02, (entries, dim)).astype(np.float32)
    C[-1] = C[0]                                    # equal losses: the lower index wins
    ref = vo.quantize_layer_vq(W, U, C, want_margins=True)
    idx = torch.empty((m, n // dim), dtype=torch.uint8, device="cuda")
    Wq, err = torch.empty((m, n), dtype=torch.float64, device="cuda"), torch.empty(m, dtype=torch.float64, device="cuda")
    ptq.ptq_quantize_layer_vq(torch.from_numpy(W).cuda(), torch.from_numpy(U).cuda(), None, torch.from_numpy(C).cuda(), block, idx, Wq, err)
    torch.cuda.synchronize()
    # a float64 walk in another order of summation: the oracle's choice wherever its margin is above the rounding
    sure = np.all(ref["second"] - ref["best"] > 1e-9 * np.abs(ref["second"]), axis=1) if entries > 2 else np.ones(m, bool)
    dup = np.any(ref["indices"] == 0, axis=1)       # a duplicated entry has no margin but a rule
    rows = sure | dup if entries > 1 else sure
    assert rows.any()
    got = idx.cpu().numpy()
    assert np.array_equal(got[rows], ref["indices"][rows].astype(np.uint8))
    assert not np.any(got == entries - 1) or entries == 1
    assert np.allclose(Wq.cpu().numpy()[rows], ref["Wq"][rows], rtol=0, atol=0)
    assert np.allclose(err.cpu().numpy()[rows], ref["row_err2"][rows], rtol=1e-10)


# n is a multiple of the vector's length only: one mini-block that is not full, a last block narrower than a mini-block, the
# last of several mini-blocks not full, a full block before it, and both forms of the block's width
@pytest.mark.parametrize("n,block", [(4, 16), (20, 16), (132, 128), (60, 64), (140, 256), (252, 256), (388, 128)])
@pytest.mark.parametrize("entries,dim", [(9, 1), (64, 2), (200, 4)])
def test_columns_past_the_last_whole_mini_block(n, block, entries, dim):
    rng = np.random.default_rng(1000 * n + entries)
    n -= dim % 4                                    # 1, 2 or 0 columns short of a multiple of 4
    m = 19
    W = rng.normal(0, 0.02, (m, n))
    U = np.triu(rng.normal(0, 0.05, (n, n)), 1) + np.diag(np.exp(rng.normal(0, 0.5, n)))
    C = rng.normal(0, 0.02, (entries, dim)).astype(np.float32)
    dead = np.zeros(n, dtype=bool)
    dead[n - 1] = True
    # outputs with a guard behind them, inputs and a workspace of their exact sizes
    idx = torch.full((m * (n // dim) + 64,), 0xEE, dtype=torch.uint8, device="cuda")
    Wq = torch.full((m * n + 64,), 7.0, dtype=torch.float64, device="cuda")
    err = torch.full((m,), float("nan"), dtype=torch.float64, device="cuda")
    ptq.ptq_quantize_layer_vq(torch.from_numpy(W).cuda(), torch.from_numpy(U).cuda(), torch.from_numpy(dead.astype(np.uint8)).cuda(),
                              torch.from_numpy(C).cuda(), block, idx[:m * (n // dim)].view(m, n // dim), Wq[:m * n].view(m, n), err)
    torch.cuda.synchronize()
    assert (idx[m * (n // dim):] == 0xEE).all() and (Wq[m * n:] == 7.0).all()
    got = idx[:m * (n // dim)].view(m, n // dim).cpu().numpy()
    rep = compare_vq(W, U, C, dead, got)
    assert rep["unflagged"] == 0 and rep["flagged"] == 0, rep["details"][:3]
    assert np.array_equal(Wq[:m * n].view(m, n).cpu().numpy(), C.astype(np.float64)[got].reshape(m, n))
    assert np.allclose(err.cpu().numpy(), rep["oracle"]["row_err2"], rtol=1e-9, atol=0)
