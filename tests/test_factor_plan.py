"""Which way a factor goes, read from the launches that the host would make: 128 columns at a time up to 5120 columns, halves
of more by the recursion, and rows of U too long for the steps' 32-bit offsets by the recursion as well."""
import pytest

import paper_2601_19675_amd as ptq
from launch_recorder import PTR, record
from paper_2601_19675_amd import binding


def _launches(n, ldu):
    ws = ptq.ptq_workspace_bytes(binding.OP_CHOLESKY_INV, 0, n)
    (rc, launches), = record([("ptq_damped_cholesky_inv", [PTR, n, n, 0.01, PTR, ldu, 0, PTR, PTR, ws, 0])])
    assert rc == 0
    return launches


@pytest.mark.parametrize("n", [1, 128, 129, 512, 4096, 5120])
def test_steps(n):
    launches = _launches(n, n)
    blocks = -(-n // 128)
    steps = [l["grid"][0] for l in launches if "step_kernel" in l["kernel"]]
    # the leaf, and for every block row below the half tiles up to its diagonal block (the leaf's own row without that)
    tiles = [0] + [2 * ((blocks - k) * (blocks + k + 1) // 2 - 1) for k in range(1, blocks)]
    assert steps == [1 + min(t, 255) for t in tiles]
    assert sum("diagonal_kernel" in l["kernel"] for l in launches) == blocks - 1
    assert not any("node_gemm" in l["kernel"] for l in launches)


@pytest.mark.parametrize("n,ldu", [(5121, 5121), (11008, 11008), (1000, (1 << 20) + 1)])
def test_recursion(n, ldu):
    launches = _launches(n, ldu)
    assert any("node_gemm" in l["kernel"] for l in launches)
    # every block of 128 columns has its leaf
    assert sum("step_kernel" in l["kernel"] for l in launches) == -(-n // 128)
    if ldu > 1 << 20:
        assert all(l["grid"][0] == 1 for l in launches if "step_kernel" in l["kernel"])


@pytest.mark.parametrize("n", [129, 300, 2000])
def test_narrow_nodes_of_long_rows(n):
    # up to about 1500 columns a node's products are bound by latency: 32 x 32 tiles
    nodes = [l["kernel"] for l in _launches(n, (1 << 20) + 1) if "node_gemm" in l["kernel"]]
    assert nodes and all("ILi1ELi1E" in k for k in nodes)


def test_wide_nodes_of_long_rows():
    # a node of 128 x 128 tiles, halves that go on halving: the early part of panel and update beside the second half of the first child
    capped = [l for l in _launches(8192, (1 << 20) + 1) if "ILi4ELi4ELb1E" in l["kernel"]]
    assert sorted(l["grid"][0] for l in capped) == [128, 192, 192]   # T, and the early part's two


@pytest.mark.parametrize("n", [100, 129, 300])
def test_row_length_past_31_bits(n):
    ws = ptq.ptq_workspace_bytes(binding.OP_CHOLESKY_INV, 0, n)
    ldu = (1 << 31) + 16
    (rc, launches), = record([("ptq_damped_cholesky_inv", [PTR, n, n, 0.01, PTR, ldu, 0, PTR, PTR, ws, 0])],
                             read={"step_kernel": dict(ldu=(0, "q", 16)), "node_gemm": dict(ldu=(0, "q", 16))})
    assert rc == 0
    rows = [l["ldu"] for l in launches if "ldu" in l]
    assert rows and all(r == ldu for r in rows)
