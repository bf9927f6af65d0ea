"""Which form of the vector walk a block goes by, read from the launches: codebooks of more than 64 entries of 4 weights have
one for blocks of one or two tiles and one that stages the block of U for three to eight."""
import pytest

import paper_2601_19675_amd as ptq
from launch_recorder import PTR, record
from paper_2601_19675_amd import binding

F32 = 0


def _forms(n, entries, dim, block, m=40):
    ws = ptq.ptq_workspace_bytes(binding.OP_QUANTIZE, m, n)
    args = [PTR, F32, n, m, n, PTR, n, 0, PTR, entries, dim, block, PTR, 0, 0, PTR, ws, 0]
    (rc, launches), = record([("ptq_quantize_layer_vq", args)])
    assert rc == 0
    return [l["kernel"].split("vq_block_kernel")[1].split("EE")[0] for l in launches if "vq_block_kernel" in l["kernel"]]


@pytest.mark.parametrize("entries", [65, 256])
@pytest.mark.parametrize("block,tiles", [(16, 2), (32, 2), (48, 8), (128, 8), (144, 16)])
def test_long_codebooks(entries, block, tiles):
    assert _forms(2 * block, entries, 4, block) == [f"ILi0ELi{tiles}ELi4ELi8ELb0"] * 2


def test_last_block():
    assert _forms(128 + 32, 256, 4, 128) == ["ILi0ELi8ELi4ELi8ELb0", "ILi0ELi2ELi4ELi8ELb0"]
    assert _forms(128 + 20, 256, 4, 128) == ["ILi0ELi8ELi4ELi8ELb0", "ILi0ELi16ELi4ELi8ELb1"]


@pytest.mark.parametrize("entries,dim,slots", [(64, 4, 2), (256, 2, 8), (256, 1, 8)])
def test_other_codebooks(entries, dim, slots):
    assert _forms(64, entries, dim, 32) == [f"ILi0ELi8ELi{dim}ELi{slots}ELb0"] * 2
