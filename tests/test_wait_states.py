"""Wait states around instructions that the kernels issue from inline assembly, where the compiler does not count them."""
import os

import pytest

from paper_2601_19675_amd import build

LOAD = "\tbuffer_load_dwordx4 v1, s[0:3], s9 offen lds"


@pytest.mark.parametrize("text", [
    "\ts_mov_b32 m0, s4\n" + LOAD,                                       # the address in m0
    "\ts_add_u32 m0, s4, 0x400\n\t;;#ASMEND\n" + LOAD,
    "\tv_readfirstlane_b32 s2, v3\n\ts_mov_b32 m0, s4\n\ts_nop 0\n" + LOAD,  # a word of the descriptor
    "\tv_readlane_b32 s9, v3, 1\n\ts_nop 3\n" + LOAD,                   # the offset
    ".LBB0_1:\n" + LOAD + "\n\tv_readfirstlane_b32 s1, v3\n\ts_cbranch_scc1 .LBB0_1",   # round a loop
])
def test_a_load_into_lds_too_close_is_found(text):
    with pytest.raises(RuntimeError):
        build.check_lds_dma_wait_states(text)


@pytest.mark.parametrize("text", [
    "\ts_mov_b32 m0, s4\n\ts_nop 0\n" + LOAD,
    "\tv_readfirstlane_b32 s2, v3\n\ts_nop 4\n" + LOAD,
    "\tv_readfirstlane_b32 s4, v3\n\ts_mov_b32 s2, s4\n" + LOAD,          # by way of a scalar instruction
    "\tv_readfirstlane_b32 s2, v3\n\ts_branch .LBB0_2\n.LBB0_1:\n" + LOAD,   # another path
])
def test_a_load_into_lds_far_enough_passes(text):
    assert build.check_lds_dma_wait_states(text) == 1


@pytest.mark.parametrize("src", sorted(s for s, c in build.ASSEMBLY_CHECKS.items() if c is build.check_lds_dma_wait_states))
def test_generated_assembly(src):
    build.check_assembly(src)


def test_every_source_with_such_loads_is_checked():
    with_loads = set()
    for src in build.SOURCES:
        with open(os.path.join(build.CSRC, src)) as f:
            if "lds_dma.h" in f.read():
                with_loads.add(src)
    assert with_loads == {s for s, c in build.ASSEMBLY_CHECKS.items() if c is build.check_lds_dma_wait_states}
