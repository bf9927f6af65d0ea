"""How the bfloat16 Hessian splits its tokens and which form of the main kernel it takes, from the launches that the host would
make (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2601_19675_amd import build
from launch_recorder import PTR, record
import test_gpu_hessian_single_split as single

BIG = {"hessian_bf16_big": {"chunk": (5, "i"), "splits": (8, "i")}}


def plan(n, t):
    """Launches of one call on bfloat16 activations."""
    (rc, launches), = record([("ptq_hessian_accumulate", [PTR, n, PTR, 1, t, n, n, PTR, 1 << 40, 0])], BIG)
    assert rc == 0
    for k in launches:
        form = re.search(r"hessian_bf16_big_kernelILb(\d)ELb(\d)ELb(\d)E", k["kernel"])
        if form:
            k["halves"], k["shared"], k["direct"] = (f == "1" for f in form.groups())
    return launches


# tokens that one float32 sum may take: what whole tiles with partial sums in memory take, also where a split is added to
# H directly or made of half tiles
@pytest.mark.parametrize("n,t,tokens", [(2048, 2048, 320), (2048, 4096, 608), (4096, 2048, 2048), (4096, 16384, 3296), (5632, 2048, 2048),
                                        (8192, 16384, 5472), (9472, 40000, 10016), (11008, 2048, 2048), (11008, 50000, 12512),
                                        (11008, 65536, 16384), (11008, 262144, 65536)])
def test_tokens_of_a_float32_sum(n, t, tokens):
    main = [k for k in plan(n, t) if "direct" in k]
    assert main and all(k["chunk"] == tokens for k in main)
    assert sum(k["splits"] for k in main) == -(-t // tokens)
    # added to H by the kernel itself exactly where there is one split
    assert all(k["direct"] == (t <= tokens) for k in main)


# where a diagonal tile's off-diagonal quadrant is shared by two waves: half tiles, and whole ones in short direct splits
@pytest.mark.parametrize("n,t,halves,shared", [(4096, 2048, True, True), (6144, 2048, True, True), (5632, 2048, False, True), (11008, 16384, False, True),
                                               (11008, 16416, False, False), (11008, 46016, False, False), (11008, 262144, False, False)])
def test_forms_of_the_main_kernel(n, t, halves, shared):
    main = [k for k in plan(n, t) if "direct" in k]
    assert main and all((k["halves"], k["shared"]) == (halves, shared) for k in main)


# the sizes at which the forms are compared with the Gram matrix take the forms that they are listed for
@pytest.mark.parametrize("cases,form", [(single.HALVES, (True, True, True)), (single.WHOLE, (False, True, True)), (single.LONG, (False, False, True)),
                                        (single.SPLIT_HALVES, (True, True, False))], ids=["halves", "whole", "long", "split halves"])
def test_sizes_of_the_single_split_tests(cases, form):
    for n, chunks in cases:
        for t in chunks:
            main = [k for k in plan(n, t) if "direct" in k]
            assert main and all((k["halves"], k["shared"], k["direct"]) == form for k in main), (n, t, main)


def test_main_kernels_keep_their_accumulators_in_registers():
    """No form of the 256 x 256-tile kernel spills: each has only the epilogue that it runs."""
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall")]
    r = subprocess.run([build._hipcc(), *flags, "-S", "--cuda-device-only", os.path.join(build.CSRC, "hessian.hip"), "-o", "-"],
                       capture_output=True, text=True, check=True)
    spills = re.findall(r"\.name:\s+(\S*hessian_bf16_big_kernel\S*)\n(?:.*\n)*?\s+\.private_segment_fixed_size: (\d+)\n"
                        r"(?:.*\n)*?\s+\.vgpr_spill_count: (\d+)", r.stdout)
    assert len(spills) == 5 and all(s[1:] == ("0", "0") for s in spills), spills
