"""Where the launches of the stored layer put what they share in the workspace, from the arguments that the host would pass
(no GPU)."""
import random

import pytest

from launch_recorder import PTR, record

WS = 1 << 32
FORWARD_ARGS = dict(xt=(0, "q", 40), y=(0, "q", 56), y_parts=(0, "q", 64), y_splits=(0, "i", 72), exponents=(0, "q", 104),
                    partial=(0, "q", 112))   # fields of the product's first argument
PLAN = dict(tokens=(1, "i"), token_blocks=(2, "i", 0), row_blocks=(2, "i", 4), splits=(2, "i", 8))


def products(tokens, m, n, r, bits=4, group=32):
    """Launches of the tile product of one call, and the size of its workspace."""
    size = workspace(tokens, m, n, r)
    (rc, launches), = record([("ptq_lopro_linear_forward", [PTR, 0, n, tokens, m, n, PTR, bits, PTR, PTR, group, PTR, n, 16, PTR, PTR, PTR, r,
                                                           PTR, PTR, m, WS, size, 0])], {"forward_tile_kernel": {**FORWARD_ARGS, **PLAN}})
    assert rc == 0
    return [k for k in launches if "splits" in k], size


def workspace(tokens, m, n, r):
    up = lambda v: -(-v // 256) * 256  # noqa: E731
    return up(4 * tokens * n) + up(4 * tokens * max(r, 1)) + up(-(-(n // 32) // 8) * 32 * m * 4) + up(-(-m // 256) * 4)


def check_disjoint(tokens, m, n, r):
    found, size = products(tokens, m, n, r)
    for k in found:
        t = k["tokens"]
        assert t >= 1 and k["token_blocks"] * 64 >= t and k["row_blocks"] * 256 >= m
        regions = [("X~", k["xt"], 4 * t * n), ("exponents", k["exponents"], 4 * t),
                   ("partial sums", k["partial"], 4 * (k["splits"] - 1) * t * m)]
        if k["y_parts"]:
            assert k["y_parts"] % 8 == 0
            regions.append(("parts of the coefficients", k["y_parts"], 8 * k["y_splits"] * t * r))
        elif r:
            regions.append(("coefficients", k["y"], 4 * t * r))
        regions = sorted((at, at + length, name) for name, at, length in regions if length)
        assert regions[0][0] >= WS and regions[-1][1] <= WS + size, (tokens, m, n, r, regions)
        for (_, end, a), (begin, _, b) in zip(regions, regions[1:]):
            assert end <= begin, f"{a} and {b} overlap: {tokens} tokens, {m} x {n}, {r} ranks: {regions}"
    return found


# layers of few rows, most with so many tokens that these go in runs, the last of which splits its columns
@pytest.mark.parametrize("tokens,m,n,last,splits", [(133, 1, 512, 5, 2), (133, 1, 4096, 133, 3), (585, 1, 4096, 9, 16), (582, 2, 2048, 6, 8),
                                                    (395, 3, 544, 11, 2), (193, 1, 32, 65, 1)])
def test_runs_of_tokens(tokens, m, n, last, splits):
    found = check_disjoint(tokens, m, n, 0)
    assert (found[-1]["tokens"], found[-1]["splits"]) == (last, splits)
    check_disjoint(tokens, m, n, 16)


@pytest.mark.parametrize("seed", range(8))
def test_no_two_regions_overlap(seed):
    rng = random.Random(seed)
    log = lambda lo, hi: int(2 ** rng.uniform(lo, hi))  # noqa: E731
    for _ in range(4):
        check_disjoint(min(4096, max(5, log(2, 12.01))), log(0, 13.4) if rng.random() < 0.5 else log(0, 4), 32 * log(0, 8.4), rng.choice([0, 1, 16, 40]))
