"""What the host returns when the runtime refuses a kernel its LDS (no GPU: the runtime is the recording stand-in)."""
import pytest

from launch_recorder import PTR, record

PTQ_ERR_HIP = 6


def forward(tokens, m, n, failing=""):
    args = [PTR, 0, n, tokens, m, n, PTR, 4, PTR, PTR, 32, PTR, n, 16, PTR, PTR, PTR, 4, PTR, PTR, m, PTR, 1 << 40, 0]
    (rc, launches), = record([("ptq_lopro_linear_forward", args)], failing=failing)
    return rc, [k["kernel"] for k in launches]


@pytest.mark.parametrize("tokens,m,kernel", [(1, 4096, "forward_rows_kernel"), (4, 100, "forward_rows_kernel"), (1, 64, "forward_prep_kernel"),
                                             (64, 64, "forward_prep_kernel")])
def test_a_stored_layer_that_is_not_launched_is_an_error(tokens, m, kernel):
    rc, launched = forward(tokens, m, 4096)
    assert rc == 0 and any(kernel in k for k in launched)
    rc, launched = forward(tokens, m, 4096, failing=kernel)
    assert rc == PTQ_ERR_HIP and not any(kernel in k for k in launched)
