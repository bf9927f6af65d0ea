"""Which form of the layer error a size takes, from the launches that the host would make (no GPU)."""
import pytest

from launch_recorder import PTR, record

F32, BF16 = 0, 1


def form(dtype, m, n):
    (rc, launches), = record([("ptq_layer_error", [PTR, dtype, n, PTR, m, n, PTR, n, PTR, PTR, 1 << 40, 0])])
    assert rc == 0
    return {name for k in launches for name in ("quad_form_wide_kernel", "quad_form_split_kernel") if name in k["kernel"]}


# bfloat16: 448 tiles, 384 from twelve rows of tiles on; float32: 384 of both traces; never seven rows
@pytest.mark.parametrize("dtype,m,n,wide", [
    (BF16, 2048, 6144, False), (BF16, 2304, 6144, False), (BF16, 2304, 6400, True), (BF16, 2048, 7168, True), (BF16, 2561, 5120, False),
    (BF16, 3072, 4096, True), (BF16, 2816, 4480, False), (BF16, 3072, 3968, False), (BF16, 11008, 4096, True), (BF16, 1792, 11008, False),
    (BF16, 1536, 11008, True), (F32, 1024, 6144, True), (F32, 1024, 6016, False), (F32, 640, 8192, True), (F32, 640, 8064, False),
    (F32, 1792, 4096, False), (F32, 1665, 11008, False), (F32, 1793, 4096, True), (F32, 512, 512, False)])
def test_forms(dtype, m, n, wide):
    assert form(dtype, m, n) == {"quad_form_wide_kernel" if wide else "quad_form_split_kernel"}
