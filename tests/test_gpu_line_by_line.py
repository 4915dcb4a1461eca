"""The line-by-line kernels against the fp64 oracle on ordinary shapes, in the three storage types: the global scan, GSPN-local,
weights as logits, direction masks, forward, forward with h_save and backward.  They take the calls no other kernel takes and
are what the fast kernels are compared with, so GSPN_FORCE_GENERIC=1 runs them here on maps that others normally take."""
import pytest

from test_gpu_local import check_local
from test_gpu_logits import check_logits

pytestmark = pytest.mark.gpu

DTYPES = ["f32", "bf16", "f16"]
# a single row and column, odd and even sides, lines of one and of several turns of the workgroup, 12 and 64 channels per group,
# a plane beyond the LDS tile
SHAPES = [(1, 2, 1, 37, 1), (1, 2, 37, 1, 2), (2, 6, 9, 13, 3), (1, 4, 33, 70, 2), (2, 24, 28, 28, 2), (1, 64, 33, 35, 1), (1, 1, 300, 5, 1),
          (1, 1, 210, 230, 1)]


@pytest.fixture(autouse=True)
def line_by_line(monkeypatch):
    monkeypatch.setenv("GSPN_FORCE_GENERIC", "1")


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_global_scan(shape, dtype):
    check_local(shape + (dtype,), 1 << 14)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape,kchunk,mask", [((2, 6, 9, 13, 3), 4, 15), ((1, 4, 33, 70, 2), 1, 15), ((1, 8, 28, 28, 2), 10, 6), ((1, 2, 64, 65, 1), 64, 9)],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_local_stretches_and_direction_masks(shape, kchunk, mask, dtype):
    check_local(shape + (dtype,), kchunk, mask=mask, poison_starts=dtype != "f16")


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape,kchunk,mask", [((2, 6, 9, 13, 3), None, 15), ((1, 4, 41, 73, 2), 16, 15), ((1, 24, 28, 28, 2), None, 15), ((1, 2, 130, 67, 2), None, 5)],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_weights_as_logits(shape, kchunk, mask, dtype):
    check_logits(shape + (dtype,), kchunk=kchunk, mask=mask, poison=dtype != "f16")
