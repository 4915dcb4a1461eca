"""The tests of the kernels that hold whole planes, on calls of few planes, with those calls kept on them (GSPN_NO_APART=1): by
themselves they run every direction in a workgroup of its own (test_gpu_apart.py).  Calls of fewer than four directions never do: their
tests are left to their own modules (conftest.py)."""
import importlib
import os

import pytest

from test_gpu_big_maps import *          # noqa: F401,F403
from test_gpu_bwd import *               # noqa: F401,F403
from test_gpu_bwd_twopass import *       # noqa: F401,F403
from test_gpu_f16 import *               # noqa: F401,F403
from test_gpu_fwd import *               # noqa: F401,F403
from test_gpu_local import *             # noqa: F401,F403
from test_gpu_logits import *            # noqa: F401,F403
from test_gpu_never_read import *        # noqa: F401,F403
from test_gpu_ragged import *            # noqa: F401,F403
from test_gpu_ragged_shapes import *     # noqa: F401,F403

pytestmark = pytest.mark.gpu

# tests of one name in two of the modules: the later import hides the earlier one, which is brought back under its module's name too
for _module in ("big_maps", "bwd", "bwd_twopass", "f16", "fwd", "local", "logits", "never_read", "ragged", "ragged_shapes"):
    for _name, _test in list(vars(importlib.import_module("test_gpu_" + _module)).items()):
        if _name.startswith("test_") and globals().get(_name) is not _test:
            globals()[_name + "__" + _module] = _test


@pytest.fixture(autouse=True)
def whole_planes():
    from paper_2512_07884_amd import binding
    before = os.environ.get("GSPN_NO_APART")
    os.environ["GSPN_NO_APART"] = "1"
    binding.gspn_reload_env()
    yield
    os.environ.pop("GSPN_NO_APART") if before is None else os.environ.__setitem__("GSPN_NO_APART", before)
    binding.gspn_reload_env()
