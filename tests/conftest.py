import os
import sys

# numpy's products in the same order on every host (before numpy is loaded): OpenBLAS chooses its kernels by the CPU, and the last iterations of a
# minimisation in fp64 go one way or the other by the last bit (test_lbfgs_step_rules_and_convergence passed on hosts with AVX-512 only)
os.environ.setdefault("OPENBLAS_CORETYPE", "Prescott")

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def _have_gpu():
    try:
        import torch
        return torch.cuda.is_available()
    except Exception:
        return False


def pytest_collection_modifyitems(config, items):
    if _have_gpu():
        return
    skip = pytest.mark.skip(reason="no GPU in this container")
    for it in items:
        if "gpu" in it.keywords:
            it.add_marker(skip)
