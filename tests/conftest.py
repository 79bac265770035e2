import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def pytest_collection_modifyitems(config, items):
    """GPU tests are skipped, loudly, when no device is present."""
    import torch
    if torch.cuda.is_available():
        return
    skip = pytest.mark.skip(reason="no GPU in this process")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)


@pytest.fixture(autouse=True)
def default_kernel_path(request):
    """The switch of rpo_set_kernel_path is process-wide: every GPU test starts without a forced path, whichever test ran
    before it (a model test would otherwise compare a forced kernel with itself)."""
    if "gpu" in request.keywords:
        from paper_2601_19404_amd import binding
        binding.rpo_set_kernel_path(0)
