import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def golden_rows(name):
    """Non-comment, non-empty lines of tests/golden/<name>, split on whitespace."""
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", name)
    rows = []
    with open(path) as f:
        for line in f:
            line = line.strip()
            if line and not line.startswith("#"):
                rows.append(line.split())
    return rows


@pytest.fixture(params=["as dispatched", "gemm"])
def route(request):
    """The call as the dispatch serves it, and once more kept on the GEMM kernels (33 rows and more, scale-byte format): the
    small-batch kernel takes most small products, the GEMM kernels' ragged tiles and K-slices want testing all the same.
    A forced shape of that family that no kernel has, so that the number of K-slices stays the heuristic's."""
    import paper_2501_04052_amd as razer
    from paper_2501_04052_amd import binding
    if request.param == "gemm":
        razer.razer_tune_force(binding.TUNE_GEMM_SLICES, (0,))
    yield request.param
    razer.razer_tune_force(binding.TUNE_GEMM_SLICES, None)


@pytest.fixture(scope="session")
def oracle():
    import oracle as o
    o.lib()
    return o
