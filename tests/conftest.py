import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def oracle():
    import oracle as _o
    _o.lib()
    return _o


@pytest.fixture
def launched_kernels():
    """Names of the kernels that a call launches."""
    import torch
    from paper_2511_11664_amd import binding as B

    def launched(call):
        B.rans_profile_reset()
        B.rans_profile_enable("all")
        try:
            call()
            torch.cuda.synchronize()
            return set(B.rans_profile_read())
        finally:
            B.rans_profile_enable(None)
            B.rans_profile_reset()
    return launched
