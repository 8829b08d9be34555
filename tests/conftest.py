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
    from oracle import mfa_oracle
    mfa_oracle.lib()
    return mfa_oracle


@pytest.fixture(params=[0, 256], ids=["any", "cut"])
def get_ctx(request):
    """Contexts that distribute work as the library sees fit, where little work is not cut or goes in runs; and with 256 workgroups asked for, which is what the
    default aims for too, but then for every call: little work as well goes through the kernels and the schedule that larger work does."""
    import gpu_util
    return lambda **kw: gpu_util.get_ctx(**kw, **({"target_workgroups": request.param} if request.param else {}))
