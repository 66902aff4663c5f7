import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def orc():
    import oracle

    oracle.build()
    return oracle


@pytest.fixture(scope="session")
def listings(tmp_path_factory):
    """{source: the gfx950 listing of its kernels}, all translation units of the library compiled side by side."""
    if shutil.which("hipcc") is None:
        pytest.skip("needs hipcc")
    from paper_2107_01460_amd import build
    folder = tmp_path_factory.mktemp("listings")

    def listing(src):
        out = str(folder / src.replace(".hip", ".s"))
        subprocess.check_call(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, src), "-o", out])
        with open(out) as f:
            return f.read()

    with ThreadPoolExecutor(max_workers=min(os.cpu_count() or 8, 8)) as ex:
        return dict(zip(build.SOURCES, ex.map(listing, build.SOURCES)))
