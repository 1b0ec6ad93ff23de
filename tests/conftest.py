import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu on the GPU box)")


def pytest_collection_modifyitems(config, items):
    # the no-allocation entry point's test (if present) must be collected last
    items.sort(key=lambda it: ("test_zz_" in it.nodeid, ))


@pytest.fixture(scope="session")
def golden_dir():
    return os.path.join(ROOT, "tests", "golden")


@pytest.fixture(scope="session")
def assembly(tmp_path_factory):
    """csrc/sqllm_quant.hip as the compiler emits it for the GPU"""
    from paper_2306_07629_amd import build
    assert shutil.which(build.HIPCC), "hipcc is needed to build the library"
    out = tmp_path_factory.mktemp("asm") / "quant.s"
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    src = [s for s in build.sources() if s.endswith("sqllm_quant.hip")]
    subprocess.run([build.HIPCC, *flags, "--cuda-device-only", "-S", "-I" + build.CSRC, *src, "-o", str(out)], check=True, capture_output=True)
    return out.read_text()
