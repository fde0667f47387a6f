import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: long-running CPU test")


@pytest.fixture(scope="session")
def gpu():
    """Skip unless a GPU is visible; returns the loaded library binding."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_2509_16686_amd import binding
    return binding.lib()


@pytest.fixture(scope="session")
def tok_pieces(tmp_path_factory):
    """Runs the host build of the decode plan and the d_c 128 decode's balanced schedule (tok_pieces_host.cpp)."""
    cxx = shutil.which("g++") or shutil.which("c++")
    assert cxx, "no C++ compiler"
    exe = str(tmp_path_factory.mktemp("tok_pieces") / "tok_pieces_host")
    csrc = os.path.join(ROOT, "paper_2509_16686_amd", "csrc")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "tok_pieces_host.cpp"), os.path.join(csrc, "host_plan.cpp"),
                    "-o", exe], check=True)

    def run(*args, text=""):
        r = subprocess.run([exe, *map(str, args)], input=text, capture_output=True, text=True)
        assert r.returncode == 0, (args, r.stdout, r.stderr)
        return [tuple(map(int, line.split())) for line in r.stdout.splitlines()]
    return run
