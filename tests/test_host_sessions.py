"""Sessions of libplse on a stand-in for the HIP runtime (no GPU): lifetimes of
streams, events and graphs, work left running, launch shapes and the split of
the distances.  The check program defines the runtime's functions itself, and
the library it is linked with calls those."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2103_10453_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(
    not shutil.which(HIPCC) or not os.path.exists(os.path.join(PKG, "libplse.so")),
    reason="hipcc or libplse.so missing")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = tmp_path_factory.mktemp("sessions") / "host_sessions_check"
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                    os.path.join(HERE, "host_sessions_check.cpp"), "-o", str(exe), "-L", PKG,
                    "-lplse", "-Wl,-rpath," + PKG, "-Wl,--export-dynamic"],
                   check=True, capture_output=True)

    def run(scenario):
        out = subprocess.run([str(exe), scenario], capture_output=True, text=True, timeout=300)
        assert out.returncode == 0 and out.stdout.strip().endswith("ok"), out.stdout + out.stderr
    return run


def test_single_sessions(check):
    check("single")


def test_distance_units_once(check):
    check("units")


def test_batch_sessions(check):
    check("batch")


def test_failing_calls_settle(check):
    check("errors")


def test_launches_within_64k_lds(check):
    check("lds64")
