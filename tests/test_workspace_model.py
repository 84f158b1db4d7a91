"""A plan's workspace on a model of the HIP runtime (workspace_model.cpp): the
C ABI's host code, compiled as it is, with streams that race, handles that are
given out again, captures and memory that is refused; and the paths it chooses
for frames and batches that were measured on each."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("model") / "workspace_model")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1503_06202_amd", "csrc"),
                    os.path.join(HERE, "workspace_model.cpp"), "-o", exe],
                   check=True, timeout=300)
    return exe


@pytest.mark.parametrize("shape", [0, 1, 2], ids=["small", "channel", "packed"])
@pytest.mark.parametrize("scenario", ["streams_in_turn", "per_thread", "reused_handles", "growth",
                                      "refused", "captured", "two_devices", "last_segment", "bounded_slices", "one_shot", "paths", "batches"])
def test_workspace(model, scenario, shape):
    res = subprocess.run([model, scenario, str(shape)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout == "ok\n", res.stdout + res.stderr
