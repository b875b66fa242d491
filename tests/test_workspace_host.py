"""The workspace memory on the host (no GPU): what a call and a release do when
the HIP runtime says that the null stream is busy or that a capture forbids
operations on it (tests/workspace_host.cpp runs csrc/workspace.h against a
scripted runtime)."""
import os
import subprocess

import pytest

from conftest import ROOT

NOT_READY, CAPTURE_IMPLICIT = 600, 906  # hipErrorNotReady, hipErrorStreamCaptureImplicit
MIB = 1 << 20


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("workspace") / "workspace_host")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include",
                    os.path.join(ROOT, "tests", "workspace_host.cpp"), "-o", exe, "-lpthread"], check=True)

    def go(*args):
        out = subprocess.run([exe, *args], check=True, capture_output=True, text=True).stdout
        steps = []
        for line in out.splitlines():
            name, *fields = line.split()
            f = dict(x.split("=", 1) for x in fields)
            steps.append((name, {k: int(v) for k, v in f.items() if k != "calls"}, f["calls"].split(",")[:-1]))
        return steps

    return go


def test_block_is_kept_and_given_back(run):
    (_, first, c0), (_, rel, c1), (_, again, _), (_, last, _) = run()
    assert first["kept"] == 4 * MIB and c0 == ["alloc"]
    assert rel["status"] == 0 and rel["kept"] == 0 and rel["live"] == 0
    assert c1[-1] == "trim" and c1.index("free") < c1.index("wait")
    assert again["kept"] == 4 * MIB and last["live"] == 0


def test_release_waits_for_no_call(run):
    """Work on the null stream: nothing is waited for, and the block that the
    work may use stays for a later release."""
    _, (_, rel, calls), (_, again, c), (_, last, _) = run(f"query={NOT_READY}")
    assert "wait" not in calls and "free" not in calls and calls[-1] == "trim"
    assert rel["status"] == 0 and rel["kept"] == 4 * MIB and rel["last"] == 0
    assert c == [] and last["live"] == 0


def test_release_beside_a_capture_leaves_the_null_stream_alone(run):
    _, (_, rel, calls), _, (_, last, _) = run(f"capturing={CAPTURE_IMPLICIT}")
    assert calls == ["capturing", "trim"]
    assert rel["status"] == 0 and rel["kept"] == 4 * MIB and rel["last"] == 0
    assert last["live"] == 0
