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


def test_refused_free_keeps_the_block(run):
    """A free that is refused loses no block, is reported by the release, and
    leaves no error behind for the launches of the call that wanted more."""
    _, (_, grow, c0), (_, rel, c1), (_, again, c2), (_, last, _) = run("grow", "free=1")
    assert c0 == ["free", "alloc", "free"]  # refused; pool memory of the call's own, whose free is refused too
    assert grow["kept"] == 4 * MIB and grow["live"] == 2
    assert rel["status"] == 8 and rel["detail"] == 1 and rel["kept"] == 4 * MIB and rel["live"] == 2
    assert c1[-1] == "trim" and c1[-2] == "global" and "wait" not in c1
    assert c2 == [] and last["status"] == 0 and last["live"] == 1  # the pool memory that the call could not free


def test_release_reports_a_failed_wait(run):
    _, (_, rel, _), _, (_, last, _) = run("wait=1")
    assert rel["status"] == 8 and rel["detail"] == 1 and rel["kept"] == 0 and rel["last"] == 0
    assert last["status"] == 0 and last["live"] == 0


def test_block_that_cannot_grow(run):
    """No memory for a larger block: the old one is given back, the call reports
    that it has no workspace either."""
    _, (_, grow, c), _, (_, again, _), (_, last, _) = run("grow", "alloc=2")
    assert c == ["free", "alloc", "alloc"] and grow["status"] == 7 and grow["kept"] == 0 and grow["live"] == 0
    assert again["kept"] == 4 * MIB and last["live"] == 0
