"""The library's host code on a model of the HIP runtime in which asynchronous
work runs as late as it may (tests/host_model.cpp), under AddressSanitizer and
UndefinedBehaviorSanitizer: what a call returns must not rest on work that it
has not waited for."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2406_17656_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_model") / "host_model")
    cmd = ["g++", "-std=c++17", "-g", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=undefined", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", "/opt/rocm/include",
           "-o", exe, os.path.join(HERE, "host_model.cpp"), os.path.join(CSRC, "sam_capi.cpp"),
           os.path.join(CSRC, "sam_sequence.cpp")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def check(model, *args):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:halt_on_error=1", UBSAN_OPTIONS="halt_on_error=1")
    r = subprocess.run([model, *args], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]


@pytest.mark.parametrize("made", ["plan", "sequence"])
def test_made_on_one_stream_used_on_another(model, made):
    """sam_plan_create and sam_sequence_create synchronise: their buckets are
    there for a build on any stream."""
    check(model, made)


@pytest.mark.parametrize("changed", ["outputs", "select"])
def test_sequence_changed_while_it_runs(model, changed):
    """Other outputs, or other classes, while the last run is still on its way,
    on the same stream or another: no graph is destroyed and no bucket is
    rewritten under a run."""
    check(model, changed)


def test_which_runs_a_graph_takes(model):
    """The fifth run in a row with the same pointers is captured, four graphs at
    most, none of them after its classes have changed, and no stream or event is
    captured with twice."""
    check(model, "graphs")


@pytest.mark.parametrize("seed", range(6))
def test_sequence_orders(model, seed):
    """Selections, refused ones among them, between runs on two streams with
    other outputs: every column of every run is served once, by a class it
    fits."""
    check(model, "orders", str(seed))
