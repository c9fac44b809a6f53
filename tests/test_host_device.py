"""The host code of an engine on a device (work sets, page table, graphs, launches), run without a GPU: the library's objects
linked with tests/host/engine_on_a_fake_runtime.cpp in the place of the HIP runtime."""
import os
import subprocess

import pytest

from paper_2509_19128_amd import build as plbuild

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    objs = [os.path.join(plbuild.OBJ, s.replace(".hip", ".o")) for s in plbuild.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        plbuild.build()
    out = tmp_path_factory.mktemp("host")
    driver, exe = str(out / "driver.o"), str(out / "driver")
    src = os.path.join(ROOT, "tests", "host", "engine_on_a_fake_runtime.cpp")
    for cmd in ([plbuild.HIPCC, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-c", src, "-o", driver],
                [plbuild.HIPCC, "-no-hip-rt", "-o", exe, driver, *objs]):
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("what", ["early_return", "missing_words", "passes_synchronise", "long_waits", "step_time", "logits_behind_their_stream", "same_route", "list_capacity", "scarce_memory", "pass_rows", "pass_buffers", "pass_images", "slices_rule", "operand_limits"])
def test_engine_host_code(program, what):
    r = subprocess.run([program, what], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
