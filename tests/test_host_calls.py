"""Host side of the C ABI on a machine without a GPU: a small program stands in
for the runtime (memory from the host, kernels not run) and prints the launches
of a scenario with their grids and the device current at each."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2606_11440_amd", "libinframind.so")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(LIB):
        from paper_2606_11440_amd import build
        build.build()
    out = str(tmp_path_factory.mktemp("host") / "host_calls")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-rdynamic", "-o", out,
                           os.path.join(ROOT, "tests", "host_calls.cpp"), "-ldl"])
    return out


def run(program, *scenario):
    r = subprocess.run([program, LIB, *scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-2000:])
    return r.stdout


def launches(text):
    """(kernel, grid, block, device) of each launch."""
    found = re.findall(r"launch (\S+) grid (\d+) block (\d+) device (\d+)", text)
    return [(k, int(g), int(b), int(d)) for k, g, b, d in found]


def test_no_compute_unit_count(program):
    """A failed query of the compute units leaves a pool that routes."""
    text = run(program, "no_cu_count")
    got = launches(text)
    assert len(got) == 12 and all("route" in k for k, *_ in got), text
    assert all(g >= 1 for _, g, _, _ in got)


def test_state_calls_run_on_the_pools_device(program):
    """Reading and restoring a pool's state while another device is current works
    on the pool's device, and leaves the caller's current."""
    text = run(program, "other_device")
    got = launches(text)
    for name in ("export_kernel", "snapshot_kernel", "dual_recount_kernel"):
        assert any(name in k for k, *_ in got), text
    assert "device 1" not in text.replace("after device 1", ""), text
    assert text.endswith("after device 1\n")


def test_restore_recounts_what_it_touched(program):
    """The running totals of the dual update (1,024 shards, env e in shard e mod
    1,024) are recounted for the restored envs' shards only, a block each."""
    parts = run(program, "restore").split("envs ")[1:]
    got = {int(t.split("\n")[0]): [g for k, g, _, _ in launches(t) if "dual_recount" in k] for t in parts}
    assert got == {0: [], 1: [1], 3: [3], 1024: [1024], 2000: [1024]}
