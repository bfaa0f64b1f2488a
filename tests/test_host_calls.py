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


def f32_blocks(n, cus):
    """(32-row blocks, 16-row blocks) of the fp32 route for n rows."""
    if n <= 16 * cus:
        return 0, -(-n // 16)
    rest = n % (32 * cus)
    if rest > 16 * cus:
        return -(-n // 32), 0
    return (n - rest) // 32, -(-rest // 16)


@pytest.mark.parametrize("E,M,slots,n,hidden,cus", [(4, 2, 2, 1, 64, 8), (16, 2, 4, 1, 64, 8), (8, 2, 8, 0, 64, 8),
                                                    (8, 2, 8, 1, 128, 8), (30, 3, 8, 47, 256, 8), (9, 1, 1, 600, 64, 4),
                                                    (40, 3, 5, 40, 64, 3), (5, 1, 1, 2, 64, 256)])
def test_chain_grid_covers_every_row_count(program, E, M, slots, n, hidden, cus):
    """A chain pool's row count is known on the device only: the fp32 route's grid
    has the blocks of every count up to the bound, and they cover the rows."""
    text = run(program, "chain_grid", *map(str, (E, M, slots, n, hidden, cus)))
    grid = next(g for k, g, _, _ in launches(text) if "route_f32" in k)
    bound = n + E * M * slots
    for rows in range(bound + 1):
        pairs, singles = f32_blocks(rows, cus)
        assert pairs + singles <= grid
        assert 32 * pairs + 16 * singles >= rows and 32 * pairs <= rows + 31
    assert grid <= max(cus * -(-bound // (32 * cus)), -(-bound // 16))


def test_growing_reads_allocate_seldom(program):
    """200 reads, each of one env more than the last: the staging grows by doubling."""
    text = run(program, "growing_reads")
    assert sum("export_kernel" in k for k, *_ in launches(text)) >= 200
    assert 1 <= text.count("host memory") <= 9, text.count("host memory")   # 1 env to 200: less than 2^8


@pytest.mark.parametrize("M,slots,n,layers,tile", [(5, 8, 200, 3, 32), (5, 8, 4000, 3, 64), (8, 8, 5000, 2, 32),
                                                   (8, 8, 9000, 2, 64)])
def test_chain_rl_rows_per_tile(program, M, slots, n, layers, tile):
    """RL outputs of a chain pool run 64-row wave tiles when its arrivals alone are
    a heavy tick (8 compute units: above 3,072 rows for the three-layer shape, from
    8,192 rows on for the two-layer one), whatever the bound on its rows is."""
    text = run(program, "chain_rl", *map(str, (M, slots, n, layers)))
    kernel = next(k for k, *_ in launches(text) if "route_bf16_lds" in k)
    args = re.search(r"route_bf16_ldsI(.*)EEvNS", kernel).group(1)   # H, layers, output tiles, K blocks, LDS, waves, ED, row tiles, ...
    row_tiles = int(re.findall(r"L[ib](\d+)E", args + "E")[7])
    assert 32 * row_tiles == tile, kernel
