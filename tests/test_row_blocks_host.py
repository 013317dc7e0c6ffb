"""Row and hub blocks on the host: the blocks decode to the matrix and leave the tree and its counters alone, the automatic rules take them
where they should, and a build that runs out of memory says so."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2409_02208_amd as cbm
import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _harness(tmp_path, source, *flags):
    """The host builder with a main of its own, compiled and run; what it printed."""
    exe = str(tmp_path / "harness")
    csrc = os.path.join(ROOT, "paper_2409_02208_amd", "csrc")
    cmd = ["g++", "-std=c++17", "-O1", "-g", *flags, "-I", os.path.join(ROOT, "include"),
           "-I", csrc, os.path.join(ROOT, "tests", source), os.path.join(csrc, "cbm_builder.cpp"), "-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0 and "sanitize" in r.stderr:
        pytest.skip("sanitizer runtime not available: " + r.stderr[-200:])
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout[-500:], r.stderr[-3000:])
    return r.stdout


SANITIZED = ("-fsanitize=address,undefined", "-fno-sanitize-recover=all")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_blocks_decode_to_the_matrix(tmp_path):
    out = _harness(tmp_path, "host_blocks_main.cpp", *SANITIZED)
    assert "blocks ok" in out and "hubs ok" in out


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_out_of_memory_in_a_thread_reaches_the_caller(tmp_path):
    assert "allocations ok" in _harness(tmp_path, "host_alloc_main.cpp")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_who_takes_blocks_and_what_is_left_of_a_plan_given_up(tmp_path):
    """The automatic rules themselves (the other tests force the blocks or leave them out)."""
    assert "policy ok" in _harness(tmp_path, "host_policy_main.cpp")


def test_blocks_leave_tree_and_counters_alone(monkeypatch):
    g = wl.make_graph("protein", n=3000, knn=40)
    handles = []
    for want in ("0", "1"):
        monkeypatch.setenv("CBM_ROW_BLOCKS", want)
        handles.append(cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True, host_only=True))
    a, b = (cbm.cbm_stats(h) for h in handles)
    assert {k: v for k, v in a.items() if k != "build_seconds"} == {k: v for k, v in b.items() if k != "build_seconds"}
    for x, y in zip(cbm.cbm_get_tree(handles[0]).values(), cbm.cbm_get_tree(handles[1]).values()):
        assert np.array_equal(x, y)


def test_bench_figures_are_of_what_runs():
    """With launches over blocks the bytes and gathered rows are those of the launch records, not of the tree's deltas."""
    import bench

    stats = dict(m=100, n=100, num_delta_plus=5000, num_delta_minus=1000, num_roots=20)
    k = 32
    paths = {0: dict(deltas=12000, bytes=0), 2: dict(deltas=0, bytes=0)}
    assert bench.method_figures(stats, k, True, paths, 2) == (bench.algorithmic_bytes(stats, k, True), 6000, bench.compulsory_bytes(stats, k, True))
    blocks = {5: dict(deltas=1280, bytes=2000000)}   # two products
    assert bench.method_figures(stats, k, True, blocks, 2) == (1000000, 640, 4 * k * 200 + 640 * 24 + 100 * 8)
    hubs = {5: dict(deltas=1280, bytes=200000), 1: dict(deltas=400, bytes=300000), 0: dict(deltas=800, bytes=500000)}
    assert bench.method_figures(stats, k, True, hubs, 2) == (500000, 1240, 4 * k * 200 + 640 * 24 + 600 * 8 + 100 * 8)


def test_bench_knows_every_kernel_of_a_product():
    """The counter children match dispatches to launch records by their order, so no kernel of a product may be missing; the roofline names what ran."""
    import glob
    import os
    import re

    import bench

    sources = [open(p).read() for p in glob.glob(os.path.join(os.path.dirname(cbm.__file__), "csrc", "*.hip")) if "gemm" not in p and "build" not in p]
    kernels = {k for s in sources for k in re.findall(r"__global__[^;{]*?void (cbm_\w+_kernel)\(", s)} - {"cbm_entry_weights_kernel"}  # (once per handle)
    assert kernels == set(bench.PRODUCT_KERNELS)
    counted = [dict(kind=6, level=1, kernel="cbm_sum_sets_kernel"), dict(kind=6, level=2, kernel="cbm_sum_rows_kernel"), dict(kind=0, level=1, kernel="cbm_flat_kernel")]
    assert [bench.dominant_kernel(kind, counted) for kind in (0, 6)] == ["cbm_flat_kernel", "cbm_sum_rows_kernel"]
    assert [bench.dominant_kernel(kind, None) for kind in (0, 5, 6)] == ["cbm_level_kernel", "cbm_block_kernel", "cbm_sum_rows_kernel"]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_panel_kernel_takes_an_unaligned_b_where_that_was_measured_to_pay(tmp_path):
    """(M, N, K, staged kernel, panel kernel: microseconds, or the panel's time over the staged kernel's) on both sides of the rule's lines."""
    measured = [(132534, 17, 32, 10.3, 14.8), (132534, 47, 32, 13.2, 18.5), (132534, 65, 32, 17.8, 24.2), (40000, 250, 32, 21.5, 25.7),
                (20000, 17, 100, 8.3, 10.3), (20000, 50, 64, 8.4, 10.0), (40000, 33, 100, 13.0, 14.7), (28000, 17, 256, 1.0, 1.42),
                (100000, 47, 64, 1.0, 1.06), (132534, 47, 100, 31.9, 28.7), (132534, 17, 64, 1.0, 0.92), (132534, 130, 64, 1.0, 0.61),
                (40000, 250, 64, 1.0, 0.84), (200000, 33, 48, 1.0, 0.90), (50000, 47, 100, 1.0, 0.93), (40000, 17, 256, 1.0, 0.73),
                (34000, 17, 100, 1.0, 0.93), (34000, 50, 128, 1.0, 0.91), (32768, 17, 100, 1.0, 1.23), (32768, 63, 200, 1.0, 1.06), (40000, 47, 256, 1.0, 0.91),
                (9000, 17, 100, 1.0, 0.92), (12000, 17, 100, 1.0, 1.08), (8192, 50, 100, 1.0, 0.84), (18000, 50, 100, 1.0, 1.15), (8192, 47, 120, 1.0, 1.12)]
    main = tmp_path / "rule.cpp"
    main.write_text('#include <cstdio>\n#include "cbm_internal.h"\nint main() {\n' +
                    "".join(f"    std::printf(\"%d\", cbm_panel_takes_unaligned({m}, {n}, {k}));\n" for m, n, k, _, _ in measured) + "}\n")
    exe = str(tmp_path / "rule")
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2409_02208_amd", "csrc"), str(main), "-o", exe],
                   check=True)
    taken = [c == "1" for c in subprocess.run([exe], capture_output=True, text=True, check=True).stdout]
    assert taken == [panel < staged for _, _, _, staged, panel in measured]
