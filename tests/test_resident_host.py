"""Host logic of the one-launch solves: the layouts that resident_host.cpp
builds on its threads (16-bit columns, halo lists, exchange slots), checked
against brute force, under AddressSanitizer with UndefinedBehaviorSanitizer and
under ThreadSanitizer (CPU only)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads as w

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_09812_amd", "csrc")
SANITIZERS = {"address": ["-fsanitize=address", "-fsanitize=undefined", "-fno-sanitize-recover=all"],
              "thread": ["-fsanitize=thread"]}


@pytest.fixture(scope="module", params=list(SANITIZERS))
def tool(request, tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp(request.param)
    exe = str(d / "resident_check")
    flags = [x for f in SANITIZERS[request.param] for x in ("-Xarch_host", f)]
    subprocess.check_call([hipcc, "-O1", "-g", "-fno-omit-frame-pointer", "-std=c++17", "-pthread"] + flags +
                          ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                           os.path.join(ROOT, "tests", "host", "resident_check.cpp")] +
                          [os.path.join(CSRC, f) for f in ("mesh_prep.cpp", "gs_rows.cpp", "resident_host.cpp")] +
                          ["-o", exe], stderr=subprocess.DEVNULL)
    return exe, d


def _block(a, b, c):
    """a x b x c nodes in a box one cell larger: nothing periodic, so any number of unique nodes."""
    ijk = np.stack(np.meshgrid(np.arange(a), np.arange(b), np.arange(c), indexing="ij"), -1)
    at = np.arange(a * b * c).reshape(a, b, c)
    unit = w.kuhn_cube(2, 1.0)
    corner = unit.xyz.astype(int)[unit.tets]
    cells = ijk[:-1, :-1, :-1].reshape(-1, 1, 1, 3) + corner[None]
    tets = at[cells[..., 0], cells[..., 1], cells[..., 2]].reshape(-1, 4)
    xyz = ijk.reshape(-1, 3).astype(float)
    return xyz, tets, np.ones(len(tets), np.uint8), np.zeros(3), np.array([a, b, c], float)


def _cube(n, **kw):
    m = w.small_cube(n, seed=n, L=8e-8, jitter=0.15, **kw).mesh
    return m.xyz, m.tets, m.tags, m.lo, m.hi


# unique nodes, compute units: one workgroup; a ragged last block; rows without entries; blocks of 64, 128 (fewer
# workgroups), several rows a thread (few units); orders with long halo lists; a last block of a single row
CASES = {
    "64_one_workgroup": (lambda: _cube(5), 256, 0, 512),
    "125": (lambda: _cube(6), 256, 0, 64),
    "729_sphere_shuffled": (lambda: _cube(10, sphere=0.4, shuffle=True), 256, 0, 512),
    "1331": (lambda: _cube(12), 256, 1, 128),
    "4096_five_sphere": (lambda: _cube(17, sphere=0.3, split="five"), 256, 0, 512),
    "4913_callers_order_shuffled": (lambda: _cube(18, shuffle=True), 256, 1, 256),
    "8000_rcm": (lambda: _cube(21), 256, 2, 512),
    "13824_of_2048_rows": (lambda: _cube(25, sphere=0.25), 7, 0, 512),
    "4161_last_block_of_one_row": (lambda: _block(3, 19, 73), 256, 0, 512),
    "1089_blocks_of_128": (lambda: _block(3, 11, 33), 256, 1, 64),
}


@pytest.mark.parametrize("name", list(CASES))
def test_layouts_match_brute_force_under_sanitizers(tool, name):
    exe, d = tool
    mesh, cus, reorder, rows = CASES[name]
    xyz, tets, tags, lo, hi = mesh()
    path = str(d / f"{name}.bin")
    with open(path, "wb") as f:
        np.array([len(xyz), len(tets)], np.int64).tofile(f)
        for a, t in ((lo, np.float64), (hi, np.float64), (xyz, np.float64), (tets, np.int32), (tags, np.uint8)):
            np.ascontiguousarray(a, dtype=t).tofile(f)
    r = subprocess.run([exe, path, str(cus), str(reorder), str(rows)], capture_output=True, text=True,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=1"), timeout=300)
    print(r.stdout.strip())
    assert r.returncode == 0, r.stdout + r.stderr[-3000:]
    assert "Sanitizer" not in r.stderr and "runtime error" not in r.stderr, r.stderr[-3000:]


def test_memory_and_threads_that_run_out(tmp_path):
    """A failing allocation on any thread reaches the caller as std::bad_alloc, a thread that cannot be had is done without."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "resident_faults")
    subprocess.check_call([hipcc, "-O1", "-g", "-std=c++17", "-pthread", "-I" + os.path.join(ROOT, "include"),
                           "-I" + CSRC, os.path.join(ROOT, "tests", "host", "resident_faults.cpp"),
                           os.path.join(CSRC, "resident_host.cpp"), "-ldl", "-o", exe], stderr=subprocess.DEVNULL)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout.strip())
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]
