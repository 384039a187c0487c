"""The library's host code (every .cpp of csrc) through its C interface under
AddressSanitizer and UndefinedBehaviorSanitizer, with a stand-in for the HIP
runtime on host memory (tests/host/hip_on_host.cpp) and kernels that do nothing
(CPU only).  Every device and pinned buffer is a heap block of its own size, so
an access past any of them, a leak or a use after a release ends the run."""
import glob
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads as w

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_09812_amd", "csrc")
SAN = ["-fsanitize=address", "-fsanitize=undefined", "-fno-sanitize-recover=all"]
FLAGS = ["-O1", "-g", "-fno-omit-frame-pointer", "-std=c++17", "-pthread"] + [x for f in SAN for x in ("-Xarch_host", f)]


def test_host_code_on_host_memory(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    clang = "/opt/rocm/llvm/bin/clang++"
    if not (os.path.exists(hipcc) and os.path.exists(clang)):
        pytest.skip("compilers not available")
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC]
    host = os.path.join(ROOT, "tests", "host")
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.cpp"))) + [os.path.join(host, f) for f in ("hip_on_host.cpp",
                                                                                            "lib_check.cpp")]
    objs, jobs = [], []
    for s in srcs:
        objs.append(str(tmp_path / (os.path.basename(s) + ".o")))
        jobs.append(subprocess.Popen([hipcc] + FLAGS + inc + ["-c", s, "-o", objs[-1]], stderr=subprocess.DEVNULL))
    assert all(j.wait() == 0 for j in jobs)
    # the launchers nothing above defines: functions that return at once
    names = lambda flag: {line.split()[-1] for o in objs for line in subprocess.check_output(
        ["nm", flag, o], text=True).splitlines() if line.strip() and ":" not in line}
    missing = sorted(n for n in names("-u") - names("--defined-only") if n.startswith("_ZN4gspm"))
    assert any("launch_field_rhs" in n for n in missing) and not any("operator_rows" in n for n in missing)
    stub = tmp_path / "stubs.s"
    stub.write_text(".text\n" + "".join(f".globl {n}\n{n}:\n xorl %eax, %eax\n ret\n" for n in missing)
                    + '.section .note.GNU-stack,"",@progbits\n')
    exe = str(tmp_path / "lib_check")
    subprocess.check_call([clang] + SAN + objs + [str(stub), "-pthread", "-o", exe])
    paths = []
    for name, mesh in (("4", w.small_cube(4, seed=4, jitter=0.1).mesh), ("9", w.small_cube(9, seed=9, sphere=0.3).mesh),
                       ("14s", w.small_cube(14, seed=14, shuffle=True).mesh),
                       ("17", w.small_cube(17, seed=17, split="five", sphere=0.25).mesh)):
        paths.append(str(tmp_path / (name + ".bin")))
        with open(paths[-1], "wb") as f:
            np.array([len(mesh.xyz), len(mesh.tets)], np.int64).tofile(f)
            for a, t in ((mesh.lo, np.float64), (mesh.hi, np.float64), (mesh.xyz, np.float64), (mesh.tets, np.int32),
                         (mesh.tags, np.uint8)):
                np.ascontiguousarray(a, dtype=t).tofile(f)
    r = subprocess.run([exe] + paths, capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=1"))
    print(r.stdout.strip()[-2000:])
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-4000:]
    assert "Sanitizer" not in r.stderr and "runtime error" not in r.stderr, r.stderr[-4000:]
