"""The launches the library's host code makes, on the CPU: its host objects
linked against a stand-in for the HIP runtime (tests/host_launch/probe.cpp)
that records kernels, grids and dynamic LDS."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2210_15763_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
CLANG = "/opt/rocm/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(CLANG)),
                                reason="hipcc / ROCm clang not found")


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """launches(calls): for each call (a line of text) its output lines."""
    tmp = str(tmp_path_factory.mktemp("host_launch"))
    srcs = [os.path.join(CSRC, f) for f in ("bandeig.hip", "spmm.hip", "tallskinny.hip")]
    srcs.append(os.path.join(ROOT, "tests", "host_launch", "probe.cpp"))
    jobs, objs = [], []
    for src in srcs:
        objs.append(os.path.join(tmp, os.path.basename(src) + ".o"))
        cmd = [HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-x", "hip", "-O0", "-g0",
               "-std=c++17", "-Wno-unused-command-line-argument", "-I" + CSRC, "-c", src, "-o",
               objs[-1]]
        jobs.append(subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                                     text=True))
    for p in jobs:
        out = p.communicate()[0]
        assert p.returncode == 0, out[-4000:]
    exe = os.path.join(tmp, "probe")
    # the device code's symbol is the only one left open
    r = subprocess.run([CLANG, "-no-pie", "-Wl,--unresolved-symbols=ignore-all"] + objs +
                       ["-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def run(calls):
        r = subprocess.run([exe], input="\n".join(calls) + "\n", capture_output=True, text=True,
                           timeout=60)
        assert r.returncode == 0, r.stderr[-4000:]
        parts = r.stdout.split("end\n")
        assert len(parts) == len(calls) + 1 and parts[-1] == ""
        return [p.splitlines() for p in parts[:-1]]

    return run


def test_band_eig_lds_limits_hold_on_every_device(launches):
    """A kernel's dynamic LDS limit is a device's own: a second device gets
    every launch the first one gets."""
    calls = ["band %d %d %d" % c for c in ((900, 8, 10), (1448, 8, 10), (1000, 16, 16),
                                           (3000, 4, 16), (2600, 10, 4), (9000, 12, 4))]
    out = launches(calls + ["device 1"] + calls)
    first, second = out[:len(calls)], out[len(calls) + 1:]
    assert all(len(o) > 4 for o in first)
    big = [l for o in first for l in o if int(l.split()[3]) > 65536]
    assert len(big) >= 6
    for call, a, b in zip(calls, first, second):
        assert not any("refused" in l or l.startswith("error") for l in a + b), (call, a, b)
        assert a == b


def test_band_eig_factors_in_lds(launches):
    """Up to 150 KB of factors and vector a target's inverse iteration keeps
    them in LDS, one workgroup a target."""
    calls = ["band %d %d 10" % (19200 // (kd + 2), kd) for kd in (1, 2, 4, 8, 10)]
    for call, out in zip(calls, launches(calls)):
        assert any(l.startswith("k_invit_two<") and l.split()[1] == "11" for l in out), (call, out)


def test_band_eig_wide_bands_beyond_lds(launches):
    """At bandwidth 16 with factors beyond LDS a target's inverse iteration has
    a workgroup (k_invit), as at the bandwidths without a register window."""
    calls = ["band %d %d %d" % c for c in ((1136, 16, 4), (1136, 16, 32), (8192, 16, 16),
                                           (15, 16, 5), (900, 12, 5))]
    for call, out in zip(calls, launches(calls)):
        k = call.split()[-1]
        assert any(l.split()[:2] == ["k_invit", k] for l in out), (call, out)


F32, F64 = 1, 2


def spmm_kernel(launches, calls):
    """Name of the one kernel of each call (n, nonzeros a row, type, width)."""
    out = launches(["spmm %d %d %d %d %d" % (n, n * z, dt, b, dt) for n, z, dt, b in calls])
    assert all(len(o) == 1 for o in out)
    return [o[0].split()[0] for o in out]


def test_spmm_lanes_of_short_matrices(launches):
    """Widths without a compiled kernel keep 16 lanes a row on matrices past
    3072 rows (their reduction covers 32 columns), compiled ones up to 64."""
    generic = [(n, z, dt, b) for n in (3073, 4000, 6000, 8192) for z in (5, 31, 121)
               for dt in (F32, F64) for b in (7, 9, 13, 28, 31)]
    for call, k in zip(generic, spmm_kernel(launches, generic)):
        assert k.startswith("k_spmm_generic<") and k.endswith(",16>"), (call, k)
    rest = [((1000, 61, F32, 7), 64), ((2000, 61, F64, 13), 32),
            ((3000, 31, F64, 13), 16), ((3000, 121, F64, 13), 32), ((6000, 300, F64, 7), 16), ((1000, 121, F32, 8), 64),
            ((4000, 121, F64, 4), 64), ((4000, 300, F32, 10), 32), ((6000, 121, F32, 8), 32),
            ((8000, 300, F32, 10), 16), ((8000, 300, F32, 12), 16), ((9000, 450, F64, 8), 32)]
    for (call, lanes), k in zip(rest, spmm_kernel(launches, [c for c, _ in rest])):
        assert k.endswith(",%d>" % lanes), (call, k)


def test_spmm_of_short_rows(launches):
    """Rows of V of 32 to 80 bytes: a lane takes whole rows where a row of the
    matrix has some 10 to 40 entries and V outgrows the caches, groups share them elsewhere."""
    own = [(n, z, dt, b) for n in (400000, 2000000) for z in (17, 22)
           for dt, b in ((F32, 8), (F32, 12), (F32, 16), (F32, 20), (F64, 4), (F64, 8), (F64, 10))]
    own += [(100000, 31, F32, 8), (400000, 37, F64, 4), (2000000, 9, F32, 12), (2000000, 13, F32, 16),
            (400000, 33, F64, 10), (400000, 61, F32, 10), (400000, 61, F64, 3)]
    for call, k in zip(own, spmm_kernel(launches, own)):
        assert k.startswith("k_spmm<"), (call, k)
    shared = [(n, z, dt, b) for n in (9000, 400000, 2000000) for z in (5, 41, 211, 420)
              for dt, b in ((F32, 8), (F32, 16), (F64, 4), (F64, 10))]
    shared += [(n, z, dt, b) for n in (9000, 2000000) for z in (5, 17, 33, 61)
               for dt, b in ((F32, 24), (F32, 32), (F64, 12), (F64, 16))]
    shared += [(400000, 9, F32, 8), (400000, 31, F64, 8), (4000, 17, F32, 8), (30000, 17, F32, 8),
               (100000, 17, F64, 8), (100000, 33, F64, 10)]
    for call, k in zip(shared, spmm_kernel(launches, shared)):
        assert k.startswith("k_spmm_split<"), (call, k)


def test_gram_grids(launches):
    """Kernels and grids of the products of narrow blocks: 8-wide FP64 blocks
    of any number on matrix cores; no short matrix with few blocks held to 64
    row chunks; more than six 10-wide FP64 blocks on as many workgroups as
    the chip holds at once (768)."""
    def one(n, dt, b, nblk):
        out = launches(["gram %d %d %d %d" % (n, dt, b, nblk)])[0]
        assert len(out) == 2 and out[1].startswith("parts ")
        name, grid = out[0].split()[:2]
        return name.split("<")[0], int(grid), int(out[1].split()[1])

    for n in (500, 65000, 130000, 2000000):
        for nblk in (2, 3, 8, 9, 45):
            assert one(n, F64, 8, nblk)[0] == "k_gram_quads"
    for dt, b, n, nblk in ((F32, 4, 65000, 20), (F32, 4, 40000, 45), (F64, 8, 65000, 9),
                           (F64, 8, 20000, 45)):
        assert one(n, dt, b, nblk)[2] > 64
    assert one(65000, F64, 8, 45)[2] <= 64
    for n in (65000, 400000):
        for nblk in (7, 16, 20, 45, 80, 120, 150, 180):
            name, grid, _ = one(n, F64, 10, nblk)
            assert name == "k_gram_rows" and 640 < grid <= 768, (n, nblk, grid)
    for dt, b in ((F32, 4), (F64, 4)):
        assert one(400000, dt, b, 4)[0] == "k_gram_rows"
