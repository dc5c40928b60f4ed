"""Launches of the library's host code on a recording HIP runtime, without a GPU.

Every library source is compiled for the host only and linked with
tests/host/launch_checks.hip, whose runtime records launches and runs no
kernel.  The driver solves over the shapes whose lines or planes one block
holds; the largest dynamic LDS that each kernel was launched with, added to
what the kernel declares itself (the metadata of the built library's code
objects), has to fit the 160 KB of a compute unit.
"""
import os
import re
import subprocess

import pytest

from tests import codeobj

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1607_05816_amd", "csrc")
SOURCES = ["uot_kernels.hip", "uot_grid_tf.hip", "uot_dense_mf.hip", "uot_api.hip", "uot_net.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LLVM = codeobj.LLVM
LDS = 160 * 1024

pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(LLVM + "/clang++")),
                                reason="needs the ROCm toolchain")


def _run(cmd, **kw):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, **kw)
    return r.returncode, r.stdout.decode(errors="replace")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("launches")
    objs, procs = [], []
    for src in [os.path.join(CSRC, s) for s in SOURCES] + [os.path.join(ROOT, "tests", "host", "launch_checks.hip")]:
        objs.append(str(d / os.path.basename(src).replace(".hip", ".o")))
        procs.append(subprocess.Popen(
            [HIPCC, "-O1", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "--offload-host-only", "--offload-new-driver",
             "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"), "-c", src, "-o", objs[-1]],
            stdout=subprocess.PIPE, stderr=subprocess.STDOUT))
    for p in procs:
        out, _ = p.communicate()
        assert p.returncode == 0, out.decode(errors="replace")
    exe = str(d / "launch_checks")
    rc, out = _run([LLVM + "/clang++", *objs, "-o", exe])
    assert rc == 0, out
    return exe


@pytest.fixture(scope="module")
def static_lds(tmp_path_factory):
    if not codeobj.available():
        pytest.skip("needs the built library")
    return {k: v["lds"] for k, v in codeobj.kernels(tmp_path_factory.mktemp("codeobj")).items()}


@pytest.mark.parametrize("what", ["lines", "planes", "barycenters"])
def test_lds_of_every_shape_fits(driver, static_lds, what):
    rc, out = _run([driver, what], timeout=300)
    assert rc == 0 and "launch checks passed" in out, out
    seen = 0
    for line in out.splitlines():
        m = re.match(r"(_Z\S+) (\d+) (.*)", line)
        if not m:
            continue
        name, dynamic, shape = m.group(1), int(m.group(2)), m.group(3)
        assert name in static_lds, name
        assert dynamic + static_lds[name] <= LDS, (name, shape, dynamic, static_lds[name])
        seen += "k_line" in name or "k_plane" in name
    assert seen >= 4


def test_every_loop_and_plane_kernel_is_reached(driver, static_lds):
    rc, out = _run([driver, "instances"], timeout=300)
    assert rc == 0 and "launch checks passed" in out, out
    for kernel in ("k_line_loop", "k_plane_pair"):
        built = {name for name in static_lds if kernel in name}
        launched = {name for name in re.findall(r"^(_Z\S+)", out, re.M) if kernel in name}
        assert built and built == launched


def test_a_failing_launch_is_reported_by_its_call(driver):
    """Every launch of a solve fails in turn, with and without a graph,
    synchronous and asynchronous: the call returns the error, no error is left for
    the next one, and the context goes on working."""
    rc, out = _run([driver, "failing"], timeout=300)
    assert rc == 0 and "launch checks passed" in out, out


# where the line passes are the faster ones (see line_min_lines, line_plane_pays):
# L lines, P lines and planes in pairs, S a line pass per launch, - the other passes
ROUTES = {
    "f32": {(8, 512): "L", (8, 2048): "-", (200, 2048): "L", (2048, 8): "-", (8, 2050): "-", (2050, 8): "L",
            (8, 32, 32): "P", (8, 64, 64): "P", (8, 16, 256): "S", (8, 80, 80): "-", (30, 80, 80): "S"},
    "f64": {(8, 512): "L", (8, 2048): "-", (200, 2048): "L", (2048, 8): "L", (8, 2050): "-", (2050, 8): "L",
            (8, 32, 32): "P", (8, 64, 64): "S", (8, 16, 256): "S", (8, 80, 80): "S", (30, 80, 80): "S"},
}


@pytest.fixture(scope="module")
def routes(driver):
    rc, out = _run([driver, "routes"], timeout=300)
    assert rc == 0 and "launch checks passed" in out, out
    return out


def test_routes_of_grid_solves(routes):
    got = {"f32": {}, "f64": {}}
    for m in re.finditer(r"route solve (f\d\d) (\d+)x(\d+)x(\d+) \S+ \d+ c \S+:(.*)", routes):
        shape = tuple(int(x) for x in m.group(2, 3, 4) if x != "0")
        if len(shape) == 1:
            continue
        names = m.group(5)
        got[m.group(1)][shape] = ("P" if "k_plane_pair" in names else "L" if "k_line_pair" in names
                                  else "S" if "6k_lineI" in names else "-")
    assert got == ROUTES


def test_whole_iterations_build_no_kernel_table(routes):
    for dtype in ("f32", "f64"):
        names = {int(n): names for n, names in re.findall(rf"route solve {dtype} (\d+)x0x0 \S+ \d+ c \S+:(.*)", routes)}
        for n in (40, 500):
            assert "k_line_loop" in names[n] and "k_gtab" not in names[n]
        assert "k_line_loop" not in names[1000] and "k_gtab" in names[1000]


def test_the_timed_half_step_is_the_one_that_runs(routes):
    got = {}
    for what, dtype, n, names in re.findall(r"route (half-step|timed) (f\d\d) (\d+)x0x0 \S+ \d+ c \S+:(.*)", routes):
        got.setdefault((dtype, int(n)), {})[what] = names
    assert len(got) == 6
    for key, names in got.items():
        assert names["timed"] == names["half-step"], key


# ... and the paired passes with the combine among them (line_bary_root_passes): B paired,
# S a line pass per launch, - the other passes
BARY_ROUTES = {
    "f32": {(2, 64, 64): "B", (8, 50, 50): "B", (10, 80, 80): "-", (10, 81, 81): "S", (10, 150, 150): "B", (12, 48, 48): "B",
            (16, 64, 64): "B", (20, 50, 50): "-", (24, 20, 40): "-", (24, 96, 96): "S", (30, 64, 64): "-",
            (33, 40, 60): "S", (60, 32, 32): "-"},
    "f64": {(2, 64, 64): "B", (8, 50, 50): "B", (10, 80, 80): "S", (10, 81, 81): "S", (10, 150, 150): "B", (12, 48, 48): "-",
            (16, 64, 64): "S", (20, 50, 50): "-", (24, 20, 40): "-", (24, 96, 96): "S", (30, 64, 64): "S",
            (33, 40, 60): "S", (60, 32, 32): "S"},
}


def test_routes_of_barycenters(routes):
    got = {"f32": {}, "f64": {}}
    others = {}
    for m in re.finditer(r"route barycentre (\S+) (f\d\d) (\d+)x(\d+)x\S+ fields (\d+) c \S+:(.*)", routes):
        kind, dtype, n0, n1, nb = m.group(1), m.group(2), *(int(x) for x in m.group(3, 4, 5))
        names = m.group(6)
        way = "B" if re.search(r"k_line_pairI\S+Li2EE", names) else "S" if "6k_lineI" in names else "-"
        if kind == "TV":
            got[dtype][nb, n0, n1] = way
        else:
            others[kind, dtype, nb, n0, n1] = way
    assert got == BARY_ROUTES
    # a mean needs no search; a range without a lower bound has one breakpoint an input
    for dtype in ("f32", "f64"):
        assert others["KL", dtype, 24, 96, 96] == "B" and others["KL", dtype, 24, 20, 40] == "B"
        assert others["RG", dtype, 24, 96, 96] == "S"
    assert others["RG", "f64", 24, 20, 40] == "-" and others["RG", "f64", 12, 48, 48] == "B"


# tap slices of WF lines (grid_contig_splits) where one count was measured ahead of its
# neighbours: (fields, cells, cut in lengths of the line)
SLICES = {
    "f32": {(1, 3000, 0.3): 7, (1, 4096, 0.3): 8, (1, 4096, 4.0): 16},
    "f64": {(1, 2500, 4.0): 6, (1, 3000, 0.3): 5, (1, 3000, 4.0): 10, (1, 4096, 0.3): 8, (1, 4096, 4.0): 16,
            (2, 3000, 4.0): 8, (2, 4000, 4.0): 14, (5, 4000, 4.0): 4},
}


def test_slices_of_lines(driver):
    rc, out = _run([driver, "slices"], timeout=300)
    assert rc == 0 and "launch checks passed" in out, out
    got = {"f32": {}, "f64": {}}
    for m in re.finditer(r"slices (f\d\d) fields (\d+) cells (\d+) cut (\S+): (\d+)", out):
        got[m.group(1)][int(m.group(2)), int(m.group(3)), float(m.group(4))] = int(m.group(5))
    for dtype, want in SLICES.items():
        assert len(got[dtype]) == 56
        for key, k in want.items():
            assert got[dtype][key] == k, (dtype, key)
    # the launches of a flow of several species have a column of blocks more, for the control step
    flows = {tuple(int(x) for x in m[:2]): int(m[2])
             for m in re.findall(r"flow f64 fields (\d+) cells (\d+) cut 4: (\d+)", out)}
    assert len(flows) == 28
    for key, k in {(1, 3000): 10, (1, 4096): 16, (2, 1500): 5, (2, 2000): 7, (2, 3000): 8, (2, 4000): 14, (3, 1500): 3,
                   (3, 3000): 7, (3, 4000): 8}.items():
        assert flows[key] == k, key
    assert got["f64"][2, 2000, 4.0] == 4 and got["f64"][3, 3000, 4.0] == 9
