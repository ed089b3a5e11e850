"""The line and tile kernels of the general transform run on the CPU: the
kernel sources built against a stand-in HIP runtime (tests/host/emu) whose
threads switch at barriers only, in two opposite orders of workgroups, waves
and lanes.  Every result must have the same bits in both orders (a read that no
barrier orders after the write it needs has not) and lie within the FP32 bound
(relative L2 error 1e-5) of 64-bit sums; 16-bit scores within their storage
bound.  The driver also fails on a barrier that not all waves reach and on
writes past the LDS of a launch, its outputs or its workspace."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1505_07690_amd", "csrc")
HOST = os.path.join(ROOT, "tests", "host")
CLANG = os.environ.get("ROCM_CLANG", "/opt/rocm/llvm/bin/clang++")
BOUND = {"forward_bf16": 4e-3, "forward_fp16": 5e-4}
LINES, PLANES = 0, 2  # routes: y and x lines, whole planes


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("clang++ not available")
    d = str(tmp_path_factory.mktemp("kernels"))
    # the inline assembly only hides values from the optimiser; dynamic LDS becomes a global array
    for name in sorted(os.listdir(CSRC)):
        if name.endswith(".h") or name in ("kernels_fft.hip", "kernels_line.hip", "kernels_tile.hip"):
            with open(os.path.join(CSRC, name)) as f:
                s = f.read()
            s = re.sub(r"\basm( volatile)?\(", "EMU_ASM(", s).replace("extern __shared__", "extern")
            s = s.replace('"../../include/os3d.h"', '"os3d.h"')
            with open(os.path.join(d, name.replace(".hip", ".cpp")), "w") as f:
                f.write(s)
    sources = [os.path.join(d, f"kernels_{k}.cpp") for k in ("fft", "line", "tile")]
    sources += [os.path.join(CSRC, "host_setup.cpp"), os.path.join(HOST, "kernel_driver.cpp")]
    exe = os.path.join(d, "kernel_driver")
    r = subprocess.run([CLANG, "-std=c++17", "-O0", "-w", "-ffp-contract=off", "-I", d, "-I",
                        os.path.join(HOST, "emu"), "-I", os.path.join(ROOT, "include"), *sources, "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def run(driver, shape, rows, paired, route, split=0, batch=1, pairs_per_launch=None, only=""):
    """{result: checksum} of a case, after the checks that every case has to pass."""
    env = dict(os.environ)
    env.pop("OS3D_PAIR_BATCH", None)
    if pairs_per_launch:
        env["OS3D_PAIR_BATCH"] = str(pairs_per_launch)
    args = [*shape, rows, int(paired), route, split, batch, only]
    r = subprocess.run([driver, *map(str, args)], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0, r.stdout[-500:] + r.stderr[-500:]
    out = {}
    for line in r.stdout.splitlines():
        f = line.split()
        if f[0] == "workspace":
            out["workspace"] = int(f[1])
            continue
        name, err, order, checksum = f
        assert order == "same", line
        assert float(err) < BOUND.get(name, 1e-5), line
        out[name] = checksum
    assert len(out) == (3 if only == "forward" else 10) + 1
    return out


# lengths of y whose first stage joins two factors (radix 6, 9, 10, 12, 15), and some whose first has one
@pytest.mark.parametrize("ny", [6, 10, 12, 15, 81, 90, 108, 135, 150, 162, 243, 250, 270, 324, 8, 20, 64, 125, 240])
def test_y_lines_of_16_bit_scores(driver, ny):
    lines = run(driver, (2, ny, 3), 2, True, LINES, batch=2, only="forward")
    planes = run(driver, (2, ny, 3), 2, True, PLANES, batch=2, only="forward")
    # one order of the sums however the work is divided: the same stored words
    for name in ("forward_bf16", "forward_fp16"):
        assert lines[name] == planes[name]


def intermediates(rows, cap=64):
    """Pairs per launch: the fewest launches of at most `cap` pairs, evenly filled."""
    launches = -(-rows // cap)
    return -(-rows // launches)


# (shape, rows, paired, route, split, batch, OS3D_PAIR_BATCH): pair sums shared
# by several workgroups, in one launch and in several, on every route
SHARED_SUMS = [((6, 5, 9), 70, False, PLANES, 0, 2, 24),
               ((8, 9, 5), 81, False, LINES, 0, 1, None),
               ((5, 12, 15), 12, True, LINES, 2, 2, None),
               ((9, 16, 10), 12, True, LINES, 4, 1, 7),
               ((16, 6, 10), 21, True, PLANES, 0, 2, 9),
               ((40, 3, 4), 12, False, LINES, 0, 1, None),
               ((2, 4, 3), 64, False, PLANES, 0, 2, None)]  # the bounds of many pairs on the least grid


@pytest.mark.parametrize("shape,rows,paired,route,split,batch,pairs", SHARED_SUMS)
def test_workspace_holds_the_pairs_and_two_volumes(driver, shape, rows, paired, route, split, batch, pairs):
    got = run(driver, shape, rows, paired, route, split, batch, pairs)
    v = shape[0] * shape[1] * shape[2]
    assert got["workspace"] <= (2 + max(2, intermediates(rows, pairs or 64))) * 8 * v + 256


# every kind of plan with a batch of two: one, two and three factors an axis,
# several planes in a tile, ragged tiles, each split, unpaired sets
@pytest.mark.parametrize("shape,rows,paired,route,split", [
    ((9, 4, 5), 2, True, PLANES, 0), ((12, 30, 18), 2, False, PLANES, 0), ((4, 50, 12), 1, True, PLANES, 0),
    ((20, 6, 36), 2, True, LINES, 0), ((18, 24, 10), 1, False, LINES, 0),
    ((5, 18, 25), 2, True, LINES, 2), ((32, 12, 9), 1, False, LINES, 4), ((2, 48, 8), 2, True, LINES, 8)])
def test_plans_in_both_orders(driver, shape, rows, paired, route, split):
    run(driver, shape, rows, paired, route, split, batch=2)
