"""The arenas that GPU tests take for a way of launching the outer step do reach it: the library's host code is asked on the
CPU, with stand-ins for the HIP runtime and the kernel launchers."""
import glob
import os
import re
import subprocess

import pytest

import step_shapes as shapes
import workloads
from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2506_10911_amd", "csrc")
ROCM_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")   # HIP API declarations only
STREAMING, THROUGH, KEPT = 0, 1, 2


@pytest.fixture(scope="module")
def launches_of(tmp_path_factory):
    exe = tmp_path_factory.mktemp("routes") / "route_driver"
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    "-I", ROCM_INCLUDE, os.path.join(ROOT, "tests", "route_driver.cpp"), os.path.join(CSRC, "api.cpp"),
                    os.path.join(CSRC, "launch_plan.cpp"), "-o", str(exe)], check=True)

    def ask(calls):
        """A list of launches for each call (bf16, between, (segments, stride, W, sizes))."""
        lines = []
        for bf16, between, (segments, stride, W, sizes) in calls:
            runs = " ".join(f"{o} {n}" for o, n in segments)
            lines.append(f"{int(bf16)} {W} {stride} {between} {len(segments)} {runs} {len(sizes)} " + " ".join(map(str, sizes)))
        out = subprocess.run([str(exe)], input="\n".join(lines) + "\n", check=True, capture_output=True, text=True, timeout=60).stdout
        names = ("n", "groups", "in_order", "together", "paced", "stores", "phases", "class_shift")
        return [[dict(zip(names, map(int, launch.split()))) for launch in line.split(";") if launch.strip()] for line in out.splitlines()]

    return ask


@pytest.mark.parametrize("kind", shapes.KINDS)
def test_phases(launches_of, kind):
    cases = [(n, bf16) for n in shapes.PHASED for bf16 in (False, True)]
    for (n, bf16), got in zip(cases, launches_of([(bf16, 0, shapes.phased(n, bf16, kind)) for n, bf16 in cases])):
        want = dict(phases=1, class_shift=shapes.PHASED[n][bf16][0].bit_length() - 1, n=n, together=0, stores=THROUGH)
        assert len(got) == 1 and {k: got[0][k] for k in want} == want, (n, bf16, got)


@pytest.mark.parametrize("kind", shapes.KINDS)
def test_phases_far_apart(launches_of, kind):
    cases = [(shape, bf16) for shape in shapes.PHASED_FAR_APART for bf16 in (False, True)]
    calls = [(bf16, shapes.FAR_APART, shapes.phased_far_apart(*shape, kind)) for shape, bf16 in cases]
    for (shape, bf16), got in zip(cases, launches_of(calls)):
        assert len(got) == 1 and got[0]["phases"] == 1 and 1 << got[0]["class_shift"] == shape[1], (shape, bf16, got)


def test_delta_in_registers(launches_of):
    """kernels.hip takes in-order launches of 17 to 48 members without phases to that kernel up to 1024 pieces."""
    for segments in shapes.HELD:
        pieces = sum((o + n - 1) // 256 - o // 256 + 1 for o, n in segments)
        assert (2 * pieces <= 1024) == (segments != shapes.HELD[-1]) and pieces <= 513
        calls = [(bf16, 0, (segments, shapes.stride_of(segments), 2 * n, [n, n])) for n in shapes.HELD_SIZES for bf16 in (False, True)]
        for got in launches_of(calls):
            assert len(got) == 1 and got[0]["groups"] == 2 and got[0]["in_order"] == 1 and got[0]["phases"] == 0, got


def test_narrowing(launches_of):
    for columns, phases, got in zip(shapes.NARROWED, (0, 1), launches_of([(True, 0, ([(0, c)], c, 17, [17])) for c in shapes.NARROWED])):
        assert len(got) == 1 and got[0]["in_order"] == 1 and got[0]["phases"] == phases, (columns, got)


def test_mixed_sizes(launches_of):
    cases = [(case, bf16) for case in shapes.MIXED for bf16 in (False, True)]
    for ((way, sizes, _, _), bf16), got in zip(cases, launches_of([(bf16, 0, shapes.mixed(*case[1:])) for case, bf16 in cases])):
        assert [launch["n"] for launch in got] == sorted(set(sizes)), (way, sizes, bf16, got)
        for launch in got:
            assert launch["together"] == 1 and launch["in_order"] == 1 and launch["phases"] == 0, (way, sizes, bf16, got)
            assert launch["stores"] == (KEPT if way == "kept" else THROUGH), (way, sizes, bf16, got)
        assert way != "paced" or all(launch["paced"] for launch in got), (way, sizes, bf16, got)


def test_profiles_are_of_the_kernels_that_run(launches_of):
    """Every traffic profile of an outer step names the kernels that its command launches now; the benchmark quotes them."""
    third = 96 << 30
    for path in sorted(glob.glob(os.path.join(ROOT, "profiles", "outer_step_*_hbm_traffic.txt"))):
        text = open(path).read()
        command = re.search(r"-- python3 bench.py(.*)", text)[1].split()
        option = {name: value for name, value in zip(command, command[1:]) if name.startswith("--")}
        wl = workloads.make(option.get("--workload", "stage6p8b"))
        W, n = int(option.get("--workers", 0)) or wl.W, int(option.get("--subgroup", 0))
        spread = option.get("--placement", "spread") == "spread" and 1 << 30 <= W * wl.stride * 4 <= third
        sizes = sorted({n} if n else set(wl.n_schedule))
        calls = [(wl.theta_dtype == "bf16", third if spread else 0, (wl.segments, wl.stride, W, [k] * (W // k))) for k in sizes]
        want = {(k, bool(launch["phases"])) for k, got in zip(sizes, launches_of(calls)) for launch in got}
        names = re.findall(r"^outer_step_(fixed|held|phi_resident)<(\d+), .*?(Phased|InOrder)Args.*: fetched", text, re.M)
        up_to = {k: k if k <= 16 else -(-k // 8) * 8 for k in sizes}
        assert {(int(size), how == "Phased") for _, size, how in names} == {(up_to[k], phased) for k, phased in want}, path
