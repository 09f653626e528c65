"""GPU parity of the outer step over every kind of kernel and launch: subgroup sizes at the edges of the
kernels' ranges, arenas of one run (odd start and end) and of many, launches below and above the size
from which they are paced. Whole arenas, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from harness import SmallCase

pytestmark = pytest.mark.gpu

import paper_2506_10911_amd as nl

nl.library_path()          # loads libnoloco.so now; a missing library is an error, not a skip


def workload(theta_dtype, W, segments, seed):
    wl = workloads.Workload("shapes", [(f"t{i}", n) for i, (_, n) in enumerate(segments)], segments, W=W,
                            theta_dtype=theta_dtype, n_schedule=(1,), sigma=1e-3, steps=1, seed=seed)
    return wl


def one_step(theta_dtype, W, n, segments, seed):
    case = SmallCase(workload(theta_dtype, W, segments, seed), nl)
    rng = np.random.default_rng(seed)
    S = case.wl.stride
    for arr, dev, std in ((case.phi, case.d_phi, 1e-3), (case.delta, case.d_delta, 1e-3)):
        arr += rng.standard_normal((W, S), dtype=np.float32) * np.float32(std)       # NaN canaries stay NaN
        dev.copy_(torch.from_numpy(arr))
    case.inner_phase(0)
    members, offsets = nl.plan_groups(seed, 0, W, n)
    case.step(0, members, offsets)
    case.check(f"W={W} n={n} {theta_dtype}, {len(segments)} segments, {case.wl.P} elements")


def runs_of(total, pieces, seed):
    """`pieces` runs of odd sizes around total / pieces with 1..9 unowned elements between them."""
    rng = np.random.default_rng(seed)
    segs, at = [], 3
    for _ in range(pieces):
        size = int(max(1, rng.integers(1, max(2, 2 * total // pieces))))
        segs.append((at, size))
        at += size + int(rng.integers(1, 10))
    return segs


SIZES = [1, 2, 3, 5, 7, 9, 10, 11, 12, 13, 14, 15, 16, 17, 24, 25, 32, 33, 40, 41, 48, 49, 56, 57, 63, 64, 65, 100]


@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", SIZES)
def test_subgroup_sizes(n, theta_dtype):
    one_step(theta_dtype, 2 * n, n, [(1, 2 * 256 - 2)], seed=n)                     # one run inside two pieces
    one_step(theta_dtype, 2 * n, n, [(0, 1), (2, 2), (5, 255), (261, 512), (1021, 3), (1030, 700)], seed=n + 1)


@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [1, 2, 3, 8, 16, 20, 64, 70])
@pytest.mark.parametrize("pieces", [1, 200])
def test_paced_launches(n, theta_dtype, pieces):
    """State of 50 MB and more in one launch, enough for it to be paced up to n = 16."""
    W = max(n, 8 // n * n)
    total = {8: 110_000_000, 16: 210_000_000}.get(n, 56_000_000) // (W * (12 if theta_dtype == "f32" else 10)) | 1
    segments = [(5, total)] if pieces == 1 else runs_of(total, pieces, seed=n)
    if pieces > 1:
        segments.append((segments[-1][0] + segments[-1][1] + 4, total // 4 | 1))
    one_step(theta_dtype, W, n, segments, seed=n)


@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,W", [(2, 16), (8, 16), (16, 16)])
def test_many_runs_shorter_than_a_piece(n, W, theta_dtype):
    """Runs of 65 elements on average: more waves share a CU than with whole pieces; n = 2 is not paced."""
    one_step(theta_dtype, W, n, runs_of(520_000, 8000, seed=n), seed=n)


@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
def test_run_boundaries_inside_cells(theta_dtype):
    """Runs shorter than a piece, of exactly one piece, and long ones between them."""
    segs, at = [], 0
    for i, size in enumerate([1, 1, 5, 256, 256, 9000, 2, 255, 257, 3, 20_000, 64, 1] * 6):
        at += 1 + (i * 37) % 11
        if size == 256:
            at = -(-at // 256) * 256
        segs.append((at, size))
        at += size
    one_step(theta_dtype, 8, 4, segs, seed=5)
