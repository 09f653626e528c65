"""Groups of different sizes that share one launch, against a call for every size alone: every bit of all three arrays, what no
run owns and who is in no group included. (Single sizes are compared with the oracle elsewhere.)"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2506_10911_amd as nl
import step_shapes as shapes

nl.library_path()          # loads libnoloco.so now; a missing library is an error, not a skip

RUNS = {"one run": [(5, 40 * 256 + 9)], "runs": [(0, 1), (2, 3), (255, 2), (300, 700), (1001, 256), (1280, 512), (1999, 9000)]}


@pytest.mark.parametrize("kind", list(RUNS))
@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sizes", [[1, 2], [2, 2, 3], [3, 1, 4, 2], [5, 4], [8, 7, 6, 5], [9, 8], [16, 15, 1], [10, 11, 12, 13, 14],
                                   [2] * 30 + [4], [2] * 31 + [3], [16, 17]])
def test_same_bits_as_size_by_size(sizes, theta_dtype, kind):
    """62 to 65 members are the table's end; 17 has a launch of its own."""
    same_bits(sizes, theta_dtype, RUNS[kind], shapes.stride_of(RUNS[kind]), sum(sizes) + 2)


@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("way,sizes,idle,segments", shapes.MIXED)
def test_stores_and_pacing(way, sizes, idle, segments, theta_dtype):
    """Shared launches whose results are kept in the memory's cache, written through, and that are paced."""
    segments, stride, W, sizes = shapes.mixed(sizes, idle, segments)
    same_bits(sizes, theta_dtype, segments, stride, W)


def same_bits(sizes, theta_dtype, segments, stride, W):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(W)
    phi = torch.empty((W, stride), device="cuda").normal_(0.0, 0.02, generator=gen)
    delta = torch.empty((W, stride), device="cuda").normal_(0.0, 1e-3, generator=gen)
    theta = (phi + 1e-3).to(torch.bfloat16 if theta_dtype == "bf16" else torch.float32)
    plan = nl.LaunchPlan(phi, delta, theta, stride, W, nl.BF16 if theta_dtype == "bf16" else nl.F32, segments)
    members = np.random.default_rng(W).permutation(W)[:sum(sizes)].astype(np.int32)
    offsets = np.cumsum([0] + sizes).astype(np.int32)
    together, alone = [[a.clone() for a in (phi, delta, theta)] for _ in range(2)]
    hp = (0.9, 0.7, 1.0)
    nl.outer_step(plan, *together, hp, members, offsets)
    for n in set(sizes):
        groups = [members[lo:hi] for lo, hi in zip(offsets[:-1], offsets[1:]) if hi - lo == n]
        nl.outer_step(plan, *alone, hp, np.concatenate(groups), np.arange(0, len(groups) * n + 1, n, dtype=np.int32))
    torch.cuda.synchronize()
    plan.destroy()
    for got, want, before in zip(together, alone, (phi, delta, theta)):
        as_int = torch.int16 if got.dtype == torch.bfloat16 else torch.int32
        assert torch.equal(got.view(as_int), want.view(as_int))
        assert not torch.equal(got[members[0]].view(as_int), before[members[0]].view(as_int))
