"""Launches in phases (large launches of groups of 4 to 56, far apart of 2 to 48) against the same step
without them (nontemporal = 1 takes the paced launch, which other tests compare with the oracle): every bit of all three
arrays, what no run owns included. Small launches with delta in registers against the kernel without it, and the narrowing of bf16 fast weights, against torch's."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2506_10911_amd as nl

nl.library_path()          # loads libnoloco.so now; a missing library is an error, not a skip


# group size: classes and the rounds of them that a launch has to have, as (float, bf16)
LAUNCHES = {4: ((16, 48), (16, 48)), 5: ((8, 20), (16, 12)), 8: ((4, 20), (8, 12)), 12: ((4, 10), (8, 8)), 16: ((8, 20), (8, 8)),
            17: ((4, 5), (8, 6)), 24: ((8, 20), (8, 6)), 25: ((4, 5), (4, 5)), 41: ((4, 5), (4, 5)), 56: ((4, 5), (4, 5))}


def arena(W, stride, dtype, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    phi = torch.empty((W, stride), device="cuda").normal_(0.0, 0.02, generator=gen)
    delta = torch.empty((W, stride), device="cuda").normal_(0.0, 1e-3, generator=gen)
    theta = (phi + torch.empty(stride, device="cuda").normal_(0.0, 1e-3, generator=gen)).to(dtype)
    return [phi, delta, theta]


@pytest.mark.parametrize("kind", ["one run", "runs"])
@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", list(LAUNCHES))
def test_same_bits_as_without_phases(n, theta_dtype, kind):
    bf16 = theta_dtype == "bf16"
    classes, rounds = LAUNCHES[n][bf16]
    groups = 3 if n <= 8 else 1
    pieces = -(-(classes * 256 * rounds + 300) // groups)
    if kind == "one run":
        segments = [(77, pieces * 256 - 3)]
    else:                                   # few enough for groups of four: one run in 500 pieces, odd ends, gaps of 1 to 7
        segments, at = [], 3
        for i in range(pieces // 500 + 1):
            segments.append((at, (500 * 256) | 1))
            at += segments[-1][1] + 1 + i % 7
    W = groups * n + 1                      # one worker is in no group
    stride = -(-(segments[-1][0] + segments[-1][1]) // 64) * 64 + (64 if n % 2 else 0)
    arrays = arena(W, stride, torch.bfloat16 if bf16 else torch.float32, seed=n)
    plain = [a.clone() for a in arrays]
    members = [w * groups + g for g in range(groups) for w in range(n)]
    offsets = [g * n for g in range(groups + 1)]
    dtype = nl.BF16 if bf16 else nl.F32
    for state, knobs in ((arrays, None), (plain, dict(nontemporal=1))):
        plan = nl.LaunchPlan(*state, stride, W, dtype, segments)
        if knobs:
            plan.tune(**knobs)
        nl.outer_step(plan, *state, (0.9, 0.7, 1.0), members, offsets)
        torch.cuda.synchronize()
        plan.destroy()
    start = arena(W, stride, torch.bfloat16 if bf16 else torch.float32, seed=n)
    for got, want, before in zip(arrays, plain, start):
        as_int = torch.int16 if got.dtype == torch.bfloat16 else torch.int32
        assert torch.equal(got.view(as_int), want.view(as_int))
        assert not torch.equal(got[0].view(as_int), before[0].view(as_int))
        assert torch.equal(got[W - 1].view(as_int), before[W - 1].view(as_int))          # the worker in no group


@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,classes,rounds", [(2, 32, 60), (3, 32, 60), (8, 8, 60), (16, 8, 30)])
def test_same_bits_far_apart(n, classes, rounds, theta_dtype):
    """Arrays 64 GiB from each other, where groups of two and three have phases too."""
    dtype = torch.bfloat16 if theta_dtype == "bf16" else torch.float32
    total = (classes * 256 * rounds + 1) * 256 - 9
    stride = -(-(total + 5) // 256) * 256
    slab = torch.empty((128 << 30) + n * stride * 4, dtype=torch.uint8, device="cuda")
    start = arena(n, stride, dtype, seed=n)
    far = [slab[i << 36:(i << 36) + a.numel() * a.element_size()].view(a.dtype).view(a.shape).copy_(a) for i, a in enumerate(start)]
    for state, knobs in ((far, None), (start, dict(nontemporal=1))):
        plan = nl.LaunchPlan(*state, stride, n, nl.BF16 if theta_dtype == "bf16" else nl.F32, [(5, total)])
        if knobs:
            plan.tune(**knobs)
        nl.outer_step(plan, *state, (0.9, 0.7, 1.0), list(range(n)), [0, n])
        torch.cuda.synchronize()
        plan.destroy()
    for got, want in zip(far, start):
        as_int = torch.int16 if got.dtype == torch.bfloat16 else torch.int32
        assert torch.equal(got.view(as_int), want.view(as_int))


@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [17, 24, 25, 40, 41, 48])
def test_same_bits_with_delta_in_registers(n, theta_dtype):
    """Launches of 17 to 48 members of up to one wave a SIMD (1024 pieces) against the kernel that knobs ask for."""
    dtype = torch.bfloat16 if theta_dtype == "bf16" else torch.float32
    for segments in ([(0, 512 * 256)], [(1, 512 * 256)], [(0, 3), (255, 2), (300, 5000), (5307, 256 * 8)]):
        W = 2 * n
        stride = -(-(segments[-1][0] + segments[-1][1]) // 64) * 64
        arrays = arena(W, stride, dtype, seed=n)
        plain = [a.clone() for a in arrays]
        members, offsets = nl.plan_groups(3, n, W, n)
        for state, knobs in ((arrays, None), (plain, dict(group_major=1))):
            plan = nl.LaunchPlan(*state, stride, W, nl.BF16 if theta_dtype == "bf16" else nl.F32, segments)
            if knobs:
                plan.tune(**knobs)
            nl.outer_step(plan, *state, (0.9, 0.7, 1.0), members, offsets)
            torch.cuda.synchronize()
            plan.destroy()
        for got, want in zip(arrays, plain):
            as_int = torch.int16 if got.dtype == torch.bfloat16 else torch.int32
            assert torch.equal(got.view(as_int), want.view(as_int))


def test_narrowing_is_to_nearest_even():
    """A group of one with all coefficients 0 gives theta' = narrow(phi): a stride through all finite bit patterns, and
    the patterns around every tie of a few exponents."""
    spread = torch.arange(0, 1 << 32, 509, dtype=torch.int64)
    ties = ((torch.arange(0, 1 << 16, dtype=torch.int64) << 16)[:, None] + torch.tensor([0x7FFF, 0x8000, 0x8001])).reshape(-1)
    bits = torch.cat([spread, ties])
    bits = bits[(bits & 0x7F800000) != 0x7F800000]
    bits = bits[: bits.numel() // 64 * 64]
    phi = bits.to(torch.int32).view(torch.float32).cuda()[None, :].contiguous()
    want = (phi + 0.0).to(torch.bfloat16)          # -0 + 0 is +0 in the step too
    delta, theta = torch.zeros_like(phi), torch.zeros_like(want)
    S = phi.shape[1]
    plan = nl.LaunchPlan(phi, delta, theta, S, 1, nl.BF16, [(0, S)])
    nl.outer_step(plan, phi, delta, theta, (0.0, 0.0, 0.0), [0], [0, 1])
    torch.cuda.synchronize()
    plan.destroy()
    assert torch.equal(theta.view(torch.int16), want.view(torch.int16))
