"""Launches in phases (large launches of groups of 4 to 56, far apart of 2 to 48) against the same step
without them (nontemporal = 1 takes the paced launch, which other tests compare with the oracle): every bit of all three
arrays, what no run owns included. (test_step_routes.py checks that these arenas are launched in phases.) Small launches with
delta in registers against the kernel without it, and the narrowing of bf16 fast weights against its definition on the bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2506_10911_amd as nl
import step_shapes as shapes

nl.library_path()          # loads libnoloco.so now; a missing library is an error, not a skip


def arena(W, stride, dtype, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    phi = torch.empty((W, stride), device="cuda").normal_(0.0, 0.02, generator=gen)
    delta = torch.empty((W, stride), device="cuda").normal_(0.0, 1e-3, generator=gen)
    theta = (phi + torch.empty(stride, device="cuda").normal_(0.0, 1e-3, generator=gen)).to(dtype)
    return [phi, delta, theta]


@pytest.mark.parametrize("kind", shapes.KINDS)
@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", list(shapes.PHASED))
def test_same_bits_as_without_phases(n, theta_dtype, kind):
    bf16 = theta_dtype == "bf16"
    segments, stride, W, sizes = shapes.phased(n, bf16, kind)
    groups = len(sizes)
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


@pytest.mark.parametrize("kind", shapes.KINDS)
@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,classes,rounds", shapes.PHASED_FAR_APART)
def test_same_bits_far_apart(n, classes, rounds, theta_dtype, kind):
    """Arrays 64 GiB from each other, where groups of two and three have phases too."""
    dtype = torch.bfloat16 if theta_dtype == "bf16" else torch.float32
    segments, stride, W, sizes = shapes.phased_far_apart(n, classes, rounds, kind)
    apart = shapes.FAR_APART
    slab = torch.empty(2 * apart + n * stride * 4, dtype=torch.uint8, device="cuda")
    start = arena(n, stride, dtype, seed=n)
    before = [a[0].clone() for a in start]
    far = [slab[i * apart:i * apart + a.numel() * a.element_size()].view(a.dtype).view(a.shape).copy_(a) for i, a in enumerate(start)]
    for state, knobs in ((far, None), (start, dict(nontemporal=1))):
        plan = nl.LaunchPlan(*state, stride, n, nl.BF16 if theta_dtype == "bf16" else nl.F32, segments)
        if knobs:
            plan.tune(**knobs)
        nl.outer_step(plan, *state, (0.9, 0.7, 1.0), list(range(n)), [0, n])
        torch.cuda.synchronize()
        plan.destroy()
    for got, want, old in zip(far, start, before):
        as_int = torch.int16 if got.dtype == torch.bfloat16 else torch.int32
        assert torch.equal(got.view(as_int), want.view(as_int))
        assert not torch.equal(got[0].view(as_int), old.view(as_int))


@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", shapes.HELD_SIZES)
def test_same_bits_with_delta_in_registers(n, theta_dtype):
    """Launches of 17 to 48 members of up to one wave a SIMD (1024 pieces), and of 1026, against the kernel that knobs ask for."""
    dtype = torch.bfloat16 if theta_dtype == "bf16" else torch.float32
    for segments in shapes.HELD:
        W = 2 * n
        stride = shapes.stride_of(segments)
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


def narrowed(bits):
    """bf16 bits of binary32 bits: to nearest, ties to even, NaN kept as a quiet one."""
    low = bits & 0xFFFFFFFF
    nan = (low & 0x7FFFFFFF) > 0x7F800000
    return torch.where(nan, (low >> 16) | 0x40, (low + 0x7FFF + ((low >> 16) & 1)) >> 16)


# Groups of equal members: with phi = theta = 0, alpha = 1 and beta = gamma = 0 every member's phi' is its delta (a signalling NaN
# comes out quiet, -0 as +0), so that theta' = narrow(phi') for any pattern. 17 members have the hardware's conversion, in a
# launch of up to 1024 pieces without phases and in a large one with them; one member has the integer form.
@pytest.mark.parametrize("n,columns", [(1, 1 << 26), (17, shapes.NARROWED[0]), (17, shapes.NARROWED[1])])
def test_narrowing_is_to_nearest_even(n, columns):
    """All 2^32 bit patterns in launches of 2^26 columns; in the small launch those around every tie."""
    if columns < 1 << 26:
        halves = torch.arange(0, 1 << 16, device="cuda", dtype=torch.int64) << 16
        chunks = [(halves[:, None] + torch.tensor(low, device="cuda")).reshape(-1)
                  for low in ([0, 1, 0x7FFF, 0x8000], [0x8001, 0xFFFF, 0x4000, 0xC000])]
    else:
        chunks = (torch.arange(at, at + columns, device="cuda", dtype=torch.int64) for at in range(0, 1 << 32, columns))
    phi, delta = torch.empty((n, columns), device="cuda"), torch.empty((n, columns), device="cuda")
    theta = torch.empty((n, columns), device="cuda", dtype=torch.bfloat16)
    plan = nl.LaunchPlan(phi, delta, theta, columns, n, nl.BF16, [(0, columns)])
    quiet = infinite = small = 0
    for bits in chunks:
        phi.zero_(), theta.zero_()
        delta.view(torch.int32)[:] = bits.to(torch.int32)
        nl.outer_step(plan, phi, delta, theta, (1.0, 0.0, 0.0), list(range(n)), [0, n])
        got = phi.view(torch.int32)[0].to(torch.int64) & 0xFFFFFFFF
        nan = (bits & 0x7FFFFFFF) > 0x7F800000
        arrived = torch.where(nan, bits | 0x400000, torch.where(bits == 0x80000000, 0, bits))
        assert torch.equal(got, arrived)
        want = narrowed(got).to(torch.int16)
        assert all(torch.equal(row, want) for row in theta.view(torch.int16))
        quiet += int(nan.sum())
        infinite += int(((bits & 0x7FFFFFFF) == 0x7F800000).sum())
        small += int(((bits & 0x7FFFFFFF) < 0x800000).sum())
    plan.destroy()
    assert infinite == 2 and quiet > 1000 and small > 1000
