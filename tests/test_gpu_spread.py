"""GPU parity of noloco_replica_spread against the oracle: whole small arenas for every row-count
path, and the benchmark's full-size arena through small tensors the oracle can do exactly plus a
closed form that holds for every tensor."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from harness import segment_mask, theta_to_device

pytestmark = pytest.mark.gpu

import paper_2506_10911_amd as nl

nl.library_path()

# Primary check: the binary64 DEFINITION (oracle arithmetic 0), within a bound derived from the
# kernel's arithmetic.  Per element the kernel forms, in binary32 (unit roundoff u = 2^-24),
#   mean = (sum of W values) * (1/W),  v = (sum_w (x_w - mean)^2) * (1/W).
# (a) The W squared deviations are non-negative, so the roundings of dev (1), dev*dev (1), the W-1
#     additions and the final product with a rounded 1/W (2) give v a relative error of at most
#     (W + 4) u to first order; (W + 7) u leaves room for the second-order terms.
# (b) An error e in the mean shifts every deviation by the same amount; since the true deviations
#     sum to zero this adds exactly e^2 to v, with |e| <= (W + 1) u max|x| (W-1 additions of partial
#     sums up to W max|x|, then the rounded 1/W).
# Pooling over elements is binary64 on both sides (error ~1e-16 per term), so for a tensor with
# definition value s the kernel's figure lies within
#   sqrt(s^2 (1 + (W+7) u) + ((W+1) u max|x|)^2) - s      of s.
# Secondary check: the oracle's binary32-per-element mode, which repeats the kernel's element
# arithmetic and differs only in the binary64 pooling order: agreement to 1e-12 relative.
U32 = 2.0 ** -24
RTOL_SAME_ARITH = 1e-12


def definition_bound(ref, W, max_abs):
    """Largest |kernel - definition| the arithmetic above allows, per output entry."""
    ref = np.asarray(ref, dtype=np.float64)
    e = (W + 1) * U32 * max_abs
    return np.sqrt(ref * ref * (1.0 + (W + 7) * U32) + e * e) - ref + 1e-15


def max_abs_per_output(x_float, segs):
    """max |x| over each segment's elements (all rows), then over everything, as float64."""
    out = [float(np.abs(x_float[:, o:o + n]).max()) if n > 0 else 0.0 for o, n in segs]
    return np.array(out + [max(out) if out else 0.0])


def run_gpu(plan, x_dev, dtype, num_segments):
    out = torch.full((num_segments + 1,), -1.0, dtype=torch.float64, device="cuda")
    nl.replica_spread(plan, x_dev, dtype, out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("W", [1, 2, 3, 4, 5, 8, 16, 32, 48, 64, 100])
def test_small_arena(theta_dtype, W):
    wl = workloads.make_small(theta_dtype=theta_dtype, W=W, layout="gapped", total=120_000)
    S = wl.stride
    rng = np.random.default_rng(W)
    x = (np.tile(workloads.phi0_cpu(S, 3), (W, 1)) + workloads.drift_cpu((W, S), 3, W, 1e-3)).astype(np.float32)
    segs = list(wl.segments)
    order = rng.permutation(len(segs))
    segs = [segs[i] for i in order] + [(5, 0)]                      # scrambled order, one empty segment
    inside = segment_mask(wl)
    if theta_dtype == "bf16":
        xb = torch.from_numpy(x).to(torch.bfloat16)
        x_host = xb.view(torch.int16).numpy().view(np.uint16).copy()
        x_host[:, ~inside] = 0x7FC0                                # NaN canaries in the gaps
        x_dev = theta_to_device(x_host)
        dt = nl.BF16
    else:
        x_host = x.copy()
        x_host[:, ~inside] = np.nan
        x_dev = torch.from_numpy(x_host).cuda()
        dt = nl.F32
    plan = nl.LaunchPlan(x_dev, x_dev, x_dev, S, W, dt, segs)
    got = run_gpu(plan, x_dev, dt, len(segs))
    ref = oracle.replica_spread(x_host, segs, binary32=False)          # the definition
    same = oracle.replica_spread(x_host, segs, binary32=True)
    assert np.isfinite(got).all()
    x_float = torch.from_numpy(x).to(torch.bfloat16).float().numpy() if theta_dtype == "bf16" else x
    bound = definition_bound(ref, W, max_abs_per_output(x_float, segs))
    assert (np.abs(got - ref) <= bound).all(), (np.abs(got - ref) / bound).max()
    assert (bound[ref > 0] <= 6e-6 * ref[ref > 0]).all()              # the bound itself is tight: (W+7)u/2
    np.testing.assert_allclose(got, same, rtol=RTOL_SAME_ARITH, atol=0)
    assert got[len(segs) - 1] == 0.0                               # the empty segment
    again = run_gpu(plan, x_dev, dt, len(segs))
    assert np.array_equal(got.view(np.uint64), again.view(np.uint64))   # fixed pooling order


def spread_against_oracle(W, dtype, segs, stride, seed):
    rng = np.random.default_rng(seed)
    x = np.tile(rng.standard_normal(stride, dtype=np.float32) * np.float32(0.02), (W, 1))
    x += rng.standard_normal((W, stride), dtype=np.float32) * np.float32(1e-3)
    x_dev = torch.from_numpy(x).cuda()
    if dtype == "bf16":
        x_dev = x_dev.to(torch.bfloat16)
        x_host = x_dev.cpu().view(torch.int16).numpy().view(np.uint16)
        x = x_dev.float().cpu().numpy()
    else:
        x_host = x
    code = nl.BF16 if dtype == "bf16" else nl.F32
    plan = nl.LaunchPlan(x_dev, x_dev, x_dev, stride, W, code, segs)
    got = run_gpu(plan, x_dev, code, len(segs))
    ref = oracle.replica_spread(x_host, segs, binary32=False)
    bound = definition_bound(ref, W, max_abs_per_output(x, segs))
    assert (np.abs(got - ref) <= bound).all(), (np.abs(got - ref) / bound).max()
    np.testing.assert_allclose(got, oracle.replica_spread(x_host, segs, binary32=True), rtol=RTOL_SAME_ARITH, atol=0)
    again = run_gpu(plan, x_dev, code, len(segs))
    assert np.array_equal(got.view(np.uint64), again.view(np.uint64))
    plan.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("W", [6, 7, 9, 12, 13, 15, 17, 24, 25, 31, 33, 40, 41, 49, 56, 57, 63, 65])
def test_row_counts_between_the_kernels(W, dtype):
    """Every kind of row-count kernel: one per W up to 16, one per eight rows above (first, last and all
    of its conditional rows present), the first W beyond the registers. Tensors begin and end inside a
    vector and span several tiles."""
    segs = [(3, 1), (4, 2), (6, 1021), (1030, 2048), (3081, 7), (3100, 5000)]
    spread_against_oracle(W, dtype, segs, 8128, seed=W)


@pytest.mark.parametrize("W,dtype", [(3, "f32"), (5, "bf16"), (2, "f32"), (4, "bf16"), (8, "f32")])
def test_long_tensors_are_pooled_in_chunks(W, dtype):
    """Tensors on both sides of 2048 tiles, the longest one workgroup pools by itself, among many short
    and empty ones."""
    tile = 1024
    sizes = [2048 * tile, 5, 0, 2048 * tile + 1, 777, 2 * tile] + [31, 0, 64, 1500] * 30
    segs, at = [], 0
    for i, n in enumerate(sizes):
        segs.append((at, n))
        at += n + (i % 3)
    spread_against_oracle(W, dtype, segs, -(-at // 64) * 64, seed=W)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("W", [1, 2, 3, 4, 5, 8])
def test_few_rows(W, dtype):
    """Two and four vectors per thread: tensors that begin and end inside a vector, a wave, a tile, and whole tiles."""
    spread_against_oracle(W, dtype, [(3, 1), (4, 2), (6, 250), (256, 256), (513, 509), (1030, 2048), (3081, 7), (3100, 5000)], 8128, seed=W)


@pytest.mark.parametrize("W,dtype,columns", [(2, "bf16", 34_000_000), (2, "f32", 34_000_000), (1, "f32", 68_000_000), (8, "f32", 8_000_000),
                                             (12, "f32", 4_100_000), (4, "f32", 13_500_000), (7, "bf16", 16_000_000)])
def test_large_launches(W, dtype, columns):
    """Sizes from which two rows take tiles of 4096 columns, few rows longer runs per XCD, and launches are paced."""
    segs, at = [], 1
    for n in (columns // 2, 5, 4097, 1, columns // 3, 1023, columns - columns // 2 - columns // 3):
        segs.append((at, n))
        at += n + 2
    spread_against_oracle(W, dtype, segs, -(-at // 64) * 64, seed=W)


@pytest.mark.parametrize("W", [2, 4, 8])
def test_tiles_of_four_steps(W):
    """Tiles of 4096 columns, which W = 2, 4 and 8 take where the partial sums of smaller ones would not fit the static
    scratch: here because of two million empty tensors. Tensors begin and end in each of the four steps, inside vectors and
    between tiles, and span a few tiles; for W = 2 on both sides of 2048 tiles too. What no tensor owns is NaN."""
    sizes = [1, 3, 1021, 1024, 1025, 2047, 2048, 2051, 3071, 3073, 4095, 4096, 4097, 5119, 9000, 12289, 20001] * 3
    segs, at = [], 0
    if W == 2:
        segs = [(0, 2048 * 4096), (2048 * 4096, 2048 * 4096 + 1)]
        at = 2 * 2048 * 4096 + 1
    for i, n in enumerate(sizes):
        at += [0, 1, 1030, 2, 515, 7, 2055][i % 7]
        segs.append((at, n))
        at += n
    stride = -(-at // 64) * 64
    tiles = {t: sum((o + n - 1) // t - o // t + 1 for o, n in segs) for t in (1024, 4096)}
    scratch = 1 << 21                                   # doubles: tile sums, tensors, the overall sum
    empty = scratch - 1 - tiles[4096] - len(segs)
    assert tiles[1024] + len(segs) + empty + 1 > scratch
    rng = np.random.default_rng(W)
    x = rng.standard_normal((W, stride), dtype=np.float32) * np.float32(1e-3)
    x += rng.standard_normal(stride, dtype=np.float32) * np.float32(0.02)
    inside = np.zeros(stride, dtype=bool)
    for o, n in segs:
        inside[o:o + n] = True
    x[:, ~inside] = np.nan
    x32 = torch.from_numpy(x).cuda()
    plan = nl.LaunchPlan(x32, x32, x32, stride, W, nl.F32, segs + [(0, 0)] * empty)
    for x_dev, code in ((x32, nl.F32), (x32.to(torch.bfloat16), nl.BF16)):
        x_float = x_dev.float().cpu().numpy()
        x_host = x_float if code == nl.F32 else x_dev.cpu().view(torch.int16).numpy().view(np.uint16)
        ref = oracle.replica_spread(x_host, segs, binary32=False)
        same = oracle.replica_spread(x_host, segs, binary32=True)
        bound = definition_bound(ref, W, max_abs_per_output(x_float, segs))
        for spread in (nl.replica_spread, nl.replica_spread_noalloc):
            out = torch.full((len(segs) + empty + 1,), -1.0, dtype=torch.float64, device="cuda")
            spread(plan, x_dev, code, out)
            torch.cuda.synchronize()
            out = out.cpu().numpy()
            got = np.append(out[:len(segs)], out[-1])
            assert (np.abs(got - ref) <= bound).all(), (np.abs(got - ref) / bound).max()
            np.testing.assert_allclose(got, same, rtol=RTOL_SAME_ARITH, atol=0)
            assert (out[len(segs):-1] == 0).all()
    plan.destroy()


def test_more_tiles_than_the_static_scratch_holds():
    """Four rows of more than 2^21 tiles of 1024 columns: four of them to a partial sum, as the limit counts them.
    x_w[k] = w s(k) with s(k) a power of two drawn per column, so that everything is exact up to the pooled sums; the
    column between the two tensors is NaN."""
    S = (1 << 31) + (1 << 26)
    segs = [(0, S - 12345), (S - 12344, 12344)]
    x = torch.empty((4, S), dtype=torch.bfloat16, device="cuda")
    sums = [0.0, 0.0]
    for a in range(0, S, 1 << 27):
        b = min(a + (1 << 27), S)
        k = torch.arange(a, b, device="cuda")
        s = torch.exp2(-((k * 2654435761) >> 29 & 7).to(torch.float32))
        for i, (o, n) in enumerate(segs):
            lo, hi = max(a, o), min(b, o + n)
            if lo < hi:
                sums[i] += float(s[lo - a:hi - a].double().square().sum())
        for w in range(4):
            x[w, a:b] = w * s
    x[:, S - 12345] = float("nan")
    plan = nl.LaunchPlan(x, x, x, S, 4, nl.BF16, segs)
    want = np.sqrt(1.25 * np.array([sums[0] / (S - 12345), sums[1] / 12344, sum(sums) / (S - 1)]))
    out = torch.full((3,), -1.0, dtype=torch.float64, device="cuda")
    for spread in (nl.replica_spread, nl.replica_spread_noalloc):
        out.fill_(-1.0)
        spread(plan, x, nl.BF16, out)
        torch.cuda.synchronize()
        np.testing.assert_allclose(out.cpu().numpy(), want, rtol=RTOL_SAME_ARITH, atol=0)
    plan.destroy()
    del x
    torch.cuda.empty_cache()


@pytest.mark.parametrize("times", [5, 40])
def test_tensors_of_all_lengths_in_one_batch(times):
    """Tensors on both sides of the 64 tiles up to which eight lanes pool one, next to each other in a
    wave, empty ones among them, more than one batch of 32; few enough of the longer ones for a
    workgroup each, and more."""
    sizes = [64 * 1024, 64 * 1024 + 1, 0, 1, 70 * 1024, 1024, 1025, 66 * 1024] * times + [3] * 30
    segs, at = [], 0
    for n in sizes:
        segs.append((at, n))
        at += n
    spread_against_oracle(3, "f32", segs, -(-at // 64) * 64, seed=9)


def test_errors():
    x = torch.zeros((4, 64), device="cuda")
    out = torch.zeros(2, dtype=torch.float64, device="cuda")
    plan = nl.LaunchPlan(x, x, x, 64, 4, nl.F32, [(0, 64)])
    for fn, status in [(lambda: nl.replica_spread(plan, 0, nl.F32, out), 1),
                       (lambda: nl.replica_spread(plan, x, nl.F32, 0), 1),
                       (lambda: nl.replica_spread(plan, x, 5, out), 2),
                       (lambda: nl.replica_spread(plan, x.data_ptr() + 64, nl.F32, out), 5)]:
        with pytest.raises(nl.NolocoError) as e:
            fn()
        assert e.value.status == status
    empty = nl.LaunchPlan(x, x, x, 64, 4, nl.F32, [])
    nl.replica_spread(empty, x, nl.F32, out)
    torch.cuda.synchronize()
    assert float(out[0]) == 0.0


@pytest.mark.parametrize("name,dtype", [("stage6p8b", "f32"), ("stage6p8b", "bf16"), ("ragged_gapped", "f32")])
def test_full_size(name, dtype):
    """The benchmark arena at full size, as float and (the fast weights' storage) as bf16.
    (1) After a fake inner phase: every small tensor (<= 2^16 elements, all W rows) is recomputed by
    the oracle's binary64 definition and must match within the derived bound, and the binary32-per-
    element mode to 1e-12; the overall figure must equal the pooling of the per-tensor figures.
    (2) Rows set to an arithmetic progression x_w = x_0 + w d: every tensor and the total must give
    d sqrt((W^2 - 1) / 12)."""
    wl = workloads.make(name)
    W, S = wl.W, wl.stride
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    item = 4 if dtype == "f32" else 2
    assert W * S * (item + 4.0 / W) * 1.02 + (2 << 30) <= free, \
        f"{name} must fit: {W * S * item / 1e9:.0f} GB needed, {free / 1e9:.0f} GB free"
    print(f"[case] {name} {dtype}: W={W} P={wl.P}", flush=True)
    tdt, code = (torch.float32, nl.F32) if dtype == "f32" else (torch.bfloat16, nl.BF16)
    x = torch.empty((W, S), dtype=tdt, device="cuda")
    row0 = torch.empty((1, S), dtype=torch.float32, device="cuda")
    workloads.fill_phi0_device(row0, wl.seed, wl.init_std)
    for w in range(W):                                                   # common start + drift, row by row
        workloads.fake_inner_phase_device(x[w:w + 1], row0, wl.seed, w, wl.sigma)
    plan = nl.LaunchPlan(x, x, x, S, W, code, wl.segments)
    got = run_gpu(plan, x, code, len(wl.segments))
    small = [i for i, (_, n) in enumerate(wl.segments) if n <= (1 << 16)][:200]
    assert len(small) >= 40
    for i in small:
        o, n = wl.segments[i]
        piece = x[:, o:o + n].cpu()
        host = piece.view(torch.int16).numpy().view(np.uint16) if dtype == "bf16" else piece.numpy()
        host = np.ascontiguousarray(host)
        ref = oracle.replica_spread(host, binary32=False)[-1]
        bound = definition_bound(ref, W, float(piece.float().abs().max()))
        assert abs(got[i] - ref) <= bound, (i, wl.tensors[i], got[i], ref, bound)
        same = oracle.replica_spread(host, binary32=True)[-1]
        assert got[i] == pytest.approx(same, rel=RTOL_SAME_ARITH), (i, wl.tensors[i])
    numel = np.array([n for _, n in wl.segments], dtype=np.float64)
    pooled = np.sqrt((got[:-1] ** 2 * numel).sum() / numel.sum())
    assert got[-1] == pytest.approx(pooled, rel=1e-12)
    # drift N(0, sigma^2) on top of a common start: population variance over W draws is sigma^2 (W-1)/W
    # (bf16 storage adds rounding noise of about half a percent of that variance)
    expect = wl.sigma * np.sqrt((W - 1) / W)
    assert got[-1] == pytest.approx(expect, rel=2e-3 if dtype == "f32" else 2e-2)
    d = 1.0 / 1024
    if dtype == "bf16":
        x[0].fill_(0.5)            # 0.5 + w / 128 is exact in bf16 for every w < 64
        d = 1.0 / 128
    for w in range(1, W):
        x[w].copy_(x[0])
        x[w].add_(w * d)
    got = run_gpu(plan, x, code, len(wl.segments))
    want = d * np.sqrt((W * W - 1) / 12.0)
    np.testing.assert_allclose(got, want, rtol=2e-4)               # x_0 + w d rounds in binary32
    print(f"[done] {name} {dtype}", flush=True)
    plan.destroy()
    del x, row0
    torch.cuda.empty_cache()
