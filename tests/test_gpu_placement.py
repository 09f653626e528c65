"""GPU parity of the outer step over the ways its results are stored and its pieces are ordered: arrays next to each
other and far apart, results kept in the memory's cache (up to 64 MiB of state) and written through it, runs that
end inside pieces. Whole arenas, bit for bit against the oracle."""
import pytest
import torch

import workloads
from harness import SmallCase

pytestmark = pytest.mark.gpu

import paper_2506_10911_amd as nl

nl.library_path()          # loads libnoloco.so now; a missing library is an error, not a skip

FAR = 64 << 30             # bytes between the arrays from which they count as far apart


class Placed(SmallCase):
    """The same arena with its arrays carved out of one block, FAR bytes from each other."""

    def __init__(self, wl):
        super().__init__(wl, nl)
        rows = self.d_phi.numel() * 4
        block = torch.empty(2 * FAR + rows, dtype=torch.uint8, device="cuda")

        def carve(i, like):
            at = block[i * FAR:i * FAR + like.numel() * like.element_size()].view(like.dtype).view(like.shape)
            at.copy_(like)
            return at

        self.d_phi, self.d_delta, self.d_theta = (carve(i, t) for i, t in enumerate((self.d_phi, self.d_delta, self.d_theta)))
        self.plan = nl.LaunchPlan(self.d_phi, self.d_delta, self.d_theta, wl.stride, wl.W,
                                  nl.F32 if wl.theta_dtype == "f32" else nl.BF16, wl.segments)


@pytest.mark.parametrize("theta_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 16])
@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("kept", [True, False])
def test_placement_and_stores(n, theta_dtype, far, kept):
    W = max(n, 8 // n * n)
    columns = (66_000_000 if kept else 70_000_000) // (W * (12 if theta_dtype == "f32" else 10))
    # a long run, then shorter and shorter ones: whole pieces and both kinds of edges
    segments, at = [(5, columns // 2)], 5 + columns // 2 + 3
    for size in (columns // 4, 4097, 1023, 256, 255, 3, 1, columns // 8):
        segments.append((at, size))
        at += size + 1 + size % 7
    if not kept:           # more elements than the limit allows
        segments.append((at, columns - sum(m for _, m in segments)))
    wl = workloads.Workload("placed", [(f"t{i}", m) for i, (_, m) in enumerate(segments)], segments, W=W,
                            theta_dtype=theta_dtype, n_schedule=(1,), sigma=1e-3, steps=1, seed=n)
    case = Placed(wl) if far else SmallCase(wl, nl)
    for step in range(2):
        case.inner_phase(step)
        members, offsets = nl.plan_groups(n, step, W, n)
        case.step(step, members, offsets)
        case.check(f"n={n} {theta_dtype} far={far} kept={kept} step {step}")
