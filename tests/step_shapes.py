"""Arenas and groups that reach a given way of launching the outer step. The GPU tests run them; test_step_routes.py asks the
library's host code, on the CPU, which launches they get."""
KINDS = ("one run", "runs")

# Next to each other. Group size: classes and the rounds of them that a launch in phases has to have, as (float, bf16).
PHASED = {4: ((16, 48), (16, 48)), 5: ((8, 20), (16, 12)), 6: ((8, 20), (16, 12)), 7: ((8, 20), (16, 12)), 8: ((4, 20), (8, 12)),
          9: ((4, 10), (8, 8)), 10: ((4, 10), (8, 8)), 11: ((4, 10), (8, 8)), 12: ((4, 10), (8, 8)), 13: ((4, 10), (8, 8)), 14: ((4, 10), (8, 8)),
          15: ((4, 10), (8, 8)), 16: ((8, 20), (8, 8)), 17: ((4, 5), (8, 6)), 24: ((8, 20), (8, 6)), 25: ((4, 5), (4, 5)), 33: ((4, 5), (4, 5)),
          40: ((4, 5), (4, 5)), 41: ((4, 5), (4, 5)), 56: ((4, 5), (4, 5))}
# Far apart: size, classes, rounds.
FAR_APART = 64 << 30
PHASED_FAR_APART = ((2, 32, 60), (3, 32, 60), (8, 8, 60), (16, 8, 30), (24, 8, 30))


def stride_of(segments):
    return -(-(segments[-1][0] + segments[-1][1]) // 64) * 64


def pieces_of(kind, pieces):
    """About so many pieces of 256 columns: one run with odd ends, or runs of 500 pieces, few enough for groups of four."""
    if kind == "one run":
        return [(77, pieces * 256 - 3)]
    segments, at = [], 3
    for i in range(pieces // 500 + 1):
        segments.append((at, (500 * 256) | 1))
        at += segments[-1][1] + 1 + i % 7
    return segments


def phased(n, bf16, kind):
    """(segments, stride, W, group sizes): one worker is in no group."""
    classes, rounds = PHASED[n][bf16]
    groups = 3 if n <= 8 else 1
    segments = pieces_of(kind, -(-(classes * 256 * rounds + 300) // groups))
    return segments, stride_of(segments) + (64 if n % 2 else 0), groups * n + 1, [n] * groups


def phased_far_apart(n, classes, rounds, kind):
    segments = pieces_of(kind, classes * 256 * rounds + 2)
    return segments, -(-stride_of(segments) // 256) * 256, n, [n]


# Phi and delta in registers without phases: up to 1024 pieces, and one more in the last.
HELD = ([(0, 512 * 256)], [(1, 511 * 256)], [(0, 3), (255, 2), (300, 5000), (5307, 256 * 8)], [(1, 512 * 256)])
HELD_SIZES = (17, 24, 25, 32, 33, 40, 41, 48)

# Columns of one run that a group of 17 takes through the kernel that holds delta, without phases and with them.
NARROWED = (1024 * 256, 1 << 26)

# Groups of different sizes in one launch: kept in the memory's cache, written through, and written through and paced. Sizes that
# one pacing does not suit share small launches only: with workers in no group the arena is large enough to be written through.
MIXED = (("kept", [2, 2, 3], 2, [(5, 40_000)]), ("kept", [16, 3, 9], 2, [(5, 17_000), (17_100, 16_500)]),
         ("through", [1, 2], 6, [(3, 900_000)]), ("through", [9, 16, 2], 42, [(3, 50_001), (50_010, 50_000)]),
         ("paced", [2, 2, 3], 2, [(3, 2_000_000), (2_000_100, 9_001)]), ("paced", [5, 6, 7], 2, [(77, 500_001), (500_100, 500_000)]),
         ("paced", [4, 4, 7], 2, [(1, 900_000)]))


def mixed(sizes, idle, segments):
    return segments, stride_of(segments), sum(sizes) + idle, sizes
