"""The binding's CPython module takes what ctypes took: any array-like of workers, any indexable of
coefficients, integers or objects with data_ptr(). No GPU: a null plan is refused before anything else."""
import numpy as np
import pytest

import paper_2506_10911_amd as nl

nl.library_path()          # loads libnoloco.so now; a missing library is an error, not a skip

NO_PLAN = (0, 64, 4, 0)


class Buffer:
    def data_ptr(self):
        return 4096


@pytest.mark.parametrize("hparams", [(.9, .7, 1.0), [.9, .7, 1], np.array([.9, .7, 1.0]), {0: .9, 1: .7, 2: 1.0}])
@pytest.mark.parametrize("members", [[0, 1], (0, 1), np.array([0, 1]), np.arange(4, dtype=np.int32)[::2], np.array([0, 1], dtype=">i4")])
def test_argument_kinds(hparams, members):
    for phi in (0, None, np.int64(4096), Buffer()):
        assert nl.binding._calls.outer_step(NO_PLAN, phi, Buffer(), 8192, hparams, members, [0, 2], 0) == 1


def test_bad_arguments_raise():
    calls = nl.binding._calls
    for args in [(0, 0, 0, (.9, .7), [0], [0, 1], 0), (0, 0, 0, "abc", [0], [0, 1], 0), ("x", 0, 0, (1, 1, 1), [0], [0, 1], 0),
                 (0, 0, 0, (1, 1, 1), ["a"], [0, 1], 0)]:
        with pytest.raises((IndexError, ValueError, TypeError)):
            calls.outer_step(NO_PLAN, *args)
    with pytest.raises(TypeError):
        calls.outer_step(NO_PLAN, 0)


def test_seeds_wrap_like_64_bit_integers():
    a, _ = nl.plan_groups(-1, 0, 8, 2)
    b, _ = nl.plan_groups(2**64 - 1, 0, 8, 2)
    assert a.tolist() == b.tolist()
