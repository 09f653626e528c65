"""The binding's CPython module takes what ctypes took: any array-like of workers, any indexable of
coefficients, integers or objects with data_ptr(). No GPU: a null plan is refused before anything else."""
import ctypes as C
import importlib.util
import shutil

import numpy as np
import pytest
import torch

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


# ---- what reaches the library: a second copy of the module, bound to stand-ins that record their arguments ----
STEP = C.CFUNCTYPE(C.c_int, C.c_void_p, C.POINTER(nl.binding._Arena), C.POINTER(nl.binding._HParams), C.POINTER(C.c_int32),
                   C.POINTER(C.c_int32), C.c_int32, C.c_void_p)
SPREAD = C.CFUNCTYPE(C.c_int, C.c_void_p, C.c_void_p, C.c_int32, C.c_void_p, C.c_void_p)
PLAN = C.CFUNCTYPE(C.c_int, C.c_uint64, C.c_uint64, C.c_int32, C.c_int32, C.POINTER(C.c_int32), C.POINTER(C.c_int32))


@pytest.fixture(scope="module")
def recorded(tmp_path_factory):
    copy = str(tmp_path_factory.mktemp("calls") / "_calls.so")
    shutil.copy(nl.binding._calls.__file__, copy)
    spec = importlib.util.spec_from_file_location("_calls", copy)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    assert module is not nl.binding._calls
    seen = []

    def step(plan, arena, hp, members, offsets, groups, stream):
        a, h = arena.contents, hp.contents
        offsets = offsets[:groups + 1] if groups >= 0 else []
        seen.append(dict(plan=plan, phi=a.phi, delta=a.delta, theta=a.theta, stride=a.worker_stride, W=a.W, dtype=a.theta_dtype,
                         hp=(h.alpha, h.beta, h.gamma), members=members[:offsets[-1]] if offsets else [], offsets=offsets,
                         groups=groups, stream=stream))
        return 7

    def spread(plan, x, x_dtype, out, stream):
        seen.append((plan, x, x_dtype, out, stream))
        return 3

    def plan_groups(seed, at, W, n, members, offsets):
        seen.append((seed, at, W, n))
        members[W - 1], offsets[W // n] = 41, 42
        return 0

    stubs = [PLAN(plan_groups), STEP(step), SPREAD(spread), SPREAD(lambda *args: spread(*args) + 1)]
    module.bind(*(C.cast(f, C.c_void_p).value for f in stubs), nl.binding._int32)
    yield module, seen, stubs


class Pointer:
    def __init__(self, value):
        self.value = value

    def data_ptr(self):
        return self.value


class IntegerWithBuffer(int):
    def data_ptr(self):
        return 1 << 41


HP = [(.9, .7, 1.0), [.9, .7, 1], np.array([.9, .7, 1.0]), {0: .9, 1: .7, 2: 1.0}, np.array([.9, .7, 1.0], dtype=np.float32),
      torch.tensor([.9, .7, 1.0]), ("0.9", "0.7", 1)]
MEMBERS = [[3, 0, 2], (3, 0, 2), np.array([3, 0, 2]), np.array([3, 9, 0, 9, 2, 9], dtype=np.int32)[::2],
           np.array([3, 0, 2], dtype=">i4"), np.array([3., 0., 2.]), np.array([3, 0, 2], dtype=np.uint8), torch.tensor([3, 0, 2]),
           np.frombuffer(b"\0" + np.array([3, 0, 2], dtype=np.int32).tobytes(), dtype=np.uint8)[1:].view(np.int32)]


@pytest.mark.parametrize("hparams", HP, ids=range(len(HP)))
@pytest.mark.parametrize("members", MEMBERS, ids=range(len(MEMBERS)))
def test_step_arguments_reach_the_library(recorded, hparams, members):
    module, seen, _ = recorded
    for offsets in ([0, 2, 3], np.array([0, 2, 3], dtype=np.int32), np.array([0, 2, 3], dtype=">i8")):
        assert module.outer_step((123, 1 << 33, 4, 1), 1 << 40, Pointer(2 << 40), np.int64(3 << 40), hparams, members, offsets, 55) == 7
        got = seen.pop()
        assert (got["plan"], got["phi"], got["delta"], got["theta"], got["stream"]) == (123, 1 << 40, 2 << 40, 3 << 40, 55)
        assert (got["stride"], got["W"], got["dtype"]) == (1 << 33, 4, 1)
        assert got["hp"] == tuple(np.float32([.9, .7, 1.0]).tolist())
        assert got["members"] == [3, 0, 2] and got["offsets"] == [0, 2, 3] and got["groups"] == 2


@pytest.mark.parametrize("value", [1 << 40, np.int64(1 << 40), float(1 << 40), str(1 << 40)])
def test_what_data_ptr_returns_is_made_an_integer(recorded, value):
    module, seen, _ = recorded
    assert module.replica_spread((9, 0, 0, 0), Pointer(value), 1, Pointer(2 << 40), 0) == 3
    assert seen.pop() == (9, 1 << 40, 1, 2 << 40, None)


def test_spread_arguments_reach_the_library(recorded):
    module, seen, _ = recorded
    assert module.replica_spread_noalloc((9, 64, 4, 0), None, 0, IntegerWithBuffer(5), 8) == 4      # data_ptr() goes first
    assert seen.pop() == (9, None, 0, 1 << 41, 8)
    assert nl.binding._ptr(IntegerWithBuffer(5)) == 1 << 41


def test_plan_arguments_reach_the_library(recorded):
    module, seen, _ = recorded
    members, offsets = np.zeros(6, dtype=np.int32), np.zeros(4, dtype=np.int32)
    assert module.plan_groups(2**64 - 1, 5, 6, 2, members, offsets) == 0
    assert seen.pop() == (2**64 - 1, 5, 6, 2) and members[5] == 41 and offsets[3] == 42
