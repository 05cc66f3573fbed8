"""The plan that a dispatch makes for the grouped GEMMs of its call (CPU: the
kernel source run block by block)."""
import ctypes

import numpy as np
import pytest

from tests import _hip_host
from tests.test_gpu_gemm_shapes import CASES, FORWARDS

WORDS, PLAN = 16, 9  # words per GEMM in the schedule area, and before its plan
HEIGHTS = (32, 64, 128, 256)


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return _hip_host.compile_host("plan", tmp_path_factory.mktemp("hip_host"))


def _p(a):
    return ctypes.c_void_p(a.ctypes.data)


def _one_block(lib, ids, ert, alive0, alive1, S, d=1024, I=512, grid=256):
    T, k = ids.shape
    i32 = lambda n: np.full(n, -7, np.int32)
    out = dict(counts=i32(S), offsets=i32(S + 1), slot=i32((T, k)), perm=i32(T * k), row=i32((T, k)),
               unserved=i32(1), sched=i32(2 * WORDS))
    lib.one_block(_p(ids), T * k, k, _p(ert), ert.shape[0], ert.shape[1], _p(alive0), _p(alive1), S,
                  d, I, grid, *[_p(a) for a in out.values()])
    return out


@pytest.mark.parametrize("T,k,S", [(512, 8, 40), (300, 2, 3), (64, 4, 130), (1, 1, 1)])
def test_a_mask_written_during_the_dispatch_leaves_plan_and_offsets_in_agreement(plan, T, k, S):
    """A failure detector may write the mask at any time. Whatever a second
    block reads of it, the row blocks that the GEMMs walk are those of the
    offsets that the call wrote: fewer would leave rows without a result, more
    would lead the walk past the last slot."""
    rng = np.random.default_rng(S)
    E = max(S, k)
    ids = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)
    ert = np.full((E, 2), -1, np.int32)
    ert[:S, 0] = np.arange(S)
    ert[:S, 1] = (np.arange(S) + 1) % S
    alive = (rng.random(S) > 0.2).astype(np.uint8)
    alive[0] = 1
    for later in (alive, 1 - alive, np.zeros_like(alive), np.ones_like(alive)):
        out = _one_block(plan, ids, ert, alive, later, S)
        rows = np.diff(out["offsets"])
        assert np.array_equal(rows, out["counts"])
        assert np.array_equal(np.bincount(out["slot"][out["slot"] >= 0], minlength=S), rows)
        for g in range(2):
            words = out["sched"][g * WORDS:(g + 1) * WORDS]
            assert (words[:PLAN] == 0).all()
            assert 0 <= words[PLAN] <= 8
            assert words[PLAN + 1:PLAN + 5].tolist() == [int((-(-rows // h)).sum()) for h in HEIGHTS]


SHAPES = ("32x64", "32x32", "64x128", "64x64", "128x128", "128x64", "128x256", "32", "256")


def _shapes(lib, d, I, rows):
    r = np.array(rows, np.int32)
    return tuple(SHAPES[lib.choose(up, _p(r), len(r), 256, K, cols)]
                 for up, K, cols in ((1, d, I), (0, I, d)))


def test_the_shape_cases_take_the_shapes_that_they_name(plan):
    """The GPU tests compare a launch's own choice with the full tiles bit for
    bit; a case whose choice had become the full tiles would compare them with
    themselves. The base shapes are reached by many other tests too."""
    for cases in (CASES, FORWARDS):
        for d, I, rows, up, down in cases:
            assert _shapes(plan, d, I, rows) == (up, down), (d, I, rows)
        for g in (3, 4):
            assert set(SHAPES) - {c[g] for c in cases} <= {"32", "256"}
