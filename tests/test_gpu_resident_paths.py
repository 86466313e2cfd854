"""The resident solver where it is hard to see whether it ran: the tests ask the
handle whether its solves take it, and the timing counters, which count every
iteration of a resident solve and one check interval in eight of the sweeps.
Rows split between tiles over the depths of the ghost columns and the check
intervals around them; tags that run out; launches that are refused and blocks
that wait in vain, after which the sweeps go on."""
import ctypes as C
import threading

import numpy as np
import pytest
import torch

import oracle
import paper_1504_02264_amd as les
from les_inputs import log_law_profile, random_rhs

from test_gpu_resident import same

pytestmark = pytest.mark.gpu

SPIN, GATE = 1 << 21, 1 << 11   # the solver's own bounds of a wait and of the roll call
SPACING = (2.0, 3.0, 1.5)


def resident(g, spin=-2, gate=-1, early=-1, tag=0):
    f = les.lib().les_test_resident
    f.argtypes = [C.c_void_p, C.c_int32, C.c_int32, C.c_int32, C.c_uint32, C.POINTER(C.c_int32)]
    runs = C.c_int32()
    assert f(g.h, spin, gate, early, tag, C.byref(runs)) == les.LES_OK
    return runs.value


def inputs(shape):
    nx, ny, nz = shape
    return random_rhs(nx, ny, nz, seed=nx + 7 * ny + 31 * nz, smooth=1), random_rhs(nx, ny, nz, seed=5)


def make(shape, variant=None, **kw):
    g = les.LES(*shape, *SPACING, 0.05, **kw)
    if variant is not None:
        g.set_sor_variant(variant)
    assert resident(g) == (variant is None)
    return g


@pytest.mark.parametrize("nx,depth", [(223, 4), (224, 4), (150, 13), (451, 9)])
@pytest.mark.parametrize("K,R", [(1, 1), (3, 1), (4, 32), (8, 16), (0, 1), (1000, 1), (64, 2)])
def test_ghost_columns_equal_sweep_launches(nx, depth, K, R):
    """The depth itself for K = 0; intervals below, at and above it, folds in
    every interval and in few."""
    shape = (nx, 17, 9)
    K = K or depth
    rhs, p0 = inputs(shape)
    print(f"[ghosts] nx={nx} K={K} R={R}", flush=True)
    for n in (4 * depth + 3, 700):
        out = []
        for variant in (None, 1):
            g = make(shape, variant, check_every=K, rebase_every=R, timing=1)
            try:
                out.append(g.pressure_solve(rhs, p0, tol=1e-9, max_iter=n))
                if variant is None:
                    assert resident(g) and g.get_timing()["sor"][1] == out[0][1]["iters"] == n
            finally:
                g.close()
        same(*out)


@pytest.mark.parametrize("shape", [(150, 33, 11), (70, 131, 67), (300, 300, 90)])
def test_tags_run_out(shape):
    """Launches before, across and after the end of the tags' range."""
    rhs, p0 = inputs(shape)
    g, ref = make(shape, check_every=64, rebase_every=2), make(shape, 1, check_every=64, rebase_every=2)
    try:
        want = ref.pressure_solve(rhs, p0, tol=1e-9, max_iter=130)
        for tag in (0x7fffffff - 400, 0xffffffff - 800):
            assert resident(g, tag=tag)
            for _ in range(4):
                same(g.pressure_solve(rhs, p0, tol=1e-9, max_iter=130), want)
        assert resident(g)
    finally:
        g.close()
        ref.close()


def residual(rhs, p, shape):
    """The oracle's relative residual of p, and how far the solver's, whose p is a
    float32 value and an exact rest, can be from it: the rest is at most 2^-24 |p|,
    so 2^-24 || |A| |p| || / ||rhs||, and |A| |p| = A |p| + 2 diag |p| with A's
    diagonal at most 3 / dx^2 + 2 / dy^2 + 2 / dz^2."""
    o = oracle.Oracle(*shape, *SPACING, 0.05)
    dx, dy, dz = SPACING
    diag = 3 / dx ** 2 + 2 / dy ** 2 + 2 / dz ** 2
    q = np.abs(p.astype(np.float64))
    slack = np.linalg.norm(o.apply_A(q) + 2 * diag * q) / np.linalg.norm(rhs.astype(np.float64))
    return o.residual(rhs, p), 2.0 ** -24 * slack


@pytest.mark.parametrize("shape", [(64, 33, 11), (150, 33, 11), (70, 131, 67)])
@pytest.mark.parametrize("K,max_iter", [(4, 20000), (4, 7), (4, 100), (64, 640), (20, 9)])
def test_solve_goes_on_after_a_lost_launch(shape, K, max_iter):
    rhs, p0 = inputs(shape)
    g = make(shape, check_every=K, rebase_every=max(1, 128 // K), timing=1)
    ref = make(shape, 1, check_every=K, rebase_every=max(1, 128 // K))
    try:
        resident(g, spin=0)
        print(f"[lost] {shape} K={K} max_iter={max_iter}", flush=True)
        p, st, rc = g.pressure_solve(rhs, p0, tol=1e-5, max_iter=max_iter)
        assert not resident(g)
        r, slack = residual(rhs, p, shape)
        assert abs(r - st["resid"]) <= slack
        # stops as the sweeps do (150 columns take more than 20000 iterations)
        want = ref.pressure_solve(rhs, p0, tol=1e-5, max_iter=max_iter)
        print(f"[lost] sweeps: {want[1]} here: {st}", flush=True)
        assert rc == want[2] and st["converged"] == (st["resid"] <= 1e-5)
        assert st["converged"] or st["iters"] == max_iter
        # and the handle goes on, with its sweep launches
        resident(g, spin=SPIN)
        same(g.pressure_solve(rhs, p0, tol=1e-5, max_iter=300), ref.pressure_solve(rhs, p0, tol=1e-5, max_iter=300))
        assert not resident(g)
    finally:
        g.close()
        ref.close()


def test_refused_launch():
    shape = (150, 33, 11)
    rhs, p0 = inputs(shape)
    g, ref = make(shape), make(shape, 0)
    try:
        resident(g, spin=-1)
        same(g.pressure_solve(rhs, p0, max_iter=300), ref.pressure_solve(rhs, p0, max_iter=300))
        assert not resident(g, spin=SPIN)
    finally:
        g.close()
        ref.close()


def test_no_room_on_the_chip():
    """A roll call that ends too soon: the sweeps run the solve from its start, the
    handle tries again after one solve, then after three, and is resident again."""
    shape = (150, 33, 11)
    rhs, p0 = inputs(shape)
    g, ref = make(shape), make(shape, 0)
    try:
        want = ref.pressure_solve(rhs, p0, max_iter=300)
        tries = ((0, True), (0, False), (0, True), (0, False), (0, False), (0, False), (GATE, True), (GATE, True))
        for gate, now in tries:
            assert resident(g, gate=gate) == now
            same(g.pressure_solve(rhs, p0, max_iter=300), want)
        assert resident(g)
    finally:
        g.close()
        ref.close()


@pytest.mark.parametrize("shape,n", [((33, 17, 9), 20000), ((150, 33, 11), 700), ((128, 128, 64), 400)])
def test_solves_in_several_threads(shape, n):
    """Solves side by side, on a part of the chip each or in turn: each gives what
    it gives alone."""
    def run(g, seed, out):
        rhs, p0 = random_rhs(*shape, seed=seed, smooth=1), random_rhs(*shape, seed=5 + seed)
        for q in range(4):
            out[seed, q] = g.pressure_solve(rhs, p0, tol=1e-5, max_iter=n)

    handles = [make(shape) for _ in range(4)]
    try:
        alone, beside = {}, {}
        for q, g in enumerate(handles):
            run(g, q, alone)
        threads = [threading.Thread(target=run, args=(g, q, beside)) for q, g in enumerate(handles)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert len(alone) == len(beside) == 16
        for k in alone:
            same(alone[k], beside[k])
        assert all(resident(g) for g in handles)
    finally:
        for g in handles:
            g.close()


def test_solves_beside_a_persistent_ensemble():
    """Both kinds of launch whose blocks wait for each other, from two threads."""
    prof = log_law_profile(18, 2.0)

    def members():
        out = []
        for q in range(2):
            g = les.LES(40 + 8 * q, 32, 18, 4.0, 4.0, 2.0, 0.05, None, max_iter=400)
            g.set_inflow(prof, 0.01, q)
            out.append(g)
        e = les.Ensemble(out)
        e.set_mode(les.ENSEMBLE_PERSISTENT)
        return e, out

    def steps(e, ms, out):
        for _ in range(8):
            e.step(1)
        out.extend(m.get_fields() for m in ms)

    def solves(g, out):
        rhs, p0 = inputs((64, 64, 32))
        for _ in range(12):
            out.append(g.pressure_solve(rhs, p0, tol=1e-9, max_iter=300))

    (ea, a), (eb, b) = members(), members()
    gs = [make((64, 64, 32)) for _ in range(2)]
    try:
        want, got, one, two = [], [], [], []
        steps(ea, a, want)
        threads = [threading.Thread(target=steps, args=(eb, b, got)), threading.Thread(target=solves, args=(gs[0], one))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        solves(gs[1], two)
        for x, y in zip(want, got):
            assert all(np.array_equal(f, h) for f, h in zip(x, y))
        assert len(one) == len(two) == 12
        for x, y in zip(one, two):
            same(x, y)
        assert resident(gs[0]) and resident(gs[1])
    finally:
        ea.close()
        eb.close()
        for g in a + b + gs:
            g.close()


@pytest.mark.parametrize("shape", [(64, 33, 11), (150, 33, 11), (70, 131, 67)])
@pytest.mark.parametrize("K,tol", [(3, 1e-9), (4, 1e-9), (4, 1e-2), (16, 1e-9), (64, 1e-9), (600, 1e-9)])
def test_sweeps_take_the_early_intervals(shape, K, tol):
    """Sweep launches for the first 512 iterations (whole intervals) and the
    resident solver beyond, for solves that end before, at and after the change."""
    rhs, p0 = inputs(shape)
    kw = dict(check_every=K, rebase_every=max(1, 128 // K))
    g, ref = make(shape, timing=1, **kw), make(shape, 1, **kw)
    try:
        assert resident(g, early=0)
        g.pressure_solve(rhs, p0, tol=tol, max_iter=1)
        for n in (1, 300, 512, 513, 517, 1300):
            g.get_timing(reset=True)
            got = g.pressure_solve(rhs, p0, tol=tol, max_iter=n)
            same(got, ref.pressure_solve(rhs, p0, tol=tol, max_iter=n))
            beyond = got[1]["iters"] - 512 // K * K
            if beyond > 0:
                assert g.get_timing()["sor"][1] == beyond
        g.get_timing(reset=True)
        assert resident(g, early=1)
        same(g.pressure_solve(rhs, p0, tol=tol, max_iter=300), ref.pressure_solve(rhs, p0, tol=tol, max_iter=300))
    finally:
        g.close()
        ref.close()


@pytest.mark.parametrize("shape", [(33, 17, 9), (150, 33, 11), (256, 256, 64)])
@pytest.mark.parametrize("K", [3, 4, 64, 1000])
def test_tuned_solves_equal_sweep_launches(shape, K):
    """Whatever form the autotuner keeps, from a workspace that has held a
    right-hand side that is not finite."""
    rhs, p0 = inputs(shape)
    kw = dict(check_every=K, rebase_every=max(1, 128 // K))
    g, ref = make(shape, **kw), make(shape, 1, **kw)
    try:
        bad = rhs.copy()
        bad[1, 2, 3] = np.nan
        with pytest.raises(les.LesError):
            g.pressure_solve(bad, p0)
        v, us = g.autotune(reps=3)
        print(f"[tuned] {shape} K={K} variant {v} resident {resident(g)}", flush=True)
        for n in (200, 900):
            same(g.pressure_solve(rhs, p0, tol=1e-9, max_iter=n), ref.pressure_solve(rhs, p0, tol=1e-9, max_iter=n))
    finally:
        g.close()
        ref.close()


def test_ensemble_autotune_leaves_members_without_face_buffers():
    """An ensemble never uses them: a member allocates them at its own first solve."""
    shape = (150, 150, 90)
    g = make(shape)
    e = les.Ensemble([g])
    try:
        e.autotune(reps=1)
        before = torch.cuda.mem_get_info()[0]
        rhs, p0 = inputs(shape)
        g.pressure_solve(rhs, p0, max_iter=4)
        assert torch.cuda.mem_get_info()[0] < before
        assert resident(g)
    finally:
        e.close()
        g.close()


@pytest.mark.parametrize("shape,patch", [((33, 17, 9), 4), ((150, 33, 11), 4), ((187, 131, 67), 24)])
@pytest.mark.parametrize("K", [1, 2, 4, 8])
def test_solves_of_a_few_iterations(shape, patch, K):
    """Whole check intervals of up to two iterations (one interval of up to four
    with the smallest patch) take the sweep launches, of which one interval in
    eight is timed, from the first one on; longer solves are resident."""
    rhs, p0 = inputs(shape)
    g, ref = make(shape, check_every=K, timing=1), make(shape, 0, check_every=K, timing=1)
    try:
        for n in (1, 2, 3, 4, 5):
            for h in (g, ref):
                h.get_timing(reset=True)
            same(g.pressure_solve(rhs, p0, tol=1e-9, max_iter=n), ref.pressure_solve(rhs, p0, tol=1e-9, max_iter=n))
            sweeps = ref.get_timing()["sor"][1]
            whole = -(-n // K) * K
            few = whole <= (4 if n <= K and patch == 4 else 2)
            assert g.get_timing()["sor"][1] == (sweeps if few else n)
    finally:
        g.close()
        ref.close()
