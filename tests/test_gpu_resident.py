"""The resident solver (the pressure system held on the chip, one cooperative
launch per solve) against the sweep launches: the same arithmetic in the same
order, so iterates, iteration counts and statuses agree bit for bit, and the
float64 norms up to the order of their sums (2^-53 sqrt(blocks) relative,
bounded here by 1e-12).  The sweep launches are compared with the oracle in
test_gpu_parity.py."""
import numpy as np
import pytest

import paper_1504_02264_amd as les
from les_inputs import building_heights, building_mask, log_law_profile, random_rhs

pytestmark = pytest.mark.gpu

WALLS = (les.FREESLIP,) * 6


def solve(shape, variant, tol=1e-5, max_iter=600, spacing=(2.0, 3.0, 1.5), **kw):
    nx, ny, nz = shape
    g = les.LES(nx, ny, nz, *spacing, 0.05, **kw)
    try:
        if variant is not None:
            g.set_sor_variant(variant)
        rhs = random_rhs(nx, ny, nz, seed=nx + 7 * ny + 31 * nz, smooth=1)
        p0 = random_rhs(nx, ny, nz, seed=5)
        first = g.pressure_solve(rhs, p0, tol=tol, max_iter=max_iter)
        again = g.pressure_solve(rhs, p0, tol=tol, max_iter=max_iter)   # tags and buffers of a later launch
        assert np.array_equal(first[0], again[0]) and first[1] == again[1]
        return first
    finally:
        g.close()


def same(a, b):
    (pa, sa, ra), (pb, sb, rb) = a, b
    assert ra == rb and sa["iters"] == sb["iters"]
    assert np.array_equal(pa, pb)
    for k in ("resid", "rhs_norm", "reltmp2"):
        assert sa[k] == pytest.approx(sb[k], rel=1e-12)


@pytest.mark.parametrize("shape", [
    (4, 4, 4), (5, 7, 4), (64, 9, 5),               # one block; a full and an odd row
    (127, 8, 4), (128, 17, 9), (129, 16, 8),        # 64 half-cells, then rows split between tiles
    (150, 33, 11), (257, 40, 13), (451, 9, 6),      # ghost columns: 13, 10 and 4 deep, two to five tiles
    (70, 131, 67), (110, 258, 98),                  # the larger patches, rows and planes left over
    (300, 300, 90)])                                # the largest patch, three tiles per row
def test_resident_equals_sweep_launches(shape):
    print(f"[resident] {shape}", flush=True)
    n = 200 if np.prod(shape) > 1e6 else 600
    same(solve(shape, None, max_iter=n), solve(shape, 1, max_iter=n))


@pytest.mark.parametrize("K,R", [(1, 1), (3, 2), (4, 32), (8, 16), (64, 2), (1000, 1)])
@pytest.mark.parametrize("max_iter", [0, 1, 13, 130, 9001])
def test_resident_check_intervals_and_caps(K, R, max_iter):
    """Every check interval and fold schedule, solves cut inside an interval,
    and solves longer than one launch."""
    shape = (70, 21, 11)
    kw = dict(check_every=K, rebase_every=R, tol=1e-9)
    print(f"[resident] K={K} R={R} max_iter={max_iter}", flush=True)
    a, b = (solve(shape, v, max_iter=max_iter, **kw) for v in (None, 1))
    same(a, b)


def test_resident_singular_operator_and_omega():
    for omega in (0.7, 1.0, 1.9):
        same(*(solve((131, 33, 12), v, bc=WALLS, omega=omega) for v in (None, 0)))


def test_resident_edge_cases():
    g = les.LES(40, 20, 10, 2.0, 2.0, 1.0, 0.05)
    try:
        zero = np.zeros((10, 20, 40), np.float32)
        p, st, rc = g.pressure_solve(zero, None)
        assert rc == les.LES_OK and st["iters"] == 0 and not p.any()
        bad = zero.copy()
        bad[3, 4, 5] = np.inf
        with pytest.raises(les.LesError) as e:
            g.pressure_solve(bad, None)
        assert e.value.code == les.LES_ENONFINITE
        rhs = random_rhs(40, 20, 10, seed=1)
        assert g.pressure_solve(rhs, None)[2] == les.LES_OK   # and the handle goes on
    finally:
        g.close()


def test_resident_time_steps():
    """Steps of an urban case: fields bit for bit, with timing events, across a
    checkpoint, and with two handles taking turns on one GPU."""
    nx, ny, nz = 72, 40, 18
    mask = building_mask(building_heights(nx, ny, nz, 0.2, 2, 6, 2, 8, seed=3), nz)
    prof = log_law_profile(nz, 2.0)

    def make(variant, **kw):
        g = les.LES(nx, ny, nz, 4.0, 4.0, 2.0, 0.05, mask, **kw)
        if variant is not None:
            g.set_sor_variant(variant)
        g.set_inflow(prof, 0.01, 3)
        return g

    a, b, c = make(None), make(1), make(None, timing=1)
    try:
        for _ in range(2):
            its = [int(g.step(1)[2][0]) for g in (a, b, c)]
            assert its[0] == its[1] == its[2]
        c.get_timing(reset=True)
        c.set_state(a.get_state())
        its = [int(g.step(1)[2][0]) for g in (a, b, c)]
        assert its[0] == its[1] == its[2]
        assert c.get_timing()["sor"][1] == its[2]
        for x, y, z in zip(a.get_fields(), b.get_fields(), c.get_fields()):
            assert np.array_equal(x, y) and np.array_equal(x, z)
    finally:
        for g in (a, b, c):
            g.close()


def test_autotune_may_turn_it_on_again():
    rhs = random_rhs(64, 40, 12, seed=2)
    g = les.LES(64, 40, 12, 2.0, 2.0, 1.0, 0.05)
    try:
        ref = g.pressure_solve(rhs, None, max_iter=500)
        g.set_sor_variant(3)
        same(g.pressure_solve(rhs, None, max_iter=500), ref)
        v, us = g.autotune(reps=5)
        assert 0 <= v < les.NUM_SOR_VARIANTS and np.all(us > 0)
        same(g.pressure_solve(rhs, None, max_iter=500), ref)
    finally:
        g.close()
