"""A solve that faults in the middle of a large launch, beside one that does not.

A kernel that raises a flag runs while others of its own workgroups are still
to start; each of those does its work or leaves as a whole.  The fault is
reported, the faulted solve's stored state stays readable, and the solve beside
it gives the bits that it gives alone.
"""
import sys

import numpy as np
import pytest

from paper_2512_09904_amd import cases

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def sph():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_09904_amd import sph as S
    S.lib()
    return S


def _overfull():
    """Rows longer than the default capacity in every block of the bulk: the
    build raises the flag in all of some 2700 workgroups."""
    c = cases.serving_tank(700_000, 300.0, 0.04, 1e-4, seed=1)
    p = c.params
    m = 2.0 * 1.6 * p["dp"] + 3 * p["dp"]
    p.update(h_over_dp=1.6, grid_lo=(-m,) * 3, grid_hi=tuple(float(x) + m for x in c.meta["box"]))
    return c


def _three_bodies():
    """Housing particles of three bodies by turns: nearly every fluid particle
    at a wall touches all three, one more than a particle can account for, and
    the viscous/heat sweep raises the flag."""
    c = cases.serving_tank(500_000, 300.0, 0.04, 1e-4, seed=2)
    c.bodies += [cases.Body((0.0, 0.0, 0.0), (0.0, 0.0, 1.0), 0.0, c.bodies[0].T, c.bodies[0].k) for _ in range(2)]
    w = np.nonzero(c.body == 0)[0]
    c.body[w] = np.array([0, 2, 3], np.int32)[np.arange(len(w)) % 3]
    return c


def _run(sph, reqs, precision, steps):
    pool = sph.Pool(1 << 40, max_slots=len(reqs), precision=precision)
    slots = [pool.admit(c, steps) for c in reqs]
    pool.step(steps)
    out = []
    for s in slots:
        done = False
        while not done:
            done, rep = pool.poll(s)
        out.append((pool.get_fluid(s), rep))
    pool.close()
    return out


@pytest.mark.parametrize("precision", ["mixed", "fp32", "fp64"])
@pytest.mark.parametrize("make", [_overfull, _three_bodies])
def test_a_fault_in_a_large_launch_stays_in_its_solve(sph, precision, make):
    bad, good = make(), cases.tank_c1(seed=3)
    say("fault beside a solve", make.__name__, precision, bad.nf, bad.ns)
    f0, r0 = _run(sph, [good], precision, 3)[0]
    (fb, rb), (f1, r1) = _run(sph, [bad, good], precision, 3)
    assert rb["rc"] == sph.SPH_ERR_CAPACITY and rb["step"] == 0
    assert r0["rc"] == 0 and r1["rc"] == 0 and r1["step"] == 3
    for k in ("x", "v", "rho", "T"):
        assert np.array_equal(f0[k], f1[k]), k
    assert r0["t"] == r1["t"] and r0["kinetic"] == r1["kinetic"]
    if make is _overfull:
        # the build faulted: nothing has moved yet
        real = np.float32 if precision == "fp32" else np.float64
        assert np.array_equal(fb["x"], bad.xf.astype(real).astype(np.float64))
        assert np.array_equal(fb["T"], bad.Tf.astype(real).astype(np.float64))
        assert not fb["v"].any()
