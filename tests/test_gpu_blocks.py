"""Blocks of the neighbour build and the sweeps: every way in which a block of
256 particles takes its neighbours, small and large grids, and the read-out.

A block stages the records of all particles its rows can name (at most 2432,
of at most 64 runs of equal cells), or of three of its four wavefronts, or it
gathers.  Bars: neighbour sets bit for bit; one step against the FP64 oracle to
the bars of one step from identical state (1e-5 mixed, 1e-10 FP64, normalised
as in test_gpu_parity); results that must not depend on the grid, and copies,
exactly.
"""
import sys

import numpy as np
import pytest

from paper_2512_09904_amd import cases

pytestmark = pytest.mark.gpu

BLOCK, WAVE, CAP, RUNS = 256, 64, 2432, 64


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


def _tank(keep):
    """The 2 mm tank with the fluid particles of which keep(index) holds."""
    c = cases.tank_c1(seed=7)
    k = keep(np.arange(c.nf))
    c.xf, c.vf, c.rhof, c.Tf = c.xf[k], c.vf[k], c.rhof[k], c.Tf[k]
    return c


def _kinds(ora, c):
    """How each block of the sorted fluid takes its neighbours: 'whole',
    'three' (the first or the last three wavefronts staged), 'gather'."""
    rc, order = ora.sort_order(c.params, c.xf, np.arange(c.nf, dtype=np.uint32))
    _, cf = ora.cells(c.params, c.xf[order])
    xs, _, _ = ora.body_pose(c.bodies, c.xs0, c.ns0, c.body, 0.0)
    _, cs = ora.cells(c.params, xs)
    count = lambda cells: {tuple(k): int(n) for k, n in zip(*np.unique(cells, axis=0, return_counts=True))}
    nf, ns = count(cf), count(cs)
    off = np.array([(x, y, z) for z in (-1, 0, 1) for y in (-1, 0, 1) for x in (-1, 0, 1)])

    def candidates(cells):
        q = {tuple(k) for k in (np.unique(cells, axis=0)[:, None, :] + off[None]).reshape(-1, 3)}
        return -(-sum(nf.get(k, 0) for k in q) // WAVE) * WAVE + sum(ns.get(k, 0) for k in q)

    out = []
    for b in range(0, c.nf, BLOCK):
        cells = np.asarray(cf[b:b + BLOCK])
        runs = 1 + int(np.sum(np.any(np.diff(cells, axis=0), axis=1)))
        if runs > RUNS:
            out.append("gather")
        elif candidates(cells) <= CAP:
            out.append("whole")
        elif candidates(cells[:3 * WAVE]) <= CAP or (len(cells) > WAVE and candidates(cells[WAVE:]) <= CAP):
            out.append("three")
        else:
            out.append("gather")
    return out


@pytest.mark.parametrize("precision,bar", [("mixed", 1e-5), ("fp64", 1e-10)])
@pytest.mark.parametrize("name,keep,want", [
    ("tank", lambda k: k >= 0, {"whole", "three"}),
    ("ragged", lambda k: (k < BLOCK + 65) & (k % 41 != 0), {"whole"}),
    ("thinned", lambda k: k % 13 == 0, {"gather"}),
    ("isolated", lambda k: k % 997 == 5, {"whole"}),
    ("one", lambda k: k == 4000, {"whole"}),
])
def test_rows_of_every_kind_of_block(sph, ora, precision, bar, name, keep, want):
    """Neighbour sets and one step where blocks are staged whole, in part or not
    at all: whole tanks, a ragged end, more runs than are numbered, particles
    without fluid neighbours."""
    c = _tank(keep)
    kinds = _kinds(ora, c)
    say("blocks", name, precision, c.nf, {k: kinds.count(k) for k in set(kinds)})
    assert want <= set(kinds)
    xs, _, _ = ora.body_pose(c.bodies, c.xs0, c.ns0, c.body, 0.0)
    nb = ora.Nbr(c.params, c.xf, xs)
    d = ora.timestep(c.params, c.bodies, c.xs0, c.body, c.vf)
    dt, nac = d["dt_ad"], d["n_ac"]
    o = ora.State(c, fixed_dt_ad=dt, fixed_nac=nac)
    ro = o.step()
    s = sph.Solver(c, precision=precision, fixed_dt_ad=dt, fixed_nac=nac)
    fl, so = s.neighbour_sets()
    assert fl == nb.sets(0)
    assert so == nb.sets(1)
    s.step(1)
    rg = s.reduce()
    g = s.get_fluid()
    s.close()
    p, umax = c.params, c.meta["umax"]
    scale = dict(x=p["dp"], v=umax, rho=p["rho0"] * (umax / p["c0"]) ** 2, T=abs(c.bodies[0].T - c.Tf.mean()))
    e = {k: np.max(np.abs(g[k] - getattr(o, k))) / q for k, q in scale.items()}
    say("normalised errors", e)
    assert max(e.values()) <= bar, e
    assert rg["n_ac"] == ro["n_ac"]


@pytest.mark.parametrize("precision", ["mixed", "fp32", "fp64"])
def test_small_and_large_grids_agree(sph, precision):
    """Grids of up to 256 and 768 blocks build their rows and dummy velocities
    with four times and twice the wavefronts per block.  A small tank gives the
    same bits alone and beside others that take both grids past these lines."""
    a, b = cases.tank_c1(seed=8), cases.tank_c1(seed=9, dp=1.15e-3)
    blocks = lambda n: -(-n // BLOCK)
    say("grids", precision, blocks(a.nf), blocks(a.ns), blocks(a.nf) + blocks(b.nf), blocks(a.ns) + blocks(b.ns))
    assert max(blocks(a.nf), blocks(a.ns)) <= 256
    assert 256 < min(blocks(a.nf) + blocks(b.nf), blocks(a.ns) + blocks(b.ns))
    assert max(blocks(a.nf) + blocks(b.nf), blocks(a.ns) + blocks(b.ns)) <= 512
    assert min(blocks(a.nf) + 4 * blocks(b.nf), blocks(a.ns) + 4 * blocks(b.ns)) > 768
    res = []
    for reqs in ([a], [b, a], 4 * [b] + [a]):
        pool = sph.Pool(1 << 40, max_slots=len(reqs), precision=precision)
        slots = [pool.admit(c, 3) for c in reqs]
        pool.step(3)
        done = False
        while not done:
            done, rep = pool.poll(slots[-1])
        res.append((pool.get_fluid(slots[-1]), rep))
        pool.close()
    f0, r0 = res[0]
    for f1, r1 in res[1:]:
        for k in ("x", "v", "rho", "T"):
            assert np.array_equal(f0[k], f1[k]), k
        assert r0["t"] == r1["t"] and r0["kinetic"] == r1["kinetic"]
        for x, y in zip(r0["bodies"], r1["bodies"]):
            assert np.array_equal(x["force"], y["force"]) and np.array_equal(x["torque"], y["torque"])


@pytest.mark.parametrize("precision", ["mixed", "fp32", "fp64"])
@pytest.mark.parametrize("nf", [1, 255, 257])
def test_fields_read_back_in_the_callers_order(sph, precision, nf):
    """The fields read back are the stored state (anchor plus drift, velocity,
    density, temperature), particle by particle, at the edges of a block."""
    c = _tank(lambda k: (k >= 3000) & (k < 3000 + nf))
    s = sph.Solver(c, precision=precision)
    s.step(2)
    s.reduce()
    g = s.get_fluid()
    fid = s.dump("fluid_ids").astype(np.int64)
    st = s.dump("fluid_state").reshape(nf, 16)
    s.close()
    assert np.array_equal(np.sort(fid), np.arange(nf))
    assert np.array_equal(g["x"][fid], st[:, 0:3] + st[:, 3:6])
    assert np.array_equal(g["v"][fid], st[:, 6:9])
    assert np.array_equal(g["rho"][fid], st[:, 9])
    assert np.array_equal(g["T"][fid], st[:, 11])


def _wide(c, hod):
    """The case with the smoothing length hod dp and rows that hold its neighbours."""
    p = c.params
    m = 2.0 * hod * p["dp"] + 3 * p["dp"]
    p.update(h_over_dp=hod, grid_lo=(-m,) * 3, grid_hi=tuple(float(x) + m for x in c.meta["box"]),
             max_fluid_nbrs=int(48 * hod ** 3) + 32, max_solid_nbrs=int(32 * hod ** 3) + 48)
    return c


@pytest.mark.parametrize("heated", [False, True])
@pytest.mark.parametrize("precision", ["mixed", "fp32"])
@pytest.mark.parametrize("hod", [1.0, 2.0])
def test_staged_and_gathered_launches_agree(sph, precision, hod, heated):
    """A solve with a narrow or a wide kernel gathers when it runs alone; beside
    one whose kernel is between them the launch stages its candidates.  The same
    bits, with and without dissipation heating and two materials."""
    a, b = _wide(cases.tank_c1(seed=8), hod), cases.tank_c1(seed=9)
    if heated:
        for c in (a, b):
            c.params.update(viscous_heating=1, materials=[(0.13, 2000.0), (0.45, 1300.0)])
            c.material = (c.xf[:, 0] > 0.05).astype(np.int32)
    res = []
    for reqs in ([a], [b, a]):
        pool = sph.Pool(1 << 40, max_slots=2, precision=precision)
        slots = [pool.admit(c, 4) for c in reqs]
        pool.step(4)
        done = False
        while not done:
            done, rep = pool.poll(slots[-1])
        assert rep["rc"] == 0
        res.append((pool.get_fluid(slots[-1]), rep))
        pool.close()
    (f0, r0), (f1, r1) = res
    for k in ("x", "v", "rho", "T"):
        assert np.array_equal(f0[k], f1[k]), k
    assert r0["t"] == r1["t"] and r0["kinetic"] == r1["kinetic"] and r0["diss_total"] == r1["diss_total"]
    for x, y in zip(r0["bodies"], r1["bodies"]):
        for k in ("force", "torque", "heat_int"):
            assert np.array_equal(x[k], y[k]), k


def _in_fp32(c):
    f32 = lambda a: np.asarray(a, dtype=np.float32).astype(np.float64)
    c.xf, c.rhof, c.Tf, c.vf = f32(c.xf), f32(c.rhof), f32(c.Tf), f32(c.vf)
    return c


KINDS = [
    ("wide", lambda k: k >= 0, 1.6, {"whole", "three", "gather"}),
    ("tank", lambda k: k >= 0, 1.3, {"whole", "three"}),
    ("ragged", lambda k: (k < BLOCK + 65) & (k % 41 != 0), 1.3, {"whole"}),
    ("thinned", lambda k: k % 13 == 0, 1.3, {"gather"}),
    ("isolated", lambda k: k % 997 == 5, 1.3, {"whole"}),
    ("one", lambda k: k == 4000, 1.3, {"whole"}),
]


@pytest.mark.parametrize("precision,name,keep,hod,want",
                         [("mixed",) + KINDS[0]] + [("fp32",) + k for k in KINDS])
def test_rows_of_every_kind_of_block_wide_and_in_fp32(sph, ora, precision, name, keep, hod, want):
    """As above with blocks that gather because their candidates do not fit (few
    runs, a wide kernel), and in all-FP32 arithmetic.  Bars: mixed as above; FP32
    those of one step in that mode (test_gpu_parity): sets up to pairs within 1e-5
    of the cutoff, x, rho, T within 20 ulps, v within what 20 ulps of the density
    imply through the pressure."""
    c = _tank(keep)
    if hod != 1.3:
        c = _wide(c, hod)
    if precision == "fp32":
        c = _in_fp32(c)
    kinds = _kinds(ora, c)
    say("blocks", name, precision, c.nf, {k: kinds.count(k) for k in set(kinds)})
    assert want <= set(kinds)
    rc, order = ora.sort_order(c.params, c.xf, np.arange(c.nf, dtype=np.uint32))
    cf = np.asarray(ora.cells(c.params, c.xf[order])[1])
    runs = [1 + int(np.sum(np.any(np.diff(cf[b:b + BLOCK], axis=0), axis=1))) for b in range(0, c.nf, BLOCK)]
    if name == "wide":
        assert max(runs) <= RUNS   # the candidates decide
    xs, _, _ = ora.body_pose(c.bodies, c.xs0, c.ns0, c.body, 0.0)
    nb = ora.Nbr(c.params, c.xf, xs)
    d = ora.timestep(c.params, c.bodies, c.xs0, c.body, c.vf)
    dt, nac = d["dt_ad"], d["n_ac"]
    o = ora.State(c, fixed_dt_ad=dt, fixed_nac=nac)
    ro = o.step()
    s = sph.Solver(c, precision=precision, fixed_dt_ad=dt, fixed_nac=nac)
    fl, so = s.neighbour_sets()
    cut2 = (2.0 * c.params["h_over_dp"] * c.params["dp"]) ** 2
    for got, ref, x in ((fl, nb.sets(0), c.xf), (so, nb.sets(1), np.asarray(xs))):
        for i in range(c.nf):
            for j in got[i] ^ ref[i]:
                assert precision == "fp32", (i, j)
                assert abs(float(np.sum((c.xf[i] - x[j]) ** 2)) - cut2) <= 1e-5 * cut2, (i, j)
    s.step(1)
    rg = s.reduce()
    g = s.get_fluid()
    s.close()
    p, umax = c.params, c.meta["umax"]
    scale = dict(x=p["dp"], v=umax, rho=p["rho0"] * (umax / p["c0"]) ** 2, T=abs(c.bodies[0].T - c.Tf.mean()))
    bar = {k: 1e-5 * q for k, q in scale.items()}
    if precision == "fp32":
        ulp = lambda a: float(np.spacing(np.float32(np.max(np.abs(a)))))
        drho = 20 * ulp(o.rho)
        bar = dict(x=20 * ulp(o.x), v=dt * 6.0 * p["c0"] ** 2 * drho / (p["rho0"] * p["h_over_dp"] * p["dp"]),
                   rho=drho, T=20 * ulp(o.T))
    e = {k: np.max(np.abs(g[k] - getattr(o, k))) for k in scale}
    say("errors over bars", {k: e[k] / bar[k] for k in e})
    for k in e:
        assert e[k] <= bar[k], (k, e[k], bar[k])
    assert rg["n_ac"] == ro["n_ac"]


@pytest.mark.parametrize("precision", ["mixed", "fp32", "fp64"])
def test_dummy_velocities_outlast_a_contact_reading(sph, precision):
    """The contact factor's sort and build leave the last step's dummy velocities
    and their kernel sums as they are (the walls at rest keep their places)."""
    c = cases.tank_c1(seed=4)
    s = sph.Solver(c, precision=precision)
    s.step(2)
    s.reduce()
    sid = s.dump("solid_ids").copy()
    d0 = s.dump("solid_dummy").reshape(c.ns, 4).copy()
    assert (d0[:, 3] > 0).any()
    s.contact_factor()
    still = (s.dump("solid_ids") == sid) & (c.body[sid] == 0)
    assert still.any()
    d1 = s.dump("solid_dummy").reshape(c.ns, 4)
    s.close()
    assert np.array_equal(d0[still], d1[still])
