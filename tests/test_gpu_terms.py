"""Terms of the force and energy evaluations at the edges of their ranges, GPU against the oracle.

The step kernel takes (pi - theta) / sin(theta) from a polynomial up to 45 degrees from the straight angle and from
an arctangent beyond, and reads a dihedral from either end: molecules of three and four beads sit on both sides of the
switch, at the straight angle itself and at both resting angles a model uses."""
import dataclasses
import math

import numpy as np
import pytest

import synth
from gpu_common import both, forces_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.init()


BENDS = [0.0, 1e-9, 1e-6, 1e-3, 0.3, math.radians(44.9999), math.radians(45.0001), 1.2, 0.5 * math.pi, 2.2,
         math.radians(170)]
TORSIONS = [0.0, 1e-3, 0.7, -0.7, 0.5 * math.pi, -2.0, 3.0, math.pi]


def _molecules(kind, seed):
    rng = np.random.default_rng(seed)
    xs, angles, dihedrals = [], [], []
    pitch, per = 8.0, 8
    cases = BENDS if kind == "angle" else TORSIONS
    m = 0
    for value in cases:
        for rep in range(6):
            if kind == "angle":
                w = np.array([math.cos(value), math.sin(value), 0.0]) * (0.8 + 0.1 * rep)
                p = np.array([[-1.0, 0.0, 0.0], [0.0, 0.0, 0.0], w])
            else:
                p = np.array([[0.3 + 0.1 * rep, 1.0, 0.0], [0.0, 0.0, 0.0], [0.0, 0.0, 1.1],
                              [-0.2 + math.cos(value), math.sin(value), 1.3]])
                p[0] = [math.cos(0.0), math.sin(0.0), 0.2 - 0.1 * rep]
            centre = np.array([m % per, m // per % per, m // (per * per)]) * pitch + 4.0
            base = 4 * m if kind == "dihedral" else 3 * m
            xs.append(p @ synth._rotation(rng).T + centre)
            # stored from either end
            ids = list(range(base, base + len(p)))
            ids = ids if rep % 2 == 0 else ids[::-1]
            # a right-angle rest is singular at the straight angle: only for bends from 0.3
            kind2 = rep % 2 if kind == "dihedral" or value >= 0.3 else 0
            (angles if kind == "angle" else dihedrals).append((1 + kind2, *ids))
            m += 1
    x = np.concatenate(xs)
    n, L = x.shape[0], per * pitch
    return synth.System(L=L, x=synth.wrap(x, L), v=np.zeros((n, 3)), type=np.ones(n, dtype=np.int32),
                        reactive=np.zeros(n, dtype=np.uint8), bonds=np.zeros((0, 4), dtype=np.int32),
                        angles=np.array(angles, dtype=np.int32).reshape(-1, 4),
                        dihedrals=np.array(dihedrals, dtype=np.int32).reshape(-1, 5))


@pytest.mark.parametrize("kind", ["angle", "dihedral"])
@pytest.mark.parametrize("pair", ["wca", "dpd"])
@pytest.mark.parametrize("precision", [0, 1])
def test_bends_and_torsions_match_oracle(precision, pair, kind):
    """Tolerances: a force is good to a unit roundoff (1.1e-16, 6e-8) times some twenty operations, over the sine of
    the angle where the resting angle makes that count, least at 170 degrees of bend (1 / 0.17 = 6): 1.4e-14 and
    7e-6, so 1e-12 (separations of a 64-edge box hold 1e-14) and 1e-5; energies likewise."""
    s = _molecules(kind, 3)
    ff = dataclasses.replace(synth.ForceField(eps=0.0, gamma=0.0), pair=pair, dpd_a=0.0, dpd_gamma=0.0, rc=1.0)
    ff.angles = {1: (10.0, math.pi), 2: (3.0, 0.5 * math.pi)}
    ff.dihedrals = {1: (5.0, 0.0), 2: (2.0, 1.1)}
    g, o = both(s, ff, synth.RuleSet(every=0), precision=precision, generate=False)
    tol = 1e-12 if precision == 0 else 1e-5
    ok, msg = forces_close(g.forces(), o.forces(), tol)
    assert ok, msg
    eg, eo = g.energy(), o.energy()
    for k in (3, 4):
        assert abs(eg[k] - eo[k]) <= tol * max(1.0, abs(eo[k])), (k, eg[k], eo[k])


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,L", [(1, 2.2), (60, 2.2), (257, 2.9), (300, 3.3), (1000, 4.1)])
def test_evaluation_from_cells_matches_oracle(n, L, precision):
    """One, two, three and four cells per edge (a list cutoff of 1.02), from a lone bead to a density of 14 where
    most beads have more candidates than the staged rows hold.  The DPD pairs are soft, so every term is good to
    some twenty roundings of numbers of order 25, summed over at most about 100 pairs."""
    s = synth.random_gas(n, L, seed=n)
    ff = synth.ff_dpd(gamma_dpd=20.0)
    g, o = both(s, ff, synth.RuleSet(every=0), precision=precision, generate=False)
    tol = 1e-12 if precision == 0 else 1e-5
    if n > 1:
        ok, msg = forces_close(g.forces(), o.forces(), tol)
        assert ok, msg
    eg, eo = g.energy(), o.energy()
    assert np.all(np.abs(eg - eo) <= 10 * tol * np.maximum(1.0, np.abs(eo))), (eg, eo)


def test_forces_report_a_crowded_bead():
    """A clump whose central beads have more neighbours within the list cutoff than a list holds is an error of the
    force evaluation, though it reads no list."""
    import paper_1108_4214_amd as pk
    rng = np.random.default_rng(41)
    d = rng.normal(size=(300, 3))
    d *= 1.2 * rng.uniform(size=(300, 1)) ** (1.0 / 3.0) / np.linalg.norm(d, axis=1)[:, None]
    s = synth.System(L=20.0, x=10.0 + d, v=np.zeros_like(d), type=np.ones(300, dtype=np.int32),
                     reactive=np.zeros(300, dtype=np.uint8), bonds=np.zeros((0, 4), dtype=np.int32))
    g = pk.System(s.n, s.L, 3).configure(s, synth.ForceField(eps=0.0), synth.RuleSet(every=0))
    with pytest.raises(pk.DynBondError) as e:
        g.forces()
    assert e.value.code == pk.DB_ECAPACITY


@pytest.mark.parametrize("n", [4, 255, 256, 1025])
def test_topology_lists_come_back_sorted(n):
    """Lists read from the device are those set, canonical and sorted: beads with many entries, equal paths under
    several types, a ragged last workgroup."""
    import paper_1108_4214_amd as pk
    rng = np.random.default_rng(n)
    k = np.arange(n - 3)
    s = synth.System(L=20.0, x=rng.uniform(0, 20.0, size=(n, 3)), v=np.zeros((n, 3)), type=np.ones(n, dtype=np.int32),
                     reactive=np.zeros(n, dtype=np.uint8), bonds=np.zeros((0, 4), dtype=np.int32))
    perm = rng.permutation(n)
    bonds = np.column_stack([perm[k], perm[k + 1], 1 + k % 5, 1 + k % 7])
    angles = np.concatenate([np.column_stack([1 + (k + r) % 3, perm[k], perm[k + 1], perm[k + 2]]) for r in (0, 1)])
    dihedrals = np.concatenate([np.column_stack([1 + (k + r) % 4, perm[k], perm[k + 1], perm[k + 2], perm[k + 3]])
                                for r in (0, 2)])
    for rows in (bonds, angles, dihedrals):
        rng.shuffle(rows)
    s = dataclasses.replace(s, bonds=bonds.astype(np.int32), angles=angles.astype(np.int32),
                            dihedrals=dihedrals.astype(np.int32))
    g = pk.System(s.n, s.L, 3).configure(s, synth.ForceField(eps=0.0, gamma=0.0), synth.RuleSet(every=0))
    g.step(9)
    b = np.where((bonds[:, 0] > bonds[:, 1])[:, None], bonds[:, [1, 0, 3, 2]], bonds)
    a = np.where((angles[:, 1] > angles[:, 3])[:, None], angles[:, [0, 3, 2, 1]], angles)
    d = np.where((dihedrals[:, 1] > dihedrals[:, 4])[:, None], dihedrals[:, [0, 4, 3, 2, 1]], dihedrals)
    assert np.array_equal(g.bonds(), b[np.lexsort(b.T[::-1])])
    assert np.array_equal(g.angles(), a[np.lexsort((a[:, 0], a[:, 3], a[:, 2], a[:, 1]))])
    assert np.array_equal(g.dihedrals(), d[np.lexsort((d[:, 0], d[:, 4], d[:, 3], d[:, 2], d[:, 1]))])


@pytest.mark.parametrize("skin", [0.03, 0.08, 0.17])
@pytest.mark.parametrize("tiles,graph", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_blocks_cut_short_follow_the_oracle(tiles, graph, skin):
    """Speeds that outrun a thin skin end blocks after one, two, three ... of their steps (either buffer holding the
    state then), with launches and graphs, both kernel shapes; positions as in the other trajectory tests."""
    import paper_1108_4214_amd as pk
    from gpu_common import same_topology
    s = synth.single_strands(24, 6, L=11.0, seed_w=3, seed_d=4, T=2.0)
    g, o = both(s, synth.ff_t2(T0=2.0, T1=2.0), synth.rules_t2(p=0.7, every=7, r_kill=1.35), seed=9)
    pk.db_tune(g.ctx, skin, 2)
    pk.db_tile_shape(g.ctx, tiles)
    pk.db_graph(g.ctx, graph)
    for _ in range(3):
        g.step(8)
        o.step(8)
    assert g.stats()["rollbacks"] > 0 and g.stats()["steps"] == 24
    d = g.state()[0] - o.state()[0]
    d -= s.L * np.round(d / s.L)
    assert np.abs(d).max() < 1e-9
    assert same_topology(g, o)


def _list_forces(system, ff, precision, seed):
    """forces through the Verlet lists: the velocity change of one step from rest, over the step"""
    import paper_1108_4214_amd as pk
    g = pk.System(system.n, system.L, seed, precision).configure(system, ff, synth.RuleSet(every=0), generate=False)
    g.step(1)
    return g.state()[1] / ff.dt


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,L", [(2, 3.1), (200, 3.2), (500, 4.3), (1500, 5.5), (700, 40.0), (3000, 300.0),
                                 (3000, 3000.0), (140000, 40.0)])
def test_list_build_matches_oracle(n, L, precision):
    """Lists from two to hundreds of cells per edge: crowded cells (more candidates than the staged rows), nearly
    empty ones (a run's last group reaches far into other rows), an edge whose sixteenth-bit units are too coarse,
    one and four threads per bead.  Forces of soft pairs, so every term is good to some twenty roundings; clusters of
    beads across the corner of the box make every wrapped row count."""
    rng = np.random.default_rng(n)
    x = rng.uniform(0.0, L, size=(n, 3))
    k = n // 3
    x[:k] = np.mod(rng.normal(0.0, max(0.8, 0.25 * k ** (1.0 / 3.0)), size=(k, 3)), L)   # a cloud about the corner
    s = synth.System(L=L, x=synth.wrap(x, L), v=np.zeros((n, 3)), type=np.ones(n, dtype=np.int32),
                     reactive=np.zeros(n, dtype=np.uint8), bonds=np.zeros((0, 4), dtype=np.int32))
    ff = dataclasses.replace(synth.ff_dpd(gamma_dpd=0.0), dt=2.0 ** -10)
    import oracle
    o = oracle.Oracle.from_system(s, ff, synth.RuleSet(every=0), seed=1, generate=False)
    ok, msg = forces_close(_list_forces(s, ff, precision, 1), o.forces(), 1e-11 if precision == 0 else 1e-5)
    assert ok, msg


@pytest.mark.parametrize("n,L", [(2, 3.1), (250, 4.7), (2500, 9.0), (900, 40.0), (3000, 3000.0), (4096, 30.0),
                                 (4097, 30.0), (32768, 40.0), (32769, 40.0), (140000, 38.0)])
def test_creation_scan_matches_oracle(n, L):
    """One sweep over beads of four types, part of them not reactive, from three cells per edge to hundreds: a cloud
    about the corner of the box (more candidates than a thread's rows in the small boxes, none in the large), rules
    with and without a wildcard, lists of one thread and of four per bead, flags
    that fill a scan's tiles to the last and begin one more.  The bonds are the oracle's."""
    rng = np.random.default_rng(n + 7)
    x = rng.uniform(0.0, L, size=(n, 3))
    k = n // 3
    x[:k] = np.mod(rng.normal(0.0, max(0.9, 0.3 * k ** (1.0 / 3.0)), size=(k, 3)), L)
    kind = rng.integers(1, 5, size=n).astype(np.int32)
    s = synth.System(L=L, x=synth.wrap(x, L), v=np.zeros((n, 3)), type=kind,
                     reactive=(rng.uniform(size=n) < 0.9).astype(np.uint8), bonds=np.zeros((0, 4), dtype=np.int32))
    if n == 2:
        s.x[:] = [[0.05, 1.0, 3.05], [3.05, 1.0, 0.05]]
        s.type[:], s.reactive[:] = [1, 2], 1
    rules = synth.RuleSet(every=1, rules=[("create", 1, 1, 2, 0.99, 1.0), ("create", 2, 0, 3, 0.7, 0.6)])
    g, o = both(s, synth.ForceField(), rules, seed=3)
    g.sweep_now()
    o.sweep_now()
    assert np.array_equal(g.bonds(), o.bonds())
    if L < 100:
        assert len(g.bonds()) > 0


@pytest.mark.parametrize("want", ["both", "x", "v", "one buffer"])
def test_state_into_device_buffers(want):
    """The state written straight into the caller's device memory, or copied there where the two results share it
    (the velocities, which come second, stand): the bytes that host arrays receive."""
    import torch
    import paper_1108_4214_amd as pk
    n = 257
    rng = np.random.default_rng(4)
    s = synth.System(L=12.0, x=rng.uniform(0.0, 12.0, size=(n, 3)), v=rng.normal(size=(n, 3)),
                     type=np.ones(n, dtype=np.int32), reactive=np.zeros(n, dtype=np.uint8),
                     bonds=np.zeros((0, 4), dtype=np.int32))
    g = pk.System(n, s.L, 3, 0).configure(s, synth.ff_dpd(gamma_dpd=0.0), synth.RuleSet(every=0), generate=False)
    g.step(3)
    x, v = g.state()
    room = torch.full((2 * n, 3), -1.0, dtype=torch.float64, device="cuda")
    a, b = room[:n], room[n:]
    pk.db_get_state(g.ctx, None if want == "v" else a, None if want == "x" else (a if want == "one buffer" else b))
    room = room.cpu().numpy()
    first = {"v": -np.ones((n, 3)), "one buffer": v}.get(want, x)
    assert np.array_equal(room[:n], first)
    assert np.array_equal(room[n:], v if want in ("both", "v") else -np.ones((n, 3)))


def test_repeated_members_of_a_dihedral_come_back_once():
    """Dihedrals that name a bead twice (it holds such an entry twice), one of them set twice: the lists read from the
    device, and read again after they went back to it with an edit, are those set."""
    import paper_1108_4214_amd as pk
    rng = np.random.default_rng(5)
    d = np.array([[1, 0, 1, 2, 0], [1, 0, 1, 2, 0], [2, 0, 1, 2, 0], [1, 0, 1, 2, 3], [1, 0, 1, 1, 3], [1, 1, 2, 1, 3],
                  [3, 2, 2, 0, 3]], dtype=np.int32)
    s = synth.System(L=12.0, x=rng.uniform(0.0, 12.0, size=(4, 3)), v=np.zeros((4, 3)), type=np.ones(4, dtype=np.int32),
                     reactive=np.zeros(4, dtype=np.uint8), bonds=np.zeros((0, 4), dtype=np.int32), dihedrals=d)
    g = pk.System(s.n, s.L, 3).configure(s, synth.ForceField(), synth.RuleSet(every=0))
    want = d[np.lexsort((d[:, 0], d[:, 4], d[:, 3], d[:, 2], d[:, 1]))]
    for _ in range(2):
        g.sweep_now()
        g.set_step(g.stats()["steps"] + 1)
        assert np.array_equal(g.dihedrals(), want)
        pk.db_set_reactive(g.ctx, np.zeros(4, dtype=np.uint8))


@pytest.mark.parametrize("gamma", [0.0, 20.0])
@pytest.mark.parametrize("precision", [0, 1])
def test_dpd_energy_of_beads_on_one_point(precision, gamma):
    """The soft pair energy and its virial are finite at zero separation (a rc / 2 and 0), where the force has no
    direction.  The second pair adds a rc / 2 (1 - 1/4)^2 and the virial a (1 - 1/4) / 4."""
    import paper_1108_4214_amd as pk
    s = synth.System(L=9.0, x=np.array([[1.0, 2.0, 3.0], [1.0, 2.0, 3.0], [6.0, 6.0, 6.0], [6.25, 6.0, 6.0]]),
                     v=np.zeros((4, 3)), type=np.ones(4, dtype=np.int32), reactive=np.zeros(4, dtype=np.uint8),
                     bonds=np.zeros((0, 4), dtype=np.int32))
    g = pk.System(s.n, s.L, 3, precision).configure(s, synth.ff_dpd(gamma_dpd=gamma), synth.RuleSet(every=0))
    e = g.energy()
    tol = 1e-12 if precision == 0 else 1e-5   # as in the other evaluations
    assert abs(e[1] - 12.5 * (1.0 + 0.5625)) <= 20.0 * tol and abs(e[5] - 25.0 * 0.75 * 0.25) <= 20.0 * tol, e


@pytest.mark.parametrize("precision", [0, 1])
def test_angles_of_beads_close_together(precision):
    """Separations down to 1e-16 at the corner of the box, where positions resolve them: a wide and a slight bend, both
    ends alike.  A force is good to some twenty roundings over the sine of the bend, the oracle's to as many of its own,
    relative to the largest of the angle."""
    for size in (1e-3, 1e-8, 1e-11, 1e-16):
        for bend in (1e-3, 0.3, 1.2):
            x = size * np.array([[3.0, 1.0, 2.0], [2.0, 1.0, 2.0],
                                 [2.0 - math.cos(bend), 1.0 + math.sin(bend), 2.0]])
            s = synth.System(L=9.0, x=x, v=np.zeros((3, 3)), type=np.ones(3, dtype=np.int32),
                             reactive=np.zeros(3, dtype=np.uint8),   # bonded, so that no pair interacts
                             bonds=np.array([[0, 1, 1, 1], [1, 2, 1, 1]], dtype=np.int32),
                             angles=np.array([[1, 0, 1, 2]], dtype=np.int32))
            ff = synth.ForceField(gamma=0.0, exclude_depth=2)
            ff.bonds, ff.angles = {1: (0.0, 1.0)}, {1: (10.0, math.pi)}
            g, o = both(s, ff, synth.RuleSet(every=0), precision=precision, generate=False)
            f, want = g.forces(), o.forces()
            tol = 40.0 * (2.0 ** -53 if precision == 0 else 2.0 ** -24) / math.sin(bend)
            assert np.abs(f - want).max() <= tol * np.abs(want).max(), (size, bend, f, want)


@pytest.mark.parametrize("precision", [0, 1])
def test_energy_of_a_collapsed_system(precision):
    """Thousands of beads within reach of each other: the oracle's energies (sums of 2e6 soft pairs, each good to some
    twenty roundings), and a time that grows with the neighbours of a bead (3.8 times from 2,000 to 8,000 beads, which
    do not fill the GPU) and not with their square (14 times, by a scan for every 28 of them)."""
    import time
    import paper_1108_4214_amd as pk
    least = []
    for n in (2000, 8000):
        rng = np.random.default_rng(n)
        d = rng.normal(size=(n, 3))
        d *= 0.45 * rng.uniform(size=(n, 1)) ** (1.0 / 3.0) / np.linalg.norm(d, axis=1)[:, None]
        s = synth.System(L=20.0, x=10.0 + d, v=np.zeros_like(d), type=np.ones(n, dtype=np.int32),
                         reactive=np.zeros(n, dtype=np.uint8), bonds=np.zeros((0, 4), dtype=np.int32))
        ff = synth.ff_dpd(gamma_dpd=0.0)
        g = pk.System(n, s.L, 3, precision).configure(s, ff, synth.RuleSet(every=0))
        e = g.energy()
        if n == 2000:
            import oracle
            o = oracle.Oracle.from_system(s, ff, synth.RuleSet(every=0), seed=3).energy()
            tol = 1e-12 if precision == 0 else 1e-5
            assert np.all(np.abs(e - o) <= 10 * tol * np.maximum(1.0, np.abs(o))), (e, o)
        t = []
        for _ in range(5):
            t0 = time.perf_counter()
            g.energy()
            t.append(time.perf_counter() - t0)
        least.append(min(t))
    assert least[1] < 8.0 * least[0], least


def _apart(g, o, s):
    d = g.state()[0] - o.state()[0]
    return np.abs(d - s.L * np.round(d / s.L)).max()


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("skin", [0.05, 0.09, 0.15])
def test_dpd_blocks_cut_short_follow_the_oracle(skin, graph):
    """Blocks that end early where the step exchanges the velocity buffers too, with launches and graphs.  Soft forces
    (a = 25, a friction of 5) leave the rounding of 20 steps as it is."""
    import paper_1108_4214_amd as pk
    s = synth.dpd_solution(4, 6, 1500, 3.0, 11, 21, T=2.0)
    g, o = both(s, synth.ff_dpd(T=2.0, gamma_dpd=5.0), synth.rules_t2(p=0.7, every=7), seed=9)
    pk.db_tune(g.ctx, skin, 2)
    pk.db_graph(g.ctx, graph)
    for k in (9, 1, 10):
        g.step(k)
        o.step(k)
    assert g.stats()["rollbacks"] > 0 and g.stats()["steps"] == 20
    assert _apart(g, o, s) < 1e-9
    v, w = g.state()[1], o.state()[1]
    assert np.abs(v - w).max() < 1e-7


@pytest.mark.parametrize("graph", [0, 1])
def test_batch_and_mixed_blocks_cut_short(graph):
    """A batch whose fastest replica ends the blocks of all, and a mixed run: float forces are good to 1e-5 of some
    hundred, so 24 steps of 0.005 put positions off by 24^2 / 2 x 0.005^2 x 1e-3 at most."""
    import paper_1108_4214_amd as pk
    rules = synth.rules_t2(p=0.7, every=7, r_kill=1.35)
    reps = []
    for r, T in enumerate((0.2, 2.0, 0.5)):
        s = synth.single_strands(20 + 3 * r, 6, L=11.0, seed_w=3 + r, seed_d=4 + r, T=T)
        reps.append((s, *both(s, synth.ff_t2(T0=T, T1=T), rules, seed=9 + r)))
    s, ff = reps[1][0], synth.ff_t2(T0=2.0, T1=2.0)
    mixed = pk.System(s.n, s.L, 10, 1).configure(s, ff, rules)
    b = pk.Batch([g for _, g, _ in reps])
    for h in (b, mixed):
        pk.db_tune(h.ctx, 0.08, 2)
        pk.db_graph(h.ctx, graph)
        for _ in range(3):
            h.step(8)
        assert h.stats()["rollbacks"] > 0 and h.stats()["steps"] == 24
    for r, (s, _, o) in enumerate(reps):
        o.step(24)
        d = b.replica_state(r)[0] - o.state()[0]
        assert np.abs(d - s.L * np.round(d / s.L)).max() < 1e-9
        if r == 1:
            assert _apart(mixed, o, s) < 1e-5


@pytest.mark.parametrize("tiles,graph", [(0, 0), (0, 1), (1, 0)])
def test_block_with_a_kept_list_cut_short(tiles, graph):
    """A list kept across a sweep, its displacement bound above 0 at the block's begin.  One bead of a resting lattice is
    pulled, so its speed is the step number in units of F dt: 174 units of F dt^2 since the list of step 8, 400 more
    expected of the block from step 20 (1.25 times that are asked for), 570 made until its last step.  Half the skin is
    710 units: kept, and cut."""
    import paper_1108_4214_amd as pk
    k = np.arange(64)
    s = synth.System(L=12.0, x=1.5 + 3.0 * np.stack([k % 4, k // 4 % 4, k // 16], 1), v=np.zeros((64, 3)),
                     type=np.ones(64, dtype=np.int32), reactive=np.ones(64, dtype=np.uint8),
                     bonds=np.zeros((0, 4), dtype=np.int32))
    ff = synth.ForceField(gamma=0.0, dt=0.005)
    pulled, f = np.array([5], dtype=np.int32), np.array([[10.0, 0.0, 0.0]])
    g, o = both(s, ff, synth.RuleSet(every=20), seed=9)
    pk.db_external_force(g.ctx, pulled, f)
    o.set_external_force(pulled, f)
    pk.db_tune(g.ctx, 2.0 * 710.0 * 10.0 * ff.dt ** 2, 4)
    pk.db_tile_shape(g.ctx, tiles)
    pk.db_graph(g.ctx, graph)
    g.step(8)
    g.step(12)
    assert g.stats()["rollbacks"] == 0 and g.stats()["list_patches"] == 0
    g.step(20)
    st = g.stats()
    assert st["list_patches"] == 1 and st["rollbacks"] == 1 and st["steps"] == 40
    o.step(40)
    assert _apart(g, o, s) < 1e-9
    assert np.abs(g.state()[1] - o.state()[1]).max() < 1e-9


def test_profile_counts_the_steps_made():
    """Launches after a block's early end store nothing: with every launch timed, their number is that of the steps."""
    import paper_1108_4214_amd as pk
    s = synth.single_strands(24, 6, L=11.0, seed_w=3, seed_d=4, T=2.0)
    g = pk.System(s.n, s.L, 9).configure(s, synth.ff_t2(T0=2.0, T1=2.0), synth.rules_t2(every=7))
    pk.db_tune(g.ctx, 0.08, 2)
    pk.db_profile(g.ctx, 1)
    g.step(24)
    assert g.stats()["rollbacks"] > 0
    us, launches = pk.db_step_kernel_time(g.ctx)
    assert launches == 24 and us > 0.0


@pytest.mark.parametrize("form", ["dense one thread", "dense four threads", "dense few beads", "far box", "small boxes", "mixed batch"])
def test_list_forms_match_oracle(form):
    """Lists by the float scan: longer than the quantised scan's rows hold (a skin of 0.5 at density 3, about 44 entries,
    with one and with four threads' share of beads), in an edge beyond its reach, in boxes of two cells per edge, and a
    batch where some boxes are served and some not.  Forces of soft pairs as in the other list builds."""
    import paper_1108_4214_amd as pk
    import oracle
    ff = dataclasses.replace(synth.ff_dpd(gamma_dpd=0.0), dt=2.0 ** -10)
    sizes = {"dense one thread": [(132000, 35.3)], "dense four threads": [(66000, 28.0)], "dense few beads": [(6000, 12.6)], "far box": [(4000, 2500.0)],
             "small boxes": [(60, 2.9), (81, 3.0)], "mixed batch": [(3000, 10.0), (500, 2000.0), (70, 2.9)]}[form]
    for order in (1, -1):
        reps, want = [], []
        for n, L in sizes[::order]:
            rng = np.random.default_rng(n)
            x = rng.uniform(0.0, L, size=(n, 3))
            if L > 1000.0:
                x[:n // 2] = np.mod(rng.normal(0.0, 4.0, size=(n // 2, 3)), L)
            s = synth.System(L=L, x=synth.wrap(x, L), v=np.zeros((n, 3)), type=np.ones(n, dtype=np.int32),
                             reactive=np.zeros(n, dtype=np.uint8), bonds=np.zeros((0, 4), dtype=np.int32))
            reps.append(pk.System(n, L, 1, 0).configure(s, ff, synth.RuleSet(every=0), generate=False))
            o = oracle.Oracle.from_system(s, ff, synth.RuleSet(every=0), seed=1, generate=False)
            want.append(o.forces())
        g = pk.Batch(reps) if len(reps) > 1 else reps[0]
        pk.db_tune(g.ctx, 0.5 if form.startswith("dense") else 0.02, 8)
        g.step(1)
        got = [g.replica_state(r)[1] for r in range(len(reps))] if len(reps) > 1 else [g.state()[1]]
        for v, f in zip(got, want):
            ok, msg = forces_close(v / ff.dt, f, 1e-11)
            assert ok, msg
        if len(sizes) == 1:
            break


@pytest.mark.parametrize("beads", [60, 1499, 1501])
def test_dpd_batches_of_small_and_large_boxes(beads):
    """Steps of DPD batches in boxes on both sides of the size that chooses the step kernel's registers, mixed, against
    the oracle: float forces are good to 1e-5 of some hundred, over five steps of 0.01 with a friction of 5."""
    import paper_1108_4214_amd as pk
    ff = synth.ff_dpd(gamma_dpd=5.0)
    reps = []
    for r in range(3):
        s = synth.random_gas(beads, (beads / 3.0) ** (1.0 / 3.0), seed=r)
        reps.append((s, *both(s, ff, synth.RuleSet(every=0), seed=9 + r, precision=1, generate=False)))
    b = pk.Batch([g for _, g, _ in reps])
    b.step(5)
    for r, (s, _, o) in enumerate(reps):
        o.step(5)
        x, v = b.replica_state(r)
        d = x - o.state()[0]
        assert np.abs(d - s.L * np.round(d / s.L)).max() < 5e-6
        assert np.abs(v - o.state()[1]).max() < 1e-4


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("pair", ["wca", "dpd"])
@pytest.mark.parametrize("size", [0.0, 2.5, 4.6])
def test_evaluation_in_a_far_box_matches_oracle(size, pair, precision):
    """Edges beyond the quantised scan's reach: a sparse box, a cluster whose beads fit the staged rows and one whose
    central beads do not, half of it across the corner of the box.  Soft pairs as in the other evaluations; WCA beads on
    a lattice with 2 % noise, whose forces go with the 14th power of distances good to a rounding of the edge in
    float input and to 1e-13 in double."""
    n, L = 700, 2000.0
    rng = np.random.default_rng(7)
    if pair == "wca":
        k = np.arange(n)
        x = np.stack([k % 9, k // 9 % 9, k // 81], 1) * (1.08 if size else 200.0) + rng.normal(0.0, 0.02, size=(n, 3)) - 3.0
        ff = synth.ForceField(gamma=0.0)
    else:
        x = rng.normal(0.0, size, size=(n, 3)) if size else rng.uniform(0.0, L, size=(n, 3))
        ff = synth.ff_dpd(gamma_dpd=20.0)
    s = synth.System(L=L, x=synth.wrap(np.mod(x, L), L), v=rng.normal(size=(n, 3)), type=np.ones(n, dtype=np.int32),
                     reactive=np.zeros(n, dtype=np.uint8), bonds=np.zeros((0, 4), dtype=np.int32))
    g, o = both(s, ff, synth.RuleSet(every=0), precision=precision, generate=False)
    tol = 1e-10 if precision == 0 else 1e-5
    ok, msg = forces_close(g.forces(), o.forces(), tol)
    assert ok, msg
    eg, eo = g.energy(), o.energy()
    assert np.all(np.abs(eg - eo) <= 10 * tol * np.maximum(1.0, np.abs(eo))), (eg, eo)


@pytest.mark.parametrize("order", [1, -1])
def test_creation_scan_of_a_mixed_batch(order):
    """A sweep over a batch whose first box chooses the threads per bead, one that the quantised scan serves and one that
    it does not, either first: the bonds of the standalone handles."""
    import paper_1108_4214_amd as pk
    rules = synth.RuleSet(every=1, rules=[("create", 1, 1, 2, 0.99, 1.0), ("create", 2, 0, 3, 0.7, 0.6)])
    reps = []
    for n, L in [(2500, 9.0), (3000, 2500.0), (40, 3.4)][::order]:
        rng = np.random.default_rng(n)
        x = np.mod(rng.normal(0.0, 3.0, size=(n, 3)), L) if L > 1000.0 else rng.uniform(0.0, L, size=(n, 3))
        s = synth.System(L=L, x=synth.wrap(x, L), v=np.zeros((n, 3)), type=rng.integers(1, 5, size=n).astype(np.int32),
                         reactive=np.ones(n, dtype=np.uint8), bonds=np.zeros((0, 4), dtype=np.int32))
        reps.append(pk.System(n, L, n).configure(s, synth.ForceField(), rules))
    b = pk.Batch(reps)
    b.sweep_now()
    rows, off = b.bonds(), 0
    for g in reps:
        g.sweep_now()
        mine = rows[(rows[:, 0] >= off) & (rows[:, 0] < off + g.n)].copy()
        mine[:, :2] -= off
        assert len(mine) > 0 and np.array_equal(mine, g.bonds())
        off += g.n


@pytest.mark.parametrize("pair", ["wca", "dpd"])
def test_a_system_near_rest_keeps_its_lists(pair):
    """Speeds of 1e-12 admit more steps per list than an integer holds: blocks are as long as they may be (64 steps
    after a first of 8), not single steps."""
    import paper_1108_4214_amd as pk
    k = np.arange(125)
    rng = np.random.default_rng(3)
    s = synth.System(L=12.5, x=1.0 + 2.5 * np.stack([k % 5, k // 5 % 5, k // 25], 1), v=1e-12 * rng.normal(size=(125, 3)),
                     type=np.ones(125, dtype=np.int32), reactive=np.zeros(125, dtype=np.uint8),
                     bonds=np.zeros((0, 4), dtype=np.int32))
    ff = synth.ForceField(gamma=0.0) if pair == "wca" else synth.ff_dpd(gamma_dpd=0.0)
    g = pk.System(s.n, s.L, 3).configure(s, ff, synth.RuleSet(every=0))
    g.step(8 + 3 * 64)
    assert g.stats()["rebuilds"] <= 4 and g.stats()["steps"] == 200
