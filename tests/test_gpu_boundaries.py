"""GPU builds at the edges of tiles, groups and launch rules, against the oracle.

Sizes sit on both sides of the lines between the kernels' variants: blocks of
16 balls and groups, one quantise tile (1,024), the one-block binning (2,048),
record tiles (4,096), lanes per ball (2^13, 2^18), the joint launch of
tetrahedra and AC2 (2^16), radix tiles whose digit sums the scatter takes
(2^17), searched bucket starts (2^18) and record tiles of one block (2^22).
Simplices are equal, Sizes within the oracle comparison's tolerance.
"""
import numpy as np
import pytest

import oracle
import synth
from parity import assert_same_complex

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def acx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_05944_amd as m
    return m


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda:0")


def _check(acx, xyz, rad, alpha, label, **opt):
    print(f"[case] {label} n={len(rad)} alpha={alpha} {opt}", flush=True)
    c = acx.ac_alpha_complex_device(_dev(xyz), _dev(rad), alpha, options=opt or None)
    assert_same_complex(c, oracle.alpha_complex(xyz, rad, alpha), label)
    return c


@pytest.mark.parametrize("n", [15, 17, 255, 257, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192])
@pytest.mark.parametrize("alpha", [0.0, 2.0])
def test_sizes(acx, n, alpha):
    m = synth.molecule(n, n)
    _check(acx, m.xyz, m.radii, alpha, "size")


@pytest.mark.parametrize("n", [65536, 65537, 131072, 131073, 262145])
def test_large_sizes(acx, n):
    m = synth.molecule(n, 5)
    _check(acx, m.xyz, m.radii, 0.0, "large size")


@pytest.mark.parametrize("n", [300, 9001])
@pytest.mark.parametrize("grow_mA,alpha", [(0, 1.0), (700, 0.0), (1400, 0.5), (1400, -6.0), (2400, 0.0)])
def test_row_lengths(acx, n, grow_mA, alpha):
    """Neighbour rows of every slot, of more than the widest (counted), and
    radii of which some vanish at a negative alpha."""
    m = synth.molecule(n, 31).with_sas(grow_mA) if grow_mA else synth.molecule(n, 31)
    _check(acx, m.xyz, m.radii, alpha, f"grown by {grow_mA}")


@pytest.mark.parametrize("cell", [1200, 10922, 10923, 16383, 16384, 60000])
def test_cell_sides(acx, cell):
    """Cells on both sides of where coordinate differences in the scanned cells
    reach 2^15, in one box of cells and in few."""
    m = synth.molecule(1500, 77)
    far = np.vstack([m.xyz, m.xyz[:40] + np.array([0.0, 65.536, 0.0])])  # apart by a multiple of 2^16
    rad = np.concatenate([m.radii, m.radii[:40]])
    _check(acx, far, rad, 0.0, f"cell {cell}", cell_mA=cell)


@pytest.mark.parametrize("side,radius,alpha", [(10, 1.5, 0.0), (10, 1.5, 2.0), (7, 2.9, 0.0)])
def test_undecided_in_every_block(acx, side, radius, alpha):
    """Lattices: the float32 test leaves simplices of every block undecided."""
    p = np.stack(np.meshgrid(*[np.arange(side) * 2.0] * 3, indexing="ij"), -1).reshape(-1, 3)
    p = p[np.random.RandomState(3).permutation(len(p))]
    _check(acx, p, np.full(len(p), radius), alpha, "lattice")


@pytest.mark.parametrize("count", [8, 9, 17])
def test_sweep_chunks(acx, count):
    """One chunk of alphas, one more, and two and one, unsorted: each complex is
    that of its own build."""
    m = synth.molecule(3000, 12)
    alphas = [round(float(a), 3) for a in np.random.RandomState(count).uniform(-1.0, 2.0, count)]
    print(f"[case] sweep of {count}", flush=True)
    X, R = _dev(m.xyz), _dev(m.radii)
    for a, c in zip(alphas, acx.ac_alpha_sweep_device(X, R, alphas)):
        single = acx.ac_alpha_complex_device(X, R, a)
        assert c.counts() == single.counts(), a
        for d in range(4):
            assert np.array_equal(c.simplices(d), single.simplices(d)), (a, d)
            assert np.array_equal(c.sizes(d), single.sizes(d)), (a, d)


@pytest.mark.parametrize("copies,grow_mA", [(43, 0), (14, 1400)])
def test_copies_of_a_molecule(acx, copies, grow_mA):
    """Batches of copies of a molecule whose size is no multiple of a wave, each
    equal to the molecule's own complex: 4.3 million balls (more record tiles than
    a block adds up), and 1.4 million with so many pairs of candidate edges that
    the triangles are counted first."""
    m = synth.molecule(100003, 9)
    m = m.with_sas(grow_mA) if grow_mA else m
    print(f"[case] batch of {copies} x {m.n}", flush=True)
    X, R = _dev(m.xyz), _dev(m.radii)
    off = np.arange(copies + 1, dtype=np.int64) * m.n
    c = acx.ac_alpha_complex_batch(X.repeat(copies, 1), R.repeat(copies), off, 0.0)
    single = acx.ac_alpha_complex_device(X, R, 0.0)
    for d in range(4):
        rows, s, z = c.molecule_rows(d), c.simplices(d), c.sizes(d)
        assert np.array_equal(np.diff(rows), np.full(copies, single.count(d)))
        want_s, want_z = single.simplices(d), single.sizes(d)
        for k in (0, 1, copies // 2, copies - 2, copies - 1):
            assert np.array_equal(s[rows[k]:rows[k + 1]] - off[k], want_s), (d, k)
            assert np.array_equal(z[rows[k]:rows[k + 1]], want_z), (d, k)


def _same_as(got, want, what):
    assert got.counts() == want.counts(), what
    for d in range(4):
        assert np.array_equal(got.simplices(d), want.simplices(d)), (what, d)
        assert np.array_equal(got.sizes(d), want.sizes(d)), (what, d)


def _on_device(c, d):
    """The d-simplices and Sizes of a device result as torch tensors."""
    import torch

    class View:
        def __init__(self, p, shape, kind):
            self.__cuda_array_interface__ = {"shape": shape, "typestr": kind, "data": (p, False), "version": 2}

    s, z = c.device_pointers(d)
    return (torch.as_tensor(View(s, (c.count(d), d + 1), "<i4"), device="cuda:0"),
            torch.as_tensor(View(z, (c.count(d),), "<f8"), device="cuda:0"))


def _replayed(acx, xyz, rad, alpha, label, headroom=1.25):
    """A recorded build replayed on its own input: no stop, and the oracle's complex."""
    print(f"[case] recorded {label} n={len(rad)} alpha={alpha}", flush=True)
    X, R = _dev(xyz), _dev(rad)
    plan = acx.Plan(X, R, np.array([0, len(rad)]), alpha, headroom=headroom)
    for _ in range(2):
        plan.launch()
        got = plan.result()
        assert plan.stopped() == 0 and plan.ordinary_builds() == 0
        assert_same_complex(got, oracle.alpha_complex(xyz, rad, alpha), label)
        got.close()
    plan.close()


@pytest.mark.parametrize("n", [300, 9001])
@pytest.mark.parametrize("kind,spacing,radius", [("beads", 4.7, 3.0), ("beads", 8.0, 3.0), ("beads", 6.1, 3.8), ("ion", 0, 2.75)])
def test_recorded_builds_of_large_radii(acx, n, kind, spacing, radius):
    """Radii whose rows usually outgrow the slots, in sets whose rows do not:
    coarse beads, far apart ones, and one ion among atoms."""
    if kind == "ion":
        m = synth.molecule(n, 21)
        xyz, rad = m.xyz, m.radii.copy()
        rad[n // 3] = radius
    else:
        rng = np.random.RandomState(n)
        side = int(np.ceil(n ** (1.0 / 3.0)))
        xyz = np.stack(np.meshgrid(*[np.arange(side) * spacing] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
        xyz, rad = xyz + rng.uniform(-0.3, 0.3, xyz.shape), np.full(n, radius)
    _replayed(acx, xyz, rad, 0.0, kind)


@pytest.mark.parametrize("a,radius", [(3.8, 1.95), (3.9, 1.98), (4.2, 2.2)])
@pytest.mark.parametrize("headroom", [1.0, 2.0])
def test_recorded_lattices(acx, a, radius, headroom):
    """Close packings, about 14 candidate tetrahedra a ball: the groups' slabs of a
    recorded build hold what the recorded input needs."""
    g = np.stack(np.meshgrid(*[np.arange(10)] * 3, indexing="ij"), -1).reshape(-1, 1, 3).astype(float)
    p = (g + np.array([[0, 0, 0], [0, .5, .5], [.5, 0, .5], [.5, .5, 0]])).reshape(-1, 3) * a
    rng = np.random.RandomState(7)
    p = rng.permutation(p + rng.uniform(-0.02, 0.02, p.shape))
    _replayed(acx, p, np.full(len(p), radius), 0.0, f"lattice {a}", headroom)


@pytest.mark.parametrize("copies,headroom", [(9, 16.0), (130, 1.0)])
def test_recorded_builds_with_counted_triangles(acx, copies, headroom):
    """Recorded batches of copies of a molecule at alpha = 2 whose pairs of candidate
    edges are more than a build makes room for: by the headroom alone, and by
    themselves. Every copy has the molecule's own complex."""
    import torch
    m = synth.molecule(100003, 9)
    X, R = _dev(m.xyz).repeat(copies, 1), _dev(m.radii).repeat(copies)
    off = np.arange(copies + 1, dtype=np.int64) * m.n
    single = acx.ac_alpha_complex_device(X[:m.n].clone(), R[:m.n].clone(), 2.0)
    up = single.simplices(1)[:, 0]  # least ids of the kept edges: the pairs are at least theirs
    c = np.bincount(up).astype(np.int64)
    assert (c * (c - 1) // 2).sum() * copies * headroom > 1 << 28
    print(f"[case] recorded batch of {copies} x {m.n}, headroom {headroom}", flush=True)
    plan = acx.Plan(X, R, off, 2.0, headroom=headroom)
    for _ in range(2):
        plan.launch()
        got = plan.result()
        assert plan.stopped() == 0 and plan.ordinary_builds() == 0
        torch.cuda.synchronize()
        for d in range(4):
            rows = got.molecule_rows(d)
            assert np.array_equal(np.diff(rows), np.full(copies, single.count(d))), d
            s, z = _on_device(got, d)
            for k in (0, copies // 2, copies - 1):
                assert np.array_equal(s[rows[k]:rows[k + 1]].cpu().numpy() - off[k], single.simplices(d)), (d, k)
                assert np.array_equal(z[rows[k]:rows[k + 1]].cpu().numpy(), single.sizes(d)), (d, k)
        got.close()
    plan.close()


@pytest.mark.parametrize("copies", [32, 33, 65])
def test_gradients_of_copies(acx, copies):
    """Corners sorted by ball on both sides of 2^17 and past 2^18 balls: in a batch of
    copies every ball's gradient is that of the molecule's own complex, bit for bit."""
    import torch
    m = synth.molecule(4096, 13)
    X, R = _dev(m.xyz), _dev(m.radii)
    g = torch.tensor([0.7, -0.4], dtype=torch.float64, device="cuda:0")
    one = acx.ac_alpha_complex_device(X, R, 0.0)
    want_x, want_r = acx.ac_union_measure_backward(one, X, R, g)
    print(f"[case] gradients of {copies} copies, {copies * m.n} balls", flush=True)
    XX, RR = X.repeat(copies, 1), R.repeat(copies)
    c = acx.ac_alpha_complex_batch(XX, RR, np.arange(copies + 1, dtype=np.int64) * m.n, 0.0)
    dx, dr = acx.ac_union_measure_backward(c, XX, RR, g)
    assert torch.equal(dx.view(copies, m.n, 3), want_x.expand(copies, m.n, 3))
    assert torch.equal(dr.view(copies, m.n), want_r.expand(copies, m.n))


def test_replayed_rows_are_complete_on_return(acx):
    """The result of a replay on a stream of its own: its rows are read through
    another stream at once, and the next replay and its result come before the
    first is looked at on the host."""
    import torch
    m = synth.molecule(200000, 5)
    X, R = _dev(m.xyz), _dev(m.radii)
    shifted = _dev(m.xyz + 3.0)
    want = [acx.ac_alpha_complex_device(x, R, 0.0) for x in (X, shifted)]
    src = X.clone()
    plan = acx.Plan(src, R, np.array([0, m.n]), 0.0, headroom=1.5)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    print("[case] replays on two streams", flush=True)
    for rep in range(3):
        got = []
        for k, (st, x) in enumerate(((a, X), (b, shifted))):
            with torch.cuda.stream(st):
                src.copy_(x)
                plan.launch()
                got.append(plan.result())
            assert plan.stopped() == 0
            if rep % 2 == k:  # at once
                _same_as(got[k], want[k], (rep, k))
        for k in (0, 1):
            _same_as(got[k], want[k], (rep, k))


@pytest.mark.parametrize("n", [2049, 2304, 9001])
@pytest.mark.parametrize("cell", [12000, 17000, 22000, 60000])
def test_crowded_cells(acx, n, cell):
    """Cells of some ten to all of the balls: buckets whose cells are ranked in LDS
    and buckets that go in chunks."""
    m = synth.molecule(n, 78)
    _check(acx, m.xyz, m.radii, 0.0, f"cell {cell}", cell_mA=cell)


@pytest.mark.parametrize("far", [400.0, 640.0])
def test_dense_ball_in_a_large_box(acx, far):
    """One atom far away makes most cells empty: buckets of ordinary cells with more
    than 2,048 balls."""
    m = synth.molecule(100003, 9)
    xyz = np.vstack([m.xyz - m.xyz.mean(0) - [far / 2, 0.0, 0.0], [[far / 2, 0.0, 0.0]]])
    _check(acx, xyz, np.append(m.radii, 1.5), 0.0, f"one atom {far} A away")


@pytest.mark.parametrize("n,cell", [(3000, 60000), (30000, 60000), (30000, 3600)])
@pytest.mark.parametrize("first,second", [(0, 1), (0, -1), (-2, -1), (1500, 2900)])
def test_equal_centres_are_found(acx, n, cell, first, second):
    m = synth.molecule(n, 79)
    xyz = m.xyz.copy()
    xyz[second] = xyz[first]
    print(f"[case] equal centres n={n} cell={cell} {first} {second}", flush=True)
    with pytest.raises(acx.AlphaCxError) as ei:
        acx.ac_alpha_complex_device(_dev(xyz), _dev(m.radii), 0.0, options={"cell_mA": cell})
    assert ei.value.status == 2


@pytest.mark.parametrize("n,copies", [(300, 9), (300, 70), (2500, 3), (20, 2000)])
@pytest.mark.parametrize("cell", [0, 60000])
def test_equal_centres_of_molecules_in_crowded_buckets(acx, n, copies, cell):
    """Copies of a molecule at the same place, whose cells share crowded buckets, are
    no equal centres; two equal ones inside the last copy are."""
    m = synth.molecule(n, 80)
    X, R, off = _dev(m.xyz).repeat(copies, 1), _dev(m.radii).repeat(copies), np.arange(copies + 1, dtype=np.int64) * n
    options = {"cell_mA": cell} if cell else None
    print(f"[case] {copies} copies of {n} at one place, cell {cell}", flush=True)
    got = acx.ac_alpha_complex_batch(X, R, off, 0.0, options=options)
    single = acx.ac_alpha_complex_device(X[:n].clone(), R[:n].clone(), 0.0)
    for d in range(4):
        rows, s, z = got.molecule_rows(d), got.simplices(d), got.sizes(d)
        assert np.array_equal(np.diff(rows), np.full(copies, single.count(d))), d
        for k in (0, copies // 2, copies - 1):
            assert np.array_equal(s[rows[k]:rows[k + 1]] - off[k], single.simplices(d)), (d, k)
            assert np.array_equal(z[rows[k]:rows[k + 1]], single.sizes(d)), (d, k)
    X[-1] = X[-n]
    with pytest.raises(acx.AlphaCxError) as ei:
        acx.ac_alpha_complex_batch(X, R, off, 0.0, options=options)
    assert ei.value.status == 2


@pytest.mark.parametrize("n", [40, 300, 1500])
@pytest.mark.parametrize("grow_mA,alpha", [(2000, 0.0), (3500, 0.0), (4500, -20.0)])
def test_long_rows_in_few_balls(acx, n, grow_mA, alpha):
    """Rows so long that a group is a few balls, or one."""
    m = synth.molecule(n, 32).with_sas(grow_mA)
    _check(acx, m.xyz, m.radii, alpha, f"grown by {grow_mA}")


def _hub(k, hub, ball):
    """k balls spread over a sphere around a hub that their grown spheres cross."""
    i = np.arange(k) + 0.5
    phi, z = np.pi * (1 + 5 ** 0.5) * i, 1 - 2 * i / k
    p = np.stack([np.cos(phi) * np.sqrt(1 - z * z), np.sin(phi) * np.sqrt(1 - z * z), z], -1) * (hub + ball * 2 / 3)
    return np.vstack([[0, 0, 0], p + np.random.RandomState(k).uniform(-0.02, 0.02, p.shape)]), np.append(hub, np.full(k, ball))


@pytest.mark.parametrize("k", [60, 66, 130, 700, 1500])
@pytest.mark.parametrize("hub,ball", [(7.9, 0.45), (2.2, 0.15)])
@pytest.mark.parametrize("place", [0, 1, -1])
def test_hubs(acx, k, hub, ball, place):
    """One ball with a long row, first, in the middle and last by input id, alone and
    beside a molecule: its edges' items on both sides of what a row may hold."""
    xyz, rad = _hub(k, hub, ball)
    at = {0: 0, 1: k // 2, -1: k}[place]
    order = np.concatenate([np.arange(1, at + 1), [0], np.arange(at + 1, k + 1)])
    xyz, rad = xyz[order], rad[order]
    _check(acx, xyz, rad, 0.0, f"hub of {k} at {at}")
    m = synth.molecule(300, 33)
    _check(acx, np.vstack([xyz, m.xyz - m.xyz.mean(0) + [30.0, 0, 0]]), np.append(rad, m.radii), 0.0, "hub and molecule")


@pytest.mark.parametrize("n", [1025, 9001, 262145])
@pytest.mark.parametrize("share,radius,alpha", [(0, 2.75, 0.0), (32, 2.75, 0.0), (31, 2.75, 0.0), (1024, 3.4, 0.0), (40, 3.4, 0.0), (40, 2.5, 1.0)])
@pytest.mark.parametrize("clump", [False, True])
def test_few_large_balls(acx, n, share, radius, alpha, clump):
    """One ion, and one ball in 1,024, 40, 32 and 31, spread over a molecule or side by side
    (rows longer than the slots of 32): as one call, of a batch and of a sweep."""
    m = synth.molecule(n, 34)
    k = n // share if share else 1
    at = np.argsort(((m.xyz - m.xyz.mean(0)) ** 2).sum(1))[:k] if clump else np.arange(k) * (n // k)
    rad = m.radii.copy()
    rad[at] = radius
    _check(acx, m.xyz, rad, alpha, f"{k} of {radius} A")
    if n > 10000:
        return
    X, R = _dev(m.xyz), _dev(rad)
    single = acx.ac_alpha_complex_device(X, R, alpha)
    two = acx.ac_alpha_complex_batch(X.repeat(2, 1), R.repeat(2), np.array([0, n, 2 * n]), alpha)
    for d in range(4):
        rows, s = two.molecule_rows(d), two.simplices(d)
        for c in (0, 1):
            assert np.array_equal(s[rows[c]:rows[c + 1]] - c * n, single.simplices(d)), (c, d)
    print(f"[case] sweep with {k} of {radius} A n={n}", flush=True)
    swept = acx.ac_alpha_sweep_device(X, R, [alpha - 0.5, alpha])
    _same_as(swept[1], single, "sweep")


@pytest.mark.parametrize("n,rows", [(40, 30), (150, 60), (150, 140), (700, 40), (700, 100), (2100, 40)])
@pytest.mark.parametrize("beside", [0, 9000])
def test_small_balls_close_together(acx, n, rows, beside):
    """Long rows of small radii, alone and beside a molecule (whose short rows keep
    the kernels of small radii), also without allocation."""
    import torch
    rng = np.random.RandomState(n + rows)
    side = (n * 4 / 3 * np.pi * 0.8 ** 3 / rows) ** (1 / 3)
    xyz, rad = rng.uniform(-side / 2, side / 2, (n, 3)), rng.uniform(0.35, 0.45, n)
    if beside:
        m = synth.molecule(beside, 35)
        xyz, rad = np.vstack([xyz, m.xyz - m.xyz.mean(0) + [90.0, 0, 0]]), np.append(rad, m.radii)
    _check(acx, xyz, rad, 0.0, f"rows of {rows}")
    X, R = _dev(xyz), _dev(rad)
    single = acx.ac_alpha_complex_device(X, R, 0.0)
    simp = [torch.empty((single.count(d), d + 1), dtype=torch.int32, device="cuda:0") for d in range(4)]
    size = [torch.empty(single.count(d), dtype=torch.float64, device="cuda:0") for d in range(4)]
    assert list(acx.ac_alpha_complex_noalloc(X, R, 0.0, simp, size)) == list(single.counts())
    torch.cuda.synchronize()
    for d in range(4):
        assert np.array_equal(simp[d].cpu().numpy(), single.simplices(d)), d
        assert np.array_equal(size[d].cpu().numpy(), single.sizes(d)), d
    _same_as(acx.ac_alpha_sweep_device(X, R, [0.0, -0.05])[0], single, "sweep")
    # no apex balls: the candidate tetrahedra outgrow the slabs of a group's slices
    _same_as(acx.ac_alpha_complex_device(X, R, 0.0, options={"force_exact": 1}), single, "exact")
    _same_as(acx.ac_alpha_sweep_device(X, R, [0.0, -0.05], options={"force_exact": 1})[0], single, "exact sweep")
