"""GPU tests of the list builder's forms: the leaves' tiles, the one-launch and
the counted block split and first expansion pass, and boxes without particles."""
import numpy as np
import pytest

import workloads as W
from workloads import BoxParams

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1802_09824_amd as m
    return m


def dev(a, dtype):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype)


# tiles of 512 particles up to 131072 of them, of 2048 beyond
@pytest.mark.parametrize("n,leaf_max", [(1, 1), (2, 1024), (511, 1), (512, 32), (513, 7), (1025, 1024), (2049, 600),
                                        (5000, 1023), (131072, 32), (131073, 32), (133121, 1000)])
def test_leaf_tiles_bit_exact(pp, oracle_mod, n, leaf_max):
    """Leaves whose runs reach over tile edges, against the oracle's tree."""
    rng = np.random.default_rng(n + leaf_max)
    p = W.BoxParams(L=50.0, rs=1.0, rcut=4.5, eps=0.02, leaf_max=leaf_max)
    pos = W.mixture(rng, n, p.L, 0.6, max(1, n // 400))
    if n > 600:
        pos[:, 100:160] = pos[:, 100:101]            # a leaf at the finest level
    st = oracle_mod.structure(pos, p)
    lv = pp.pp_build_leaves(dev(st["sorted_keys"].view(np.int64), torch.int64), dev(pos[:, st["perm"]], torch.float64), p)
    got, ref = lv.export(), st["leaves"]
    assert got["begin"].size == ref["begin"].size
    for k in ("begin", "count", "level", "prefix"):
        assert np.array_equal(got[k].astype(np.int64), ref[k].astype(np.int64)), k
    assert np.array_equal(got["lo"].astype(np.int64), st["lo"])
    assert np.array_equal(got["hi"].astype(np.int64), st["hi"])


@pytest.mark.parametrize("n,leaf_max,mesh", [(131072, 32, 40), (131073, 3, 40), (262144, 32, 50), (262145, 5, 50),
                                             (300000, 2, 24)])
def test_builder_forms_cover_every_neighbour(pp, oracle_mod, n, leaf_max, mesh):
    """Pair counts from the lists (FP64 test of every listed source) against
    the oracle's brute-force counts, on both sides of 4096 chunks (one launch
    or three for the block split and the first pass) and of 131072 particles
    (the start level), with leaves small enough that expansion passes follow,
    in wide boxes (several blocks per chunk) and on periodic faces."""
    rng = np.random.default_rng(n)
    p0 = BoxParams.from_mesh(60.0, mesh)
    p = W.BoxParams(**{**p0.__dict__, "leaf_max": leaf_max})
    pos = W.mixture(rng, n, p.L, 0.4, n // 500)
    mass = W.equal_masses(n)
    plan = pp.Plan(p, n)
    for _ in range(2):                               # guessed, then known start level and capacities
        plan.accel(dev(pos, torch.float64), dev(mass, torch.float32))
        _, counts = plan.count_interactions(per_target=True)
        t = np.sort(rng.choice(n, 300, replace=False))
        ref = oracle_mod.accel(pos, mass.astype(np.float64), p, targets=t)
        assert np.array_equal(counts.cpu().numpy()[t], ref["n_inter"])


@pytest.mark.parametrize("ns", [(0, 700, 0, 0, 65, 1, 0), (0, 0, 3000), (2000, 0, 0), (0, 0)])
def test_batches_with_empty_boxes(pp, ns):
    """Empty boxes before, between and after the others: each other box gets
    the bits it gets alone."""
    boxes = []
    for b, n in enumerate(ns):
        rng = np.random.default_rng(50 + b)
        p = BoxParams.from_mesh(30.0 + b, 12)
        boxes.append((rng.random((3, n)) * p.L, rng.uniform(0.5, 1.5, n).astype(np.float32), p))
    bp = pp.BatchPlan([b[2] for b in boxes], list(ns))
    pos = np.concatenate([b[0] for b in boxes], 1)
    mass = np.concatenate([b[1] for b in boxes])
    acc = bp.accel(dev(pos, torch.float64), dev(mass, torch.float32)).cpu().numpy()
    off = 0
    for x, m, p in boxes:
        n = m.size
        if n:
            one = pp.Plan(p, n).accel(dev(x, torch.float64), dev(m, torch.float32)).cpu().numpy()
            assert np.array_equal(acc[:, off:off + n], one)
        off += n


def test_resized_plan_does_not_reuse_lists(pp):
    """A plan with a skin that is called with another particle count builds
    new lists for it, with the cut widened again."""
    rng = np.random.default_rng(4)
    p = BoxParams.from_mesh(40.0, 14)
    pos, mass = rng.random((3, 3000)) * p.L, W.equal_masses(3000)
    plan = pp.Plan(p, 3000)
    plan.set_skin(0.2 * p.rcut)
    for n in (3000, 2000, 3000, 2500):
        x, m = dev(pos[:, :n], torch.float64), dev(mass[:n], torch.float32)
        got = plan.accel(x, m).cpu().numpy()
        moved = dev(pos[:, :n] + 0.05 * p.rcut, torch.float64)
        again = plan.accel(moved, m).cpu().numpy()   # every particle by the same vector: the same forces
        ref = pp.Plan(p, n).accel(x, m).cpu().numpy()
        scale = np.abs(ref).max()
        assert np.allclose(got, ref, rtol=1e-5, atol=1e-5 * scale)
        assert np.allclose(again, ref, rtol=1e-3, atol=1e-4 * scale)


@pytest.mark.parametrize("n,leaf_max", [(700, 64), (3000, 1), (3000, 3), (6000, 16)])
def test_monopole_windows_match_tree_oracle(pp, n, leaf_max):
    """Blocks with a few and with hundreds of accepted leaves and groups, so
    that windows of 64 nodes start, end and split inside an entry; part of the
    nodes lies beyond the cut of its block."""
    from tests import monopole_mirror as tree
    rng = np.random.default_rng(n + leaf_max)
    p0 = BoxParams.from_mesh(30.0, 16)
    p = W.BoxParams(**{**p0.__dict__, "leaf_max": leaf_max})
    pos = W.mixture(rng, n, p.L, 0.5, 4)
    mass = rng.uniform(0.5, 1.5, n).astype(np.float32)
    ref = tree.monopole_accel(pos, mass.astype(np.float64), p, 0.6)
    plan = pp.Plan(p, n)
    plan.set_monopole(0.6)
    acc = plan.accel(dev(pos, torch.float64), dev(mass, torch.float32)).cpu().numpy()
    assert plan.stats()["monopoles"] == ref["n_mono_pairs"]
    mag = np.linalg.norm(ref["acc"], axis=0)
    e = np.linalg.norm(acc.astype(np.float64) - ref["acc"], axis=0) / np.maximum(mag, 1e-300)
    assert np.median(e) <= 1e-6 and np.percentile(e, 99.9) <= 1e-4, (np.median(e), np.percentile(e, 99.9))


# 4096 particles and fewer take the library's sort, up to 131072 two passes of
# own digits, more three; tiles of 1024, 2048 and 4096
@pytest.mark.parametrize("n,mesh,spread", [(4096, 16, None), (4097, 16, None), (30000, 32, 0.02), (131072, 50, None),
                                           (131073, 50, 0.3), (150000, 420, None), (1048577, 100, None)])
def test_leading_bits_sort_orders_like_the_full_sort(pp, n, mesh, spread):
    """A box alone (leading bits, then runs) against the same box beside a
    second one (the library's sort of all bits): the same particle order, so
    the same bits.  spread: half the particles in a cloud of that width, many
    to a cell of the leading bits, some at one point."""
    rng = np.random.default_rng(n)
    p = BoxParams.from_mesh(50.0, mesh)
    pos = rng.random((3, n)) * p.L
    if spread is not None:
        pos[:, ::2] = 20.0 + spread * rng.random((3, (n + 1) // 2))
        pos[:, 100:140] = pos[:, 100:101]
    mass = rng.uniform(0.5, 1.5, n).astype(np.float32)
    other = BoxParams.from_mesh(30.0, 12)
    x, m = dev(pos, torch.float64), dev(mass, torch.float32)
    one = pp.Plan(p, n).accel(x, m)
    bp = pp.BatchPlan([p, other], [n, 65])
    y = dev(rng.random((3, 65)) * other.L, torch.float64)
    two = bp.accel(torch.cat([x, y], 1), torch.cat([m, m[:65]]))
    assert torch.equal(one, two[:, :n])


# blocks up to and beyond those of one item workgroup (1024, with the capacity's
# margin of an eighth and 64), with and without active flags
@pytest.mark.parametrize("n", [1, 64, 54500, 54700, 56000])
def test_items_of_few_and_many_blocks(pp, oracle_mod, n):
    rng = np.random.default_rng(n)
    p = BoxParams.from_mesh(40.0, 30)
    pos = W.mixture(rng, n, p.L, 0.4, 1 + n // 500)
    mass = rng.uniform(0.5, 1.5, n).astype(np.float32)
    x, m = dev(pos, torch.float64), dev(mass, torch.float32)
    plan = pp.Plan(p, n)
    acc = plan.accel(x, m)
    st = plan.stats()
    t = np.sort(rng.choice(n, min(n, 200), replace=False))
    ref = oracle_mod.accel(pos, mass.astype(np.float64), p, targets=t)
    _, counts = plan.count_interactions(per_target=True)
    assert np.array_equal(counts.cpu().numpy()[t], ref["n_inter"])
    assert st["candidates"] >= st["evaluated"] > 0
    active = torch.as_tensor(rng.random(n) < 0.3).cuda()
    some = plan.accel_active(x, m, active.to(torch.uint8), torch.zeros_like(acc))
    assert torch.equal(some[:, active], acc[:, active])


def dense_cell(n, m, seed=2):
    """n particles of which m share one cell of the leading key bits (level 7
    up to 131072 particles, 11 beyond), with distinct keys, out of order."""
    rng = np.random.default_rng(seed)
    p = BoxParams.from_mesh(100.0, max(12, int(round(n ** (1 / 3)))))
    w = p.L / (128 if n <= 131072 else 2048)
    pos = rng.random((3, n)) * p.L
    pos[:, rng.permutation(n)[:m]] = 50.0 + w * (0.02 + 0.9 * rng.random((3, m)))
    return pos, rng.uniform(0.5, 1.5, n).astype(np.float32), p


# runs of up to 2048 particles are ordered in the gather, longer ones by a second
# pass with a sort of all bits; after one of more than 256 (1024 beyond 131072
# particles, 2048 beyond 2^20) the next call takes that
@pytest.mark.parametrize("n,m", [(30000, 255), (30000, 256), (30000, 257), (30000, 258), (30000, 2047), (30000, 2048),
                                 (30000, 2049), (30000, 2050), (30000, 9000), (140000, 1024), (140000, 1025),
                                 (140000, 2048), (140000, 2049), (140000, 20000)])
def test_dense_cells_order_like_the_full_sort(pp, n, m):
    """The first call (which meets the run), the ones after it and those after
    a change to other particles and back, by every entry point: the particle
    order, and so the bits, of the library's sort in a batch of two boxes."""
    pos, mass, p = dense_cell(n, m)
    spread = np.random.default_rng(3).random((3, n)) * p.L
    other = BoxParams.from_mesh(30.0, 12)
    y = dev(np.random.default_rng(1).random((3, 65)) * other.L, torch.float64)
    mm = dev(mass, torch.float32)
    bp = pp.BatchPlan([p, other], [n, 65])

    def full(x):
        return bp.accel(torch.cat([x, y], 1), torch.cat([mm, mm[:65]]))[:, :n].clone()

    x, z = dev(pos, torch.float64), dev(spread, torch.float64)
    want, want_z = full(x), full(z)
    plan = pp.Plan(p, n)
    for _ in range(3):
        assert torch.equal(plan.accel(x, mm), want)
    on = torch.as_tensor(np.random.default_rng(4).random(n) < 0.1).cuda()
    fresh = pp.Plan(p, n)
    got = fresh.accel_active(x, mm, on.to(torch.uint8), torch.zeros_like(want))
    assert torch.equal(got[:, on], want[:, on])
    for _ in range(2):
        assert torch.equal(plan.accel(z, mm), want_z)
    assert torch.equal(plan.accel(x, mm), want)
    if n <= 65536:
        for _ in range(2):
            assert torch.equal(pp.pp_accel_scratch(p, x, mm), want)
    m64 = mm.to(torch.float64)
    a, b = pp.Plan(p, n), pp.Plan(p, n)
    b.accel(x, mm)                                   # has met the run
    assert torch.equal(a.accel_f64(x, m64), b.accel_f64(x, m64))


def test_a_dense_cell_does_not_hold_up_few_targets(pp):
    """Half of 131072 particles in one cell of the leading key bits, 5 active
    targets elsewhere: the call takes about as long as on spread particles (1.0
    times with a sort by all bits, 30 times with the square of the cell's
    particles in the gather)."""
    n = 131072
    pos, mass, p = dense_cell(n, n // 2)
    pos[:, :5] = np.random.default_rng(6).random((3, 5)) * 20.0
    spread = np.random.default_rng(3).random((3, n)) * p.L
    on = torch.zeros(n, dtype=torch.uint8, device="cuda")
    on[:5] = 1
    out, mm = torch.zeros(3, n, device="cuda"), dev(mass, torch.float32)

    def best(x):
        plan = pp.Plan(p, n)
        t = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            plan.accel_active(x, mm, on, out)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    assert best(dev(pos, torch.float64)) < 6 * best(dev(spread, torch.float64))


@pytest.mark.parametrize("theta", [0.0, 0.95])
def test_many_blocks_with_short_cuts(pp, oracle_mod, theta, monkeypatch):
    """Clumps of 16 particles in cubes 4 cuts wide, far from one another: some
    hundred thousand blocks of a few targets each, whose first entries a lane
    per block finds.  Neighbour counts against the oracle, and with monopoles
    the forces of sampled blocks against the library's acceptance restated."""
    from tests import monopole_mirror as tree
    rng = np.random.default_rng(12)
    n, rcut = 320000, 1e-4
    p = W.BoxParams(L=1.0, rs=rcut / 4.5, rcut=rcut, eps=0.01 * rcut, leaf_max=1 if theta else 8)
    centre = np.repeat(rng.random((3, n // 16)), 16, axis=1)
    centre[:, :1600] = rng.random((3, 1600)) * 2e-3                  # part of them across the faces
    pos = centre + (rng.random((3, n)) - 0.5) * 4 * rcut
    mass = rng.uniform(0.5, 1.5, n).astype(np.float32)
    x, m = dev(pos, torch.float64), dev(mass, torch.float32)
    plan = pp.Plan(p, n)
    t = np.concatenate([np.arange(0, 1600, 20), np.sort(rng.choice(n, 200, replace=False))])
    if theta == 0:
        for _ in range(2):
            acc = plan.accel(x, m)
            _, counts = plan.count_interactions(per_target=True)
            ref = oracle_mod.accel(pos, mass.astype(np.float64), p, targets=t)
            assert np.array_equal(counts.cpu().numpy()[t], ref["n_inter"])
        assert plan.stats()["nblock"] > 65536
        return
    plan.set_monopole(theta)
    for _ in range(2):
        acc = plan.accel(x, m)
    st = plan.stats()
    assert st["nblock"] > 65536 and st["monopoles"] > 0
    keep = []
    blocks = tree._blocks

    def sample(q, n_, emax):
        all_ = blocks(q, n_, emax)
        assert len(all_) == st["nblock"]
        keep.extend(all_[k] for k in range(0, len(all_), len(all_) // 400))
        return keep

    monkeypatch.setattr(tree, "_blocks", sample)
    ref = tree.monopole_accel(pos, mass.astype(np.float64), p, theta)
    assert ref["n_mono_pairs"] > 0
    perm = plan.export_lists()["perm"]
    at = np.concatenate([perm[s:s + c] for s, c, _, _ in keep])
    got, want = acc.cpu().numpy()[:, at].astype(np.float64), ref["acc"][:, at]
    mag = np.linalg.norm(want, axis=0)
    e = np.linalg.norm(got - want, axis=0)[mag > 0] / mag[mag > 0]
    assert np.all(got[:, mag == 0] == 0)
    assert np.median(e) <= 1e-6 and np.percentile(e, 99) <= 1e-4, (np.median(e), np.percentile(e, 99))
