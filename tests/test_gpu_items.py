"""GPU tests of how a box's lists are cut into work items and how the items are
launched: the finer cut of small boxes, and the two launch forms behind
persistent = 1 (queues, or one workgroup per item)."""
import numpy as np
import pytest

import workloads as W
from workloads import BoxParams
from tests import parity

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


def box(n, seed=9):
    rng = np.random.default_rng(seed + n)
    p = BoxParams.from_mesh(60.0, max(12, int(round(n ** (1 / 3)))))
    return W.mixture(rng, n, p.L, 0.5, max(1, n // 500)), rng.uniform(0.5, 1.5, n).astype(np.float32), p


@pytest.mark.parametrize("n", [1, 64, 65, 700, 1500, 6001, 20011])
def test_small_boxes_are_cut_finer(pp, oracle_mod, n):
    """The default tuning cuts a box that lists T sources in all into chunks
    of 0.01075 T^(2/3) positions, rounded to 64, at least 128 (256 from 2^17
    on) and at most the requested 2048; the results meet the oracle bars."""
    pos, mass, p = box(n)
    plan = pp.Plan(p, n)
    acc = plan.accel(dev(pos, torch.float64), dev(mass, torch.float32)).cpu().numpy()
    slen = plan.export_lists()["slen"].astype(np.int64)
    T = int(slen.sum())
    few = int(0.01075 * np.cbrt(float(T)) ** 2 / 64 + 0.5) * 64
    chunk = min(2048, max(few, 128 if T < 2 ** 17 else 256))
    assert plan.stats()["nitem"] == int(np.maximum(1, -(-slen // chunk)).sum())
    ref = oracle_mod.accel(pos, mass.astype(np.float64), p, pair_abs=True)
    s = parity.summary(acc, ref)
    assert s["zero_ok"] and s["median"] <= 1e-6 and s["p999"] <= 1e-4, s
    assert s["robust_max"] <= parity.ROBUST_MAX, s


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("k", [1, 2, 8])
def test_queue_and_per_item_launches_agree(pp, k, graph):
    """64 positions per wave: the first call, with room for more than 65536
    waves of items and no mean length yet, runs from the queues; the later
    ones, whose last items were short, one workgroup per item.  All run every
    item once, in the same arithmetic, and count the same swept sources."""
    pos, mass, p = box(60000)
    x, m = dev(pos, torch.float64), dev(mass, torch.float32)
    plan = pp.Plan(p, pos.shape[1])
    plan.set_tuning(chunk=64 * k, waves_per_block=k, persistent=1, use_graph=graph)
    first = plan.accel(x, m).cpu().numpy()
    st = plan.stats()
    assert st["nitem"] * k * 1.25 > 65536
    for _ in range(2):
        later = plan.accel(x, m).cpu().numpy()
        assert np.array_equal(first.view(np.uint32), later.view(np.uint32))
        assert plan.stats()["lane_pairs"] == st["lane_pairs"]
        assert plan.stats()["evaluated"] == st["evaluated"]
    plan.set_tuning(persistent=0, use_graph=0)
    grid = plan.accel(x, m).cpu().numpy()
    assert np.array_equal(first.view(np.uint32), grid.view(np.uint32))

@pytest.mark.parametrize("k,variant,persistent", [(1, 0, 1), (1, 0, 0), (2, 0, 1), (4, 8, 1), (8, 0, 0)])
@pytest.mark.parametrize("equal", [False, True])
def test_few_active_targets_per_block(pp, k, variant, persistent, equal):
    """Blocks with 0, 1, 15, 16, 17, 31, 32, 33, 63 and 64 active targets (the
    edges between four, two and one copies of them per wave), their lists
    ending in tiles of every remainder: the active targets get the whole
    call's bits, the others keep what they held."""
    pos, mass, p = box(20011)
    n = pos.shape[1]
    if equal:
        mass[:] = 1.0 / n
    x, m = dev(pos, torch.float64), dev(mass, torch.float32)
    plan = pp.Plan(p, n)
    plan.set_tuning(chunk=704 * k, waves_per_block=k, persistent=persistent, variant=variant)
    full = plan.accel(x, m).cpu().numpy()
    lists = plan.export_lists()
    rng = np.random.default_rng(3)
    active = np.zeros(n, np.uint8)
    for b, (a, c) in enumerate(zip(lists["bstart"], lists["bcount"])):
        want = min(int(c), (0, 1, 15, 16, 17, 31, 32, 33, 63, 64)[b % 10])
        active[lists["perm"][a + rng.permutation(int(c))[:want]]] = 1
    out = torch.full((3, n), 7.0, dtype=torch.float32, device="cuda")
    plan.accel_active(x, m, dev(active, torch.uint8), out)
    got = out.cpu().numpy()
    on = active != 0
    assert np.array_equal(got[:, on].view(np.uint32), full[:, on].view(np.uint32))
    assert np.all(got[:, ~on] == 7.0)


@pytest.mark.parametrize("n,eps", [(1, None), (2, 0.0), (64, None), (65, 0.0), (129, None), (1500, 0.0), (6001, None)])
def test_f64_pair_arithmetic(pp, oracle_mod, n, eps):
    """FP64 sums whose lists end in every kind of remainder, with and without
    softening, coincident particles among them, positions on the faces and
    boxes small enough that most sources are periodic images.  Per target the
    error is bounded by the summation (n roundings) and 32 roundings per pair
    on both sides, relative to the sum of the pairs' magnitudes."""
    rng = np.random.default_rng(100 + n)
    p0 = BoxParams.from_mesh(30.0, 12 if n < 2000 else 18)
    p = W.BoxParams(**{**p0.__dict__, "eps": p0.eps if eps is None else eps})
    pos = W.mixture(rng, n, p.L, 0.5, max(1, n // 200)) if n > 2 else rng.random((3, n)) * 0.1
    if n > 64:
        pos[:, 1] = pos[:, 0]
        pos[0, 2:6] = 0.0
        pos[1, 4:8] = np.nextafter(p.L, 0.0)
    mass = rng.uniform(0.5, 1.5, n)
    acc = pp.Plan(p, n).accel_f64(dev(pos, torch.float64), dev(mass, torch.float64)).cpu().numpy()
    ref = oracle_mod.accel(pos, mass, p, pair_abs=True)
    tol = (64 + 2 * ref["n_inter"]) * 2.0 ** -53 * ref["pair_abs"]
    err = np.linalg.norm(acc - ref["acc"], axis=0)
    assert np.all(err <= tol), (float((err / np.maximum(tol, 1e-300)).max()), int(np.argmax(err - tol)))


# results leave as one 16-byte record per particle from 262144 particles on
@pytest.mark.parametrize("n", [262143, 262144, 262145])
def test_results_by_record_and_by_row(pp, oracle_mod, n):
    """Sampled targets against the oracle on both sides of the line, the columns
    of inactive particles left alone, and one plan serving both sizes."""
    rng = np.random.default_rng(n)
    p = BoxParams.from_mesh(60.0, 52)
    pos = W.mixture(rng, n, p.L, 0.3, 300)
    mass = rng.uniform(0.5, 1.5, n).astype(np.float32)
    x, m = dev(pos, torch.float64), dev(mass, torch.float32)
    plan = pp.Plan(p, n)
    acc = plan.accel(x, m)
    t = np.sort(rng.choice(n, 200, replace=False))
    ref = oracle_mod.accel(pos, mass.astype(np.float64), p, targets=t)["acc"]
    got = acc.cpu().numpy()[:, t].astype(np.float64)
    e = np.linalg.norm(got - ref, axis=0) / np.maximum(np.linalg.norm(ref, axis=0), 1e-300)
    assert np.median(e) <= 1e-6 and np.percentile(e, 99) <= 1e-4
    on = torch.as_tensor(rng.random(n) < 0.1).cuda()
    out = torch.full_like(acc, 7.0)
    plan.accel_active(x, m, on.to(torch.uint8), out)
    assert torch.equal(out[:, on], acc[:, on]) and bool((out[:, ~on] == 7.0).all())
    small = plan.accel(x[:, :9000].contiguous(), m[:9000].contiguous())
    assert torch.equal(small, pp.Plan(p, 9000).accel(x[:, :9000].contiguous(), m[:9000].contiguous()))
    assert torch.equal(plan.accel(x, m), acc)


@pytest.mark.parametrize("key_bits,rcut,rs", [(1, 1e-4, None), (1, 1e-5, None), (4, 1e-7, None), (10, 1e-7, None),
                                              (21, 1e-11, None), (21, 1e-3, None), (21, 0.05, 1e30)])
def test_f64_pairs_at_the_cut_in_wide_cells(pp, oracle_mod, key_bits, rcut, rs):
    """Pairs just inside the cut whose offsets from the block centre are up to
    4e4 times the cut (grid cells far wider than it), and a split scale whose
    square underflows FP32: no pair is dropped, in the sums or in the counts."""
    rng = np.random.default_rng(key_bits)
    n = 1000
    p = BoxParams(L=1.0, rs=rcut / 4.5 if rs is None else rs, rcut=rcut, eps=0.01 * rcut, key_bits=key_bits)
    a, d = rng.random((3, n)), rng.normal(size=(3, n))
    pos = np.concatenate([a, a + d / np.linalg.norm(d, axis=0) * rcut * (1 - 1e-4)], 1)
    mass = rng.uniform(0.5, 1.5, 2 * n)
    plan = pp.Plan(p, 2 * n)
    acc = plan.accel_f64(dev(pos, torch.float64), dev(mass, torch.float64)).cpu().numpy()
    _, counts = plan.count_interactions(per_target=True)
    ref = oracle_mod.accel(pos, mass, p, pair_abs=True)
    assert ref["n_inter"].min() >= 1
    assert np.array_equal(counts.cpu().numpy(), ref["n_inter"])
    tol = (64 + 2 * ref["n_inter"]) * 2.0 ** -53 * ref["pair_abs"]
    # the separations of positions of size 1 hold 2^-52 / rcut, equal on both sides but for the wrap's rounding
    tol = tol + 16 * 2.0 ** -52 / rcut * ref["pair_abs"]
    err = np.linalg.norm(acc - ref["acc"], axis=0)
    assert np.all(err <= tol), float((err / tol).max())


@pytest.mark.parametrize("nbox,n", [(3, 1000), (400, 1000), (2000, 700)])
def test_many_small_boxes_share_the_item_bound(pp, oracle_mod, nbox, n):
    """By the finer cut of small boxes a batch as a whole makes at most 65536
    items more than it has blocks; few boxes keep the cut, and the bits, they
    have alone."""
    rng = np.random.default_rng(nbox)
    p = BoxParams.from_mesh(50.0, 12)
    pos = rng.random((3, nbox * n)) * p.L
    mass = rng.uniform(0.5, 1.5, nbox * n).astype(np.float32)
    bp = pp.BatchPlan([p] * nbox, [n] * nbox)
    acc = bp.accel(dev(pos, torch.float64), dev(mass, torch.float32))
    st = bp.stats()
    assert st["nitem"] <= st["nblock"] + 65536
    for b in (0, nbox - 1):
        a = slice(b * n, b * n + n)
        one = pp.Plan(p, n)
        alone = one.accel(dev(pos[:, a], torch.float64), dev(mass[a], torch.float32))
        if nbox == 3:
            assert st["nitem"] > 2 * st["nblock"]
            assert torch.equal(acc[:, a], alone)
        ref = oracle_mod.accel(pos[:, a], mass[a].astype(np.float64), p)
        s = parity.summary(acc[:, a].cpu().numpy(), ref)
        assert s["zero_ok"] and s["median"] <= 1e-6 and s["p999"] <= 1e-4, s


@pytest.mark.parametrize("theta", [0.0, 0.5])
def test_statistics_after_a_rejected_call(pp, theta):
    """A call rejected for its input swept nothing, whatever the call before it
    counted; the next good call counts again."""
    pos, mass, p = box(6001)
    x, m = dev(pos, torch.float64), dev(mass, torch.float32)
    plan = pp.Plan(p, 6001)
    plan.set_monopole(theta)
    plan.accel(x, m)
    good = plan.stats()
    bad = x.clone()
    bad[1, 77] = float("nan")
    with pytest.raises(pp.PPError):
        plan.accel(bad, m)
    st = plan.stats()
    assert good["evaluated"] > 0
    assert (st["evaluated"], st["lane_pairs"], st["monopoles"]) == (0, 0, 0)
    plan.accel(x, m)
    st = plan.stats()
    assert [st[k] for k in ("evaluated", "lane_pairs", "monopoles")] == [good[k] for k in ("evaluated", "lane_pairs", "monopoles")]


@pytest.mark.parametrize("k", [1, 4])
def test_statistics_of_packed_blocks(pp, k):
    """With 1, 20, 40 and all targets of every block active, the evaluated
    pairs are those of the active targets where only they are swept (up to 32
    of a block), and the lane slots fall to a quarter or a half plus at most one
    partial sweep per wave and item."""
    pos, mass, p = box(20011)
    n = pos.shape[1]
    x, m = dev(pos, torch.float64), dev(mass, torch.float32)
    plan = pp.Plan(p, n)
    plan.set_tuning(chunk=1024 * k, waves_per_block=k)
    plan.accel(x, m)
    full, lists = plan.stats(), plan.export_lists()
    c = full["lane_pairs"] // 64                          # staged sources of all waves
    for want, copies in ((1, 4), (20, 2), (40, 1), (64, 1)):
        on = np.zeros(n, np.uint8)
        for a, cnt in zip(lists["bstart"], lists["bcount"]):
            on[lists["perm"][a:a + min(int(cnt), want)]] = 1
        plan.accel_active(x, m, dev(on, torch.uint8), torch.zeros(3, n, device="cuda"))
        st = plan.stats()
        assert st["nitem"] == full["nitem"]
        if want == 1:
            assert st["evaluated"] == c
        elif copies == 1:
            assert (st["evaluated"], st["lane_pairs"]) == (full["evaluated"], full["lane_pairs"])
        assert st["evaluated"] <= full["evaluated"]
        assert copies * st["lane_pairs"] >= full["lane_pairs"]
        if copies > 1 and lists["bcount"].min() > 20:
            assert st["lane_pairs"] <= full["lane_pairs"] // copies + 64 * 64 * k * st["nitem"]


def test_more_items_than_one_launch_takes(pp, oracle_mod):
    """7.2 M target blocks of one particle each (a cut below half a grid cell),
    their short items shared by 8 waves: one workgroup per item would be more
    than 2^32 threads, so the queues serve the later calls too."""
    n = 7200000
    p = BoxParams(L=1.0, rs=2e-7 / 4.5, rcut=2e-7, eps=1e-9)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    a = torch.rand(3, n // 2, dtype=torch.float64, device="cuda", generator=gen) * 0.99
    pos = torch.cat([a, a + 1e-7 * torch.rand(3, n // 2, dtype=torch.float64, device="cuda", generator=gen)], 1)
    mass = torch.full((n,), 1.0 / n, dtype=torch.float32, device="cuda")
    plan = pp.Plan(p, n)
    plan.set_tuning(chunk=4096, waves_per_block=8)
    first = plan.accel(pos, mass).clone()
    for _ in range(2):
        assert torch.equal(plan.accel(pos, mass), first)
    assert plan.stats()["nitem"] * 8 * 64 > 0.8 * 2 ** 32          # its capacity has a margin of a quarter
    t = np.arange(0, n, n // 20)
    ref = oracle_mod.accel(pos.cpu().numpy(), mass.cpu().numpy().astype(np.float64), p, targets=t)["acc"]
    e = np.linalg.norm(first.cpu().numpy()[:, t] - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert np.median(e) <= 1e-5 and e.max() <= 1e-2
