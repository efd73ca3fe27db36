"""The batched table force that leaves out the pairs beyond the cutoff
(k_batch_table_near, the built-in default) and its all-pairs counterpart
(k_table_rows): no pair inside the cutoff is missed, whatever the
coordinates' offset and the list's shape, and inputs for which a pair beyond
the cutoff does not add zero take the whole path."""
import numpy as np
import pytest

import oracle
from _helpers import norm_vec_err, rms, to_dev, to_host

pytestmark = pytest.mark.gpu

E, F = 4, 6
K = 1 << (E + F)
SMAX = np.float32(2.0 ** (1 << E) * (2 - 2.0 ** -F))


@pytest.fixture(scope="module")
def pgh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1203_4037_amd as p
    return p


@pytest.fixture()
def ctx(pgh):
    c = pgh.Context(0)
    yield c
    c.close()


def _scale(rcut):
    """The float32 c of s = c |d|^2 + 2: the smallest at which rcut reaches s_max."""
    r2 = np.float32(rcut) * np.float32(rcut)
    c = np.float32((float(SMAX) - 2) / float(np.float32(rcut)) ** 2)
    while np.float32(float(r2) * float(c) + 2.0) < SMAX:
        c = np.nextafter(c, np.float32(np.inf))
    return float(c)


def _counts(items, pi, pj, rcut):
    """For each i-row the list entries whose float32 s is below s_max."""
    c = _scale(rcut)
    out = np.zeros(pi.shape[1])
    for i0, ni, j0, nj in items:
        d = pj[:, None, j0:j0 + nj] - pi[:, i0:i0 + ni, None]
        q = (d[0] * d[0]).astype(np.float64)
        for k in (1, 2):  # fused multiply-adds: exact products, one rounding
            q = (d[k].astype(np.float64) ** 2 + q).astype(np.float32).astype(np.float64)
        out[i0:i0 + ni] = ((q * c + 2).astype(np.float32) < SMAX).sum(1)
    return out


def _lists(rng, centre, spread, clustered):
    """Groups of 1 to 200 and lists of 0 to 1300 entries around the groups,
    with gaps between the groups' rows."""
    sizes_i = [1, 2, 31, 32, 33, 63, 64, 65, 96, 200]
    sizes_j = [0, 1, 31, 63, 64, 65, 127, 255, 256, 257, 512, 1300]
    items, xi, xj, i0, j0 = [], [], [], 0, 0
    for a in sizes_i:
        for b in sizes_j:
            g = centre + spread * rng.random(3)
            w = 0.02 if clustered else 0.1
            xi.append(g[:, None] + w * (rng.random((3, a + 2)) - 0.5))
            xj.append(g[:, None] + 2 * w * (rng.random((3, b)) - 0.5))
            items.append((i0, a, j0, b))
            i0 += a + 2
            j0 += b
    return (np.array(items, np.int32), np.concatenate(xi, 1).astype(np.float32),
            np.concatenate(xj, 1).astype(np.float32))


def _count_table(pgh, ctx, rcut):
    """Force table of the S2 shape and a potential table that counts pairs:
    1 on every node but the last."""
    ctx.build_table(E, F, rcut, eps=rcut / 15)
    t = np.zeros(2 * K, np.float32)
    t[0:-2:2] = 1.0
    ctx._sync_stream()
    pgh.pgh_set_pot_table(ctx.h, to_dev(t)[0])


@pytest.mark.parametrize("waves", [0, 64, 4096])
@pytest.mark.parametrize("offset,rcut,clustered", [(0.0, 0.02, False), (0.0, 0.02, True),
                                                   (37.0, 0.02, False), (-4000.0, 0.05, False),
                                                   (0.5, 1e-4, True), (0.0, 0.08, False)])
def test_every_pair_inside_the_cutoff_is_found(pgh, ctx, offset, rcut, clustered, waves):
    """The neighbour counts, exact integers, of lists at the edges of the
    kernel's blocks, on plans cut for few and for many waves."""
    items, pi, pj = _lists(np.random.default_rng(3), np.full(3, offset), 0.3, clustered)
    _count_table(pgh, ctx, rcut)
    ctx.set_plan_waves(waves)
    plan = ctx.plan(items, pi.shape[1], pj.shape[1])
    one = np.ones(pj.shape[1], np.float32)
    phi = to_host(*plan.table(*to_dev(*pi), *to_dev(*pj), to_dev(one)[0], with_phi=True))[3]
    want = _counts(items, pi, pj, rcut)
    rows = np.concatenate([np.arange(i, i + n) for i, n, _, _ in items])
    assert want.max() >= 1
    assert np.array_equal(phi[rows], want[rows])


@pytest.mark.parametrize("n", [700, 5000])
@pytest.mark.parametrize("offset,rcut", [(0.0, 0.03), (12.0, 0.03), (0.0, 0.4)])
def test_all_pairs_counts(pgh, ctx, n, offset, rcut):
    rng = np.random.default_rng(n)
    p = (offset + 0.5 * rng.random((3, n))).astype(np.float32)
    _count_table(pgh, ctx, rcut)
    d = to_dev(*p)
    ctx.set_j(*d, to_dev(np.ones(n, np.float32))[0])
    phi = to_host(*ctx.table_force(*d, with_phi=True))[3]
    assert np.array_equal(phi, _counts([(0, n, 0, n)], p, p, rcut))


@pytest.mark.parametrize("what", ["last node", "nan i", "nan j", "inf j", "huge i", "inf mass",
                                  "nan mass", "none"])
@pytest.mark.parametrize("batched", [True, False])
def test_whole_path_where_zero_is_not_certain(pgh, ctx, what, batched):
    """Against the general kernels (variant 0): the same rows are NaN or
    infinite, the others agree to the rounding of sums of up to 1000 terms
    of at most m max|g d| each."""
    rng = np.random.default_rng(5)
    items = np.array([(0, 70, 0, 300), (70, 30, 300, 1000), (100, 64, 1300, 65)], np.int32)
    pi = rng.random((3, 164)).astype(np.float32)
    pj = rng.random((3, 1365)).astype(np.float32)
    m = np.full(1365, 1.0, np.float32)
    rcut = 0.2
    table = ctx.build_table(E, F, rcut, eps=rcut / 15)
    if what == "last node":
        table[-2] = 0.5
        ctx.set_table(E, F, rcut, to_dev(table)[0])
    elif what == "nan i":
        pi[1, [3, 120]] = np.nan
    elif what == "nan j":
        pj[2, [5, 700]] = np.nan
    elif what == "inf j":
        pj[0, 310] = np.inf
    elif what == "huge i":
        pi[0, 99] = 1e30
    elif what == "inf mass":
        m[[10, 1299]] = np.inf
    elif what == "nan mass":
        m[1364] = np.nan
    di, dj = to_dev(*pi), to_dev(*pj, m)
    fam = pgh.PGH_FAMILY_TABLE_BATCH if batched else pgh.PGH_FAMILY_TABLE_ALLPAIRS
    plan = ctx.plan(items, 164, 1365)
    got = []
    for v in (0, -1):
        ctx.set_variant(fam, v)
        if batched:
            got.append(np.stack(to_host(*plan.table(*di, *dj))))
        else:
            ctx.set_j(*dj)
            got.append(np.stack(to_host(*ctx.table_force(*di))))
    a, b = got
    assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b))
    if what in ("nan i", "nan j", "inf j", "inf mass", "nan mass"):
        assert np.isnan(a).any()
    s = np.array([2.0 ** (1 + (k >> F)) * (1 + (k & 63) / 64) for k in range(K)])
    r = rcut * np.sqrt((s - 2) / (float(SMAX) - 2))
    term = max(np.abs(table[0::2] * r).max(), 0.5 * np.sqrt(3))
    fine = np.isfinite(a)
    if what != "huge i" and fine.any():
        assert np.abs(a[fine] - b[fine]).max() <= 1000 * 1000 * 2.0 ** -24 * term


def test_default_against_the_oracle_with_many_pairs_inside(pgh, ctx):
    """Lists most of whose pairs are inside the cutoff: the blocks are
    evaluated whole."""
    items, pi, pj = _lists(np.random.default_rng(9), np.zeros(3), 0.3, True)
    rcut = 0.05
    table = ctx.build_table(E, F, rcut, eps=rcut / 15)
    m = np.random.default_rng(2).uniform(0.5, 1.5, pj.shape[1]).astype(np.float32)
    plan = ctx.plan(items, pi.shape[1], pj.shape[1])
    a = np.stack(to_host(*plan.table(*to_dev(*pi), *to_dev(*pj, m))))
    ref = oracle.lut_items(items, *pi, *pj, m, E, F, float(np.float32(rcut)), table)
    has = np.nan_to_num(ref[3]) > 0
    e = norm_vec_err(a[:, has], np.stack(ref[:3])[:, has], ref[3][has])
    assert rms(e) <= 1e-5 and e.max() <= 1e-3, (rms(e), e.max())


# sizes at the edges of the columns, the chunks and the waves' shares; both
# sides of the built-in choice, which for the last two is made on the device
@pytest.mark.parametrize("ni,nj,variant", [(1, 1, "near"), (31, 64, "near"), (33, 65, "near"),
                                           (64, 513, "near"), (129, 4097, "near"),
                                           (2001, 1025, "near"), (40000, 700, "near"),
                                           (1000, 90000, None), (2000, 60000, None),
                                           (8191, 13000, None), (8193, 13000, None),
                                           (40000, 4095, None), (20001, 20001, None)])
@pytest.mark.parametrize("rcut", [0.03, 0.4])
def test_all_pairs_counts_of_the_near_kernel(pgh, ctx, ni, nj, variant, rcut):
    """Counts of up to 300 spread rows; a whole second call into fresh outputs
    agrees, so the choice made on the device leaves no row unwritten."""
    rng = np.random.default_rng(ni + nj)
    pi = (0.5 * rng.random((3, ni))).astype(np.float32)
    pj = (0.5 * rng.random((3, nj))).astype(np.float32)
    _count_table(pgh, ctx, rcut)
    fam = pgh.PGH_FAMILY_TABLE_ALLPAIRS
    names = [pgh.pgh_variant_name(fam, v) for v in range(pgh.pgh_variant_count(fam))]
    ctx.set_variant(fam, -1 if variant is None else names.index(variant))
    di = to_dev(*pi)
    ctx.set_j(*to_dev(*pj, np.ones(nj, np.float32)))
    out = [np.stack(to_host(*ctx.table_force(*di, with_phi=True))) for _ in range(2)]
    rows = np.unique(np.linspace(0, ni - 1, 300).astype(int))
    items = [(int(i), 1, 0, nj) for i in rows]
    assert np.array_equal(out[0][3][rows], _counts(items, pi, pj, rcut)[rows])
    assert np.array_equal(*out) and np.isfinite(out[0]).all()


def test_near_choice_inside_a_graph(pgh, ctx):
    """The kernel for many pairs inside is chosen on the device: a captured call
    counts right as the particles, in place, move together and apart."""
    import torch
    n, rcut = 20001, 0.05
    rng = np.random.default_rng(8)
    base = rng.random((3, n)).astype(np.float32)
    _count_table(pgh, ctx, rcut)
    d = to_dev(*base)
    one = torch.ones(n, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ctx.set_j(*d, one)
        ctx.table_force(*d, with_phi=True)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.set_j(*d, one)
        out = ctx.table_force(*d, with_phi=True)
    rows = np.unique(np.linspace(0, n - 1, 60).astype(int))
    items = [(int(i), 1, 0, n) for i in rows]
    for k in range(5):
        p = base * np.float32(0.03 if k % 2 else 1.0)
        for v, w in zip(d, to_dev(*p)):
            v.copy_(w)
        g.replay()
        torch.cuda.synchronize()
        phi = out[3].cpu().numpy().copy()
        eager = ctx.table_force(*d, with_phi=True)[3].cpu().numpy()
        assert np.array_equal(phi[rows], _counts(items, p, p, rcut)[rows]), k
        assert np.array_equal(phi, eager), k


# shapes of tables whose least |d|^2 at the last node is not an ordinary number:
# one node only (s_max = 2), a cutoff whose square is no FP32 number, and ones
# whose squared inverse or whose distance to |d|^2 = 0 leaves the range
@pytest.mark.parametrize("e,f,rcut", [(0, 0, 0.5), (0, 0, 1e19), (E, F, 1e-20), (E, F, 3e-23),
                                      (E, F, 1e19), (E, F, 3e18), (1, 0, 0.5), (6, 0, 1e-12),
                                      (6, 4, 1e19)])
@pytest.mark.parametrize("path", ["batched", "moments", "near", "rows", "default"])
def test_tables_without_an_ordinary_cutoff(pgh, ctx, e, f, rcut, path):
    """A table that is nowhere zero, given by its entries: every kernel adds
    every pair, as the general ones (variant 0) do.  Differences to the
    rounding of sums of up to 1000 terms of at most m max|G| |d| each."""
    rng = np.random.default_rng(5)
    items = np.array([(0, 70, 0, 300), (70, 30, 300, 1000), (100, 64, 1300, 65)], np.int32)
    pi = rng.random((3, 164)).astype(np.float32)
    pj = rng.random((3, 1365)).astype(np.float32)
    m = np.full(1365, 1.0, np.float32)
    k = 1 << (e + f)
    t = np.zeros(2 * k, np.float32)
    t[0::2] = rng.uniform(0.5, 1.0, k)
    ctx.set_table(e, f, rcut, to_dev(t)[0])
    di, dj = to_dev(*pi), to_dev(*pj, m)
    plan = ctx.plan(items, 164, 1365)
    batched = path in ("batched", "moments")
    fam = pgh.PGH_FAMILY_TABLE_BATCH if batched else pgh.PGH_FAMILY_TABLE_ALLPAIRS
    names = [pgh.pgh_variant_name(fam, v) for v in range(pgh.pgh_variant_count(fam))]
    ctx.set_j(*dj)
    got = []
    for v in (0, names.index(path) if path in names and not batched else -1):
        ctx.set_variant(fam, v)
        if path == "moments" and v == -1:
            got.append(np.stack(to_host(*plan.table_moments(*di, *dj)[0])))
        elif batched:
            got.append(np.stack(to_host(*plan.table(*di, *dj))))
        else:
            got.append(np.stack(to_host(*ctx.table_force(*di))))
    a, b = got
    assert np.abs(a).max() > 1.0 and np.isfinite(a).all()
    assert np.abs(a - b).max() <= 1365 * 1000 * 2.0 ** -24 * np.sqrt(3)


@pytest.mark.parametrize("variant", ["near", "rows"])
@pytest.mark.parametrize("with_phi", [False, True])
@pytest.mark.parametrize("ni,nj", [(164, 1365), (33, 65), (5, 3)])
def test_last_node_not_finite_where_no_pair_reaches_it(pgh, ctx, variant, with_phi, ni, nj):
    """Lists that end between two steps, all pairs inside the cutoff: nothing
    of the last node's infinity and NaN reaches a result."""
    rng = np.random.default_rng(6)
    pi, pj = rng.random((3, ni)).astype(np.float32), rng.random((3, nj)).astype(np.float32)
    rcut = 4.0
    table = ctx.build_table(E, F, rcut, eps=rcut / 15)
    table[-2:] = np.inf, np.nan
    ctx.set_table(E, F, rcut, to_dev(table)[0])
    if with_phi:
        t = np.zeros(2 * K, np.float32)
        t[0::2] = 1.0
        t[-2] = np.nan
        ctx._sync_stream()
        pgh.pgh_set_pot_table(ctx.h, to_dev(t)[0])
    fam = pgh.PGH_FAMILY_TABLE_ALLPAIRS
    names = [pgh.pgh_variant_name(fam, v) for v in range(pgh.pgh_variant_count(fam))]
    ctx.set_variant(fam, names.index(variant))
    ctx.set_j(*to_dev(*pj, np.ones(nj, np.float32)))
    out = np.stack(to_host(*ctx.table_force(*to_dev(*pi), with_phi=with_phi)))
    assert np.isfinite(out).all()
    if with_phi:
        assert np.array_equal(out[3], np.full(ni, float(nj)))


def _sum_bound(terms):
    """Relative error of `terms` FP32 additions of one sign, each off by at
    most half an ulp of a partial sum no larger than the result."""
    return terms * 2.0 ** -24


@pytest.mark.parametrize("order", ["together", "in turn"])
@pytest.mark.parametrize("spread", [0.4, 0.75])
def test_near_sums_do_not_grow_with_the_list(pgh, ctx, order, spread):
    """10^6 + 3 neighbours of mass 0.7 (spread 0.4: blocks evaluated whole; 0.75:
    some beyond the cutoff, in candidates' rounds where they are the most), in a
    row or among as many far ones.  The potential counts them, so each of the terms is the
    same number and a running sum errs in one direction.  Fresh sums of at most
    543 terms, so at most 62500 / 512 of them, and 16 waves: less than the 512 +
    62500 / 256 + 16 additions allowed."""
    n = 1000003
    rng = np.random.default_rng(4)
    rcut = 0.5
    _count_table(pgh, ctx, rcut)
    pj = (spread * (rng.random((3, n)) - 0.5)).astype(np.float32)
    if order == "in turn":
        pj[:, ::2] += np.float32(20.0)
    pi = (0.02 * (rng.random((3, 64)) - 0.5)).astype(np.float32)
    fam = pgh.PGH_FAMILY_TABLE_ALLPAIRS
    names = [pgh.pgh_variant_name(fam, v) for v in range(pgh.pgh_variant_count(fam))]
    ctx.set_variant(fam, names.index("near"))
    mass = np.float32(0.7)
    ctx.set_j(*to_dev(*pj, np.full(n, mass)))
    phi = to_host(*ctx.table_force(*to_dev(*pi), with_phi=True))[3]
    want = _counts([(0, 64, 0, n)], pi, pj, rcut) * float(mass)
    assert want.min() > 5e4
    e = np.abs(phi - want) / want
    assert e.max() <= _sum_bound(512 + 62500 / 256 + 16), e.max()


@pytest.mark.parametrize("spread", [0.4, 0.75])
@pytest.mark.parametrize("ni", [1, 40])
@pytest.mark.parametrize("moments", [False, True])
def test_batched_sums_do_not_grow_with_the_list(pgh, ctx, spread, ni, moments):
    """2048 lists over one range of 400000 neighbours of mass 0.7, which a plan
    does not cut: as above, or S (the moments' first row, sum of m g) where the
    table itself counts.  A lane's sum of at most 1024 terms (of a segment of 2048
    entries), n / 2048 of them, then over two halves: less than the 512 + n / 256 + 2
    additions allowed."""
    n, lists = 400000, 2048
    rng = np.random.default_rng(4)
    rcut = 0.5
    _count_table(pgh, ctx, rcut)
    if moments:
        t = np.zeros(2 * K, np.float32)
        t[0:-2:2] = 1.0
        ctx.set_table(E, F, rcut, to_dev(t)[0])
    pj = (spread * (rng.random((3, n)) - 0.5)).astype(np.float32)
    pi = (0.02 * (rng.random((3, ni * lists)) - 0.5)).astype(np.float32)
    items = np.array([(ni * k, ni, 0, n) for k in range(lists)], np.int32)
    plan = ctx.plan(items, ni * lists, n)
    mass = np.float32(0.7)
    d = to_dev(*pi), to_dev(*pj, np.full(n, mass))
    if moments:
        got = to_host(plan.table_moments(*d[0], *d[1])[1])[0][:ni * lists]
    else:
        got = to_host(*plan.table(*d[0], *d[1], with_phi=True))[3]
    rows = np.unique(np.linspace(0, ni * lists - 1, 24).astype(int))
    want = _counts([(int(r), 1, 0, n) for r in rows], pi, pj, rcut)[rows] * float(mass)
    e = np.abs(got[rows] - want) / want
    assert e.max() <= _sum_bound(512 + n / 256 + 2), e.max()


def test_every_variant_is_the_kernel_its_name_says(pgh, ctx):
    """Tuning files hold variants by name: the paper's form with two i-particles
    per lane and two records per tile sums in one order, bit for bit, whatever
    the workgroup's width, and "near" is another kernel, the built-in choice here."""
    items, pi, pj = _lists(np.random.default_rng(9), np.zeros(3), 0.3, True)
    ctx.build_table(E, F, 0.05, eps=0.05 / 15)
    m = np.random.default_rng(2).uniform(0.5, 1.5, pj.shape[1]).astype(np.float32)
    fam = pgh.PGH_FAMILY_TABLE_BATCH
    names = [pgh.pgh_variant_name(fam, v) for v in range(pgh.pgh_variant_count(fam))]
    d = to_dev(*pi), to_dev(*pj, m)
    plan = ctx.plan(items, pi.shape[1], pj.shape[1])
    out = {}
    for v in ("ki=2 tw=2 wg=4", "ki=2 tw=2 wg=16", "near", None):
        ctx.set_variant(fam, -1 if v is None else names.index(v))
        zero = to_dev(*np.zeros((3, pi.shape[1])))
        out[v] = np.stack(to_host(*plan.table(*d[0], *d[1], out=zero)))
    assert np.array_equal(out["ki=2 tw=2 wg=4"], out["ki=2 tw=2 wg=16"])
    assert np.array_equal(out["near"], out[None])
    assert not np.array_equal(out["near"], out["ki=2 tw=2 wg=4"])


# both sides of the built-in choice (16 i-particles per chunk on average), one and two
# columns, and the numbers of pairs inside at which blocks are evaluated whole
@pytest.mark.parametrize("n_i", [1, 8, 15, 16, 17, 32, 33, 64, 80])
@pytest.mark.parametrize("rcut", [0.06, 0.35, 0.5, 4.0])
@pytest.mark.parametrize("waves", [0, 16])
def test_lists_of_one_size_count(pgh, ctx, n_i, rcut, waves):
    """The neighbour counts, exact integers, of lists of one group size, from the
    potential and from the moments of a table that counts."""
    rng = np.random.default_rng(n_i)
    sizes_j = [0, 1, 63, 64, 65, 130, 257, 900] * 4
    items, j0 = [], 0
    for k, b in enumerate(sizes_j):
        items.append((n_i * k, n_i, j0, b))
        j0 += b
    items = np.array(items, np.int32)
    ni = n_i * len(sizes_j)
    pi, pj = rng.random((3, ni)).astype(np.float32), rng.random((3, j0)).astype(np.float32)
    _count_table(pgh, ctx, rcut)
    ctx.set_plan_waves(waves)
    plan = ctx.plan(items, ni, j0)
    d = to_dev(*pi), to_dev(*pj, np.ones(j0, np.float32))
    want = _counts(items, pi, pj, rcut)
    assert np.array_equal(to_host(*plan.table(*d[0], *d[1], with_phi=True))[3], want)
    t = np.zeros(2 * K, np.float32)
    t[0:-2:2] = 1.0
    ctx.set_table(E, F, rcut, to_dev(t)[0])
    assert np.array_equal(to_host(plan.table_moments(*d[0], *d[1])[1])[0][:ni], want)


# about as many chunks as CUs, where the choice begins to be made on the device
@pytest.mark.parametrize("ni,nj", [(16384, 7000), (16385, 7000), (16385, 24500)])
@pytest.mark.parametrize("rcut", [0.03, 0.4])
def test_all_pairs_counts_where_the_device_begins_to_choose(pgh, ctx, ni, nj, rcut):
    test_all_pairs_counts_of_the_near_kernel(pgh, ctx, ni, nj, None, rcut)
