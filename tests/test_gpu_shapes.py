"""GPU: the launch shapes and table sizes of the kernels at the edges of their
ranges, through the C ABI, against the CPU oracle (integer weights, so every
comparison that is not said to be otherwise is exact)."""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_2405_11658_amd import inputs as gen
from paper_2405_11658_amd import leiden as L

from .gpu_common import dev_batch, ob, og, say, to_np
from .test_gpu_async import _check_state, _graph_of

pytestmark = pytest.mark.gpu


def _stars(degrees, seed=1):
    """A hub of each of the given degrees among communities of 64 vertices:
    the hub is joined to the first vertices of a shared pool, every pool
    vertex to 6 others of its community, the first two hubs to each other."""
    rng = np.random.default_rng(seed)
    pool = max(degrees) + 64
    h = len(degrees)
    u, v = [], []
    for k, d in enumerate(degrees):
        mates = rng.permutation(pool)[:d]
        u.append(np.full(d, k))
        v.append(h + mates)
    p = np.arange(pool)
    for _ in range(6):
        u.append(h + p)
        v.append(h + np.minimum(p // 64 * 64 + rng.integers(0, 64, pool), pool - 1))
    g = gen.from_edges(h + pool, np.concatenate(u), np.concatenate(v))
    deg = np.diff(g.off)
    assert [int(x) for x in deg[:h]] == list(degrees)
    return g


@pytest.mark.parametrize("degrees", [
    (256, 257, 2048),            # wavefront and workgroup
    (257, 2048, 2049, 6144),     # and the large workgroup
    (300, 2049, 6144, 6145),     # a chunked hub, alone in its slice or not
    (6145, 6500, 7000, 400, 500, 2500) * 3,
])
@pytest.mark.parametrize("slices", [0, 1])
def test_hub_degree_classes(degrees, slices):
    """Vertices on either side of every degree class of the asynchronous hub
    slices (one slice, and the default 64): modularity, K, Sigma and 2m match
    the oracle's for the returned membership and the communities are connected.
    With the default slices the modularity of the static run is at most 5e-3
    below the oracle's (the single-run bound of the other asynchronous tests;
    hubs that all move at once end where they end)."""
    g = _stars(degrees)
    h = L.leiden_create(g.off, g.idx, g.w, L.leiden_default_params(hub_slices=slices))
    say("hub classes", degrees, "slices", slices)
    C, q, st = L.leiden_static(h)
    qo = _check_state(h, g, C, q)
    if slices == 0:
        ost, _ = oracle.static(og(g))
        assert qo - oracle.modularity(og(g), ost.C) >= -5e-3
    for mode, b in zip(("df", "nd", "ds"), gen.batch_stream(g, 200, 3, seed=3)):
        C, q, st, _ = L.leiden_update(h, dev_batch(b), mode)
        _check_state(h, _graph_of(h), C, q)


@pytest.mark.parametrize("labels", [3, 50, 5000])
@pytest.mark.parametrize("sizes", [
    (1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 4096, 4097),
    (300,) * 40 + (700,) * 30 + (1000,) * 10 + (5,) * 100,
])
def test_aggregate_segment_sizes(sizes, labels):
    """Communities whose entries fill one wavefront's registers up to, and
    one past, each size of the sorting network, with few and many equal
    neighbour communities: rows equal to a sort in torch, weights within the
    rounding of a float64 sum to float32 (2^-24 relative), and the same bits
    on a second call."""
    n, rows = 6000, len(sizes)
    rng = np.random.default_rng(5)
    cols = [np.sort(rng.permutation(n)[:z]) for z in sizes]
    off = np.zeros(n + 1, np.int64)
    off[1:rows + 1] = np.cumsum(sizes)
    off[rows + 1:] = off[rows]
    idx = np.concatenate(cols).astype(np.int32)
    w = (rng.random(len(idx)) + 0.1).astype(np.float32)
    k = max(labels, rows)
    C = rng.integers(0, k, n).astype(np.int32)
    C[:rows] = np.arange(rows)
    say("aggregate segments", len(sizes), "labels", labels)
    o, i, x = (to_np(t) for t in L.leiden_aggregate(off, idx, w, C, k))
    key = np.repeat(C[:rows].astype(np.int64), sizes) * k + C[idx]
    pair, inv = np.unique(key, return_inverse=True)
    total = np.bincount(inv, weights=w.astype(np.float64))
    assert np.array_equal(o, np.searchsorted(pair, np.arange(k + 1) * k))
    assert np.array_equal(i, pair % k)
    assert np.all(np.abs(x - total) <= 2.0 ** -24 * total * (1 + 1e-6))
    assert np.array_equal(x, to_np(L.leiden_aggregate(off, idx, w, C, k)[2]))


def test_stateless_calls_share_kept_memory():
    """Working memory kept between stateless calls: growing and shrinking
    sizes, several threads and streams, and what is kept stays under its
    bound."""
    graphs = []
    for k in (40, 3000, 200000, 900):
        n = 4 * k
        rng = np.random.default_rng(k)
        lab = rng.integers(0, k, n).astype(np.int32)
        g = gen.from_edges(n, rng.integers(0, n, 4 * n), rng.integers(0, n, 4 * n))
        t = [torch.from_numpy(np.asarray(x)).cuda() for x in (g.off, g.idx, g.w, lab)]
        want = [x.clone() for x in L.leiden_aggregate(*t, k)]
        graphs.append((t, k, want, L.leiden_modularity(*t)))
    torch.cuda.synchronize()
    bad = []

    def work(first):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for r in range(8):
                t, k, want, q = graphs[(first + r) % len(graphs)]
                got = L.leiden_aggregate(*t, k)
                s.synchronize()
                bad.extend(not torch.equal(x, y) for x, y in zip(got, want))
                bad.append(abs(L.leiden_modularity(*t) - q) > 1e-12)

    free = torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()
    ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert len(bad) == 4 * 8 * 4 and not any(bad)
    assert free - (torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()) < 2 << 30


@pytest.mark.parametrize("variant", [None, 0, 2])
def test_fleet_row_and_degree_classes(variant):
    """The fused engine's visits from registers (up to 64 and 256 edges) and by
    the workgroup, rows of 8 lanes and of a wavefront, levels and batches of
    few and of more than a tile, against the serial oracle."""
    gs = [_stars((63, 64, 65, 255, 256, 257), seed=3), _stars((300, 1030, 2100), seed=4),
          gen.from_edges(65, np.arange(64), np.arange(1, 65)), gen.from_edges(3, [0], [2])]
    fl = L.Fleet([(g.off, g.idx, g.w) for g in gs])
    if variant is not None:
        fl.set_variant(variant)
    res, _ = fl.run([(k, "static", None) for k in range(len(gs))])
    states = []
    for k, g in enumerate(gs):
        ref, st = oracle.static(og(g))
        assert np.array_equal(to_np(res[k][0]), ref.C) and res[k][3]["move_iters"] == st["move_iters"], k
        states.append(ref)
    jobs, bs = [], {}
    for k, mode in ((0, "df"), (1, "ds"), (2, "nd")):
        bs[k] = gen.random_batch(gs[k], 6, seed=k)
        jobs.append((k, mode, dev_batch(bs[k])))
    res, _ = fl.run(jobs)
    for q, (k, mode, _) in enumerate(jobs):
        new = oracle.update(states[k], ob(bs[k]), mode)[0]
        assert np.array_equal(to_np(res[q][0]), new.C), (k, mode)
        off, idx, w = fl.get_graph(k)
        assert np.array_equal(to_np(off), new.g.off) and np.array_equal(to_np(idx), new.g.idx)
        assert np.array_equal(to_np(w), new.g.w)
    fl.close()


def test_fleet_of_more_jobs_than_wide_workgroups():
    """1030 jobs in one run, and fewer in the next: either launch of the fused
    engine gives the serial oracle's result."""
    kinds = [gen.clique_ring(6, 5), gen.gnp(60, 0.1, seed=2, weights="unit"), gen.from_edges(2, [0], [1])]
    refs = [oracle.static(og(g))[0].C for g in kinds]
    fl = L.Fleet([(g.off, g.idx, g.w) for g in (kinds[k % 3] for k in range(1030))])
    for count in (1030, 1024, 5, 1025):
        res, _ = fl.run([(k, "static", None) for k in range(count)])
        assert all(np.array_equal(to_np(r[0]), refs[k % 3]) for k, r in enumerate(res)), count
    fl.close()


@pytest.mark.parametrize("nslices,n,mult", [(1, 6000, 24), (4, 6000, 24), (64, 6000, 24), (1, 40, 3), (2, 3100, 300)])
def test_sync_slice_launches(nslices, n, mult):
    """Synchronous slices whose buckets share a launch and slices with a
    launch for each (above 768 workgroups), with and without hubs, tiles of
    the frontier and their remainders: the oracle's synchronous mode."""
    rng = np.random.default_rng(n + mult)
    u, v = rng.integers(0, n, n * mult // 2), rng.integers(0, n, n * mult // 2)
    near = rng.integers(0, 40, n * mult // 2)
    g = gen.from_edges(n, np.concatenate([u, u]), np.concatenate([v, np.minimum(u // 40 * 40 + near, n - 1)]))
    g = gen.from_edges(n, np.repeat(np.arange(n), np.diff(g.off)).tolist() + [0] * (n // 2),
                       g.idx.tolist() + list(range(1, n // 2 + 1)))
    ref, st = oracle.static(og(g), oracle.make_params(sync=True, nslices=nslices))
    h = L.leiden_create(*(torch.from_numpy(np.asarray(x)).cuda() for x in (g.off, g.idx, g.w)),
                        L.leiden_default_params(sync_mode=1, nslices=nslices, hub_degree=512))
    C, q, stats = L.leiden_static(h)[:3]
    assert np.array_equal(to_np(C), ref.C)
    assert stats["move_iters"] == st["move_iters"]


@pytest.mark.parametrize("where", ["none", "first", "last", "one"])
def test_create_sorts_only_what_is_unsorted(where):
    """Rows given in order are left as they are; one row out of order (the
    first, the last, one in between of a chunk) sorts them; a repeated entry
    is refused either way."""
    g = gen.planted_partition(2048, 32, 0.1, 0.002, seed=2, permute=True)
    idx, w = g.idx.copy(), np.arange(1, g.idx.size + 1, dtype=np.float32)
    r = {"none": None, "first": 0, "last": g.n - 1, "one": 1000}[where]
    if r is not None:
        a, b = g.off[r], g.off[r + 1]
        assert b - a > 2
        idx[a:b], w[a:b] = idx[a:b][::-1], w[a:b][::-1].copy()
    dev = lambda *xs: [torch.from_numpy(np.asarray(x)).cuda() for x in xs]
    off2, idx2, w2 = L.leiden_get_graph(L.leiden_create(*dev(g.off, idx, w)))
    assert np.array_equal(to_np(idx2), g.idx)
    assert np.array_equal(to_np(w2), np.arange(1, g.idx.size + 1, dtype=np.float32))
    bad = idx.copy()
    bad[g.off[7] + 1] = bad[g.off[7]]
    with pytest.raises(L.LeidenError):
        L.leiden_create(*dev(g.off, bad, w))


@pytest.mark.parametrize("n,batch", [(2, 1), (3, 1), (255, 20), (256, 20), (257, 20), (512, 40), (1024, 1023),
                                     (1024, 1024), (1025, 1025), (4096, 3000)])
@pytest.mark.parametrize("mode", ["df", "ds", "nd"])
def test_batch_sort_bits_and_tiles(n, batch, mode):
    """Batches sorted by the bits that the ids use (n at and beside powers of
    two, the last vertex and community among them) in one tile of 4096 entries
    and in several: marking and the new graph against the oracle."""
    rng = np.random.default_rng(n)
    k = 4 * n if n > 3 else 0
    g = gen.from_edges(n, np.concatenate([np.arange(n - 1), rng.integers(0, n, k)]),
                       np.concatenate([np.arange(1, n), rng.integers(0, n, k)]))
    b = gen.random_batch(g, batch, seed=n, ins_frac=0.8 if n > 3 else 0.0)
    dev = [torch.from_numpy(np.asarray(x)).cuda() for x in (g.off, g.idx, g.w)]
    h = L.leiden_create(*dev, L.leiden_default_params(sync_mode=1))
    # singleton communities: community n - 1 is in use
    C = np.arange(n, dtype=np.int32)
    L.leiden_set_state(h, torch.from_numpy(C).cuda())
    K = np.bincount(np.repeat(C, np.diff(g.off)), weights=g.w.astype(np.float64), minlength=n)
    gt, _ = oracle.apply_batch(og(g), ob(b))
    want = oracle.mark(mode, gt, ob(b), C, K, K, float(K.sum()))
    got = L.leiden_mark_affected(h, dev_batch(b), mode)
    for x, y in zip((got["affected"], got["in_range"], got["changed"]), want):
        assert np.array_equal(to_np(x), y[:n])
    # marking has left the graph; a batch that is no batch is refused in every mode
    assert np.array_equal(to_np(L.leiden_get_graph(h)[1]), g.idx)
    for u, v in ((0, n), (-1, 1), (n - 1, n - 1)):
        with pytest.raises(L.LeidenError):
            L.leiden_mark_affected(h, L.make_batch([], [], [u], [v], [1.0]), mode)
    res = L.leiden_update(h, dev_batch(b), mode)
    off, idx, w = L.leiden_get_graph(h)
    assert np.array_equal(to_np(off), gt.off) and np.array_equal(to_np(idx), gt.idx)
    assert np.array_equal(to_np(w), gt.w) and res[2]["affected"] == int(want[0].sum())


@pytest.mark.parametrize("n,nlab,mult", [(5, 5, 1), (700, 3, 40), (40000, 40000, 1), (300000, 200000, 4),
                                         (300000, 5, 4)])
def test_modularity_merge_table(n, nlab, mult):
    """Sums by community merged per workgroup: tables that never fill, that
    fill in every chunk, rows longer than a chunk; weights that are sums of
    powers of two, so Eq. 1 follows from exact sums (each of its terms rounded
    once or twice: 4 ulp of 1 a community, added pairwise)."""
    rng = np.random.default_rng(n + nlab)
    u, v = rng.integers(0, n, n * mult), rng.integers(0, n, n * mult)
    if n == 300000:
        u[:5000] = 7  # a row of several chunks
    g = gen.from_edges(n, np.append(u, 0), np.append(v, 1))
    lab = rng.integers(0, nlab, n).astype(np.int32)
    row = np.repeat(np.arange(n), np.diff(g.off))
    w = (1.0 + ((row + g.idx) % 4)).astype(np.float32)
    inside = float(w[lab[row] == lab[g.idx]].sum(dtype=np.float64))
    S = np.bincount(lab[row], weights=w.astype(np.float64), minlength=n)
    m2 = float(S.sum())
    want = inside / m2 - float(np.sum((S / m2) ** 2))
    got = L.leiden_modularity(*(torch.from_numpy(np.asarray(x)).cuda() for x in (g.off, g.idx, w, lab)))
    assert abs(got - want) <= 4 * np.finfo(np.float64).eps * (1 + np.log2(n))
