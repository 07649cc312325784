"""The event-ordered forward against the stream of the codes and the oracle.

The event-ordered forward adds each trial's occurrence losses exactly (in
integers) and rounds the sum once, so its total differs from the oracle's
sequential binary64 sum by at most that sum's own rounding: n additions of at
most 2^-53 of the total each, and the one rounding.  Where a layer's values do
not fit the integers it streams the block's codes in the order of the stream,
bit for bit.  A YET whose mark of the event-ordered blocks is cleared takes
the stream throughout."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu-evfwd] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ara():
    import torch
    assert torch.cuda.is_available()
    import paper_1308_2572_amd as ara
    ara.library()
    return ara


class Case:
    def __init__(self, ara, w):
        import torch
        self.ara, self.w = ara, w
        self.tables = ara.EltTables.from_numpy(w.elts)
        self.yet = ara.PreparedYet.from_numpy(w.yet, transposed=False)
        self.stream = ara.PreparedYet.from_numpy(w.yet, transposed=False)
        assert self.yet.handle.reserved != 0
        self.stream.handle.reserved = 0
        self.layers = ara.Layers(w.layers.elt_off, w.layers.elt_ids)
        self.et = torch.tensor(w.elts.terms, dtype=torch.float64, device="cuda")
        self.lt = torch.tensor(w.layers.terms, dtype=torch.float64, device="cuda")

    def run(self, yet, hits, t0=0, t1=None):
        out = self.ara.ylt_forward(self.tables, yet, self.layers, self.et, self.lt, t0, t1, want_hits=hits, check=True)
        return [None if x is None else x.cpu().numpy() for x in out]

    def oracle(self):
        return oracle.forward(oracle.build_tables(self.w.elts), self.w.yet, self.w.layers, self.w.elts.terms,
                              self.w.layers.terms, n_threads=8)


def check(ara, w, bitwise=False):
    """Both paths, with and without hit counts, against the oracle; the
    event-ordered results the same in every way of asking."""
    c = Case(ara, w)
    _say(f"{w.name}: {w.yet.n_trials} trials, {w.yet.nnz} occurrences, catalogue {w.yet.catalog}")
    ref = c.oracle()
    n = int(np.diff(w.yet.offsets).max(initial=0))
    y, s, _ = c.run(c.yet, False)
    yh, sh, h = c.run(c.yet, True)
    ys, ss, hs = c.run(c.stream, True)
    assert np.array_equal(h, ref["hits"]) and np.array_equal(hs, ref["hits"])
    assert np.array_equal(s, sh) and np.array_equal(y, yh)
    for got in (s, ss):
        fin = np.isfinite(ref["s_pre"])
        assert np.array_equal(got[~fin], ref["s_pre"][~fin])
        assert np.all(np.abs(got[fin] - ref["s_pre"][fin]) <= (2 * n + 1) * 2.0 ** -53 * ref["s_pre"][fin])
    if bitwise:
        assert np.array_equal(s, ss) and np.array_equal(y, ys)
    N = w.yet.n_trials
    for t0, t1 in [(0, 1), (N // 3, N // 3 + 1), (N // 2, N), (1, max(1, N - 1))]:
        if t0 < t1:
            yr, sr, hr = c.run(c.yet, True, t0, t1)
            assert np.array_equal(sr, s[:, t0:t1]) and np.array_equal(yr, y[:, t0:t1]) and np.array_equal(hr, h[:, t0:t1])
    return c, s


def workload(name, n, mean, catalog, sizes, lists, terms, seed, mu=11.0, sigma=1.5, elt_terms=None):
    g = np.random.default_rng(seed)
    lens = g.poisson(mean, size=n)
    lens[::13] = 0
    off = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    ids = g.integers(0, catalog, size=int(off[-1]), dtype=np.int32)
    elts = synth.lognormal_elts(seed, sizes, catalog, mu=mu, sigma=sigma)
    if elt_terms is not None:
        elts.terms = np.asarray(elt_terms, np.float64)
    elt_off = np.zeros(len(lists) + 1, np.int32)
    np.cumsum([len(x) for x in lists], out=elt_off[1:])
    layers = synth.Layers(elt_off, np.concatenate([np.asarray(x, np.int32) for x in lists]).astype(np.int32),
                          np.asarray(terms, np.float64))
    return synth.Workload(name, synth.Yet(catalog, off, ids), elts, layers, 0.9)


OPEN = [0.0, np.inf, 0.0, np.inf]
TERMS = [[1e4, 5e6, 1e4, 5e8], OPEN, [2e4, 1e6, 0.0, 1e7]]


@pytest.mark.parametrize("n", [1, 15, 8191, 8192, 8193, 17_000])
@pytest.mark.parametrize("mean,catalog", [(30, 40_000), (60, 6_000)])
def test_block_edges_and_header_forms(ara, n, mean, catalog):
    """One trial to three blocks of trials; short lists and long ones."""
    check(ara, workload("edges", n, mean, catalog, [catalog // 20, catalog // 9, catalog // 30], [[0, 1, 2], [2], [1, 0]],
                        TERMS, n + mean))


@pytest.mark.parametrize("share", [0.45, 0.55, 0.95])
def test_layers_around_half_the_catalogue(ara, share):
    """Layers whose ELTs hold just under and over half the events of a table
    (65,536 here), where the records change place, and nearly all of them."""
    C = 65_536
    check(ara, workload("dense", 3000, 40, C, [int(C * share), C // 100], [[0], [0, 1], [1]], TERMS, 7))


def test_lists_of_a_whole_wavefront(ara):
    """Events that occur thousands of times in one block of trials (lists that
    a wavefront adds together), lists of fifteen and more among short ones, in
    both header forms."""
    for catalog in (50_000, 700):
        w = workload("crowded", 6000, 40, catalog, [catalog // 10, catalog // 3], [[0, 1], [1]], TERMS[:2], catalog)
        g = np.random.default_rng(catalog)
        hot = w.elts.rec_ids[:3]
        u = g.random(w.yet.nnz)
        for k, p in enumerate((0.1, 0.02, 0.0004)):
            w.yet.ids[(u >= k * 0.2) & (u < k * 0.2 + p)] = hot[k]
        check(ara, w)


@pytest.mark.parametrize("kind", ["spread", "infinite", "subnormal"])
def test_values_beyond_the_integers(ara, kind):
    """Losses some 2^120 apart, totals that overflow to infinity, and
    subnormal values beside ordinary ones: these layers are streamed, bit for
    bit as the stream; the ordinary layer beside them is not."""
    n_rec = 3000
    terms = [[1.0, 0.0, np.inf]] * 2
    w = workload(kind, 9000, 30, 30_000, [n_rec, 2000], [[0], [1], [0, 1]], [OPEN, TERMS[0], OPEN], 5, elt_terms=terms)
    g = np.random.default_rng(6)
    if kind == "spread":
        w.elts.rec_loss[:n_rec] = np.exp2(g.uniform(-60, 60, n_rec)).astype(np.float32)
    elif kind == "infinite":
        w.elts.rec_loss[:n_rec] = np.float32(3e38)
        w.elts.terms[0, 0] = 1e300
    else:
        w.elts.rec_loss[:n_rec] = np.where(g.random(n_rec) < 0.5, np.float32(1e-40), np.float32(1e5))
        w.elts.terms[0, 0] = 2.0 ** -900
        w.elts.rec_loss[0] = 3e30
    c, s = check(ara, w)
    _, ss, _ = c.run(c.stream, False)
    assert np.array_equal(s[0], ss[0]) and np.array_equal(s[2], ss[2])


def test_scaled_to_the_subnormal_range(ara):
    """A layer whose values are all subnormal or near it fits the integers:
    exact sums, so a one-occurrence trial's total is its O."""
    w = workload("tiny", 2000, 1, 5_000, [1500], [[0]], [OPEN], 8, elt_terms=[[1.0, 0.0, np.inf]])
    w.elts.terms[0, 0] = 2.0 ** -1060
    check(ara, w)


def test_many_layers(ara):
    """More layers than a wavefront has lanes."""
    g = np.random.default_rng(1)
    lists = [g.choice(6, size=int(g.integers(0, 5)), replace=False) for _ in range(70)]
    check(ara, workload("layers", 500, 30, 9_000, [300, 900, 100, 700, 50, 2000], lists,
                        [TERMS[k % 3] for k in range(70)], 2))


@pytest.mark.parametrize("kind", ["uneven", "even", "few", "five"])
def test_layers_walking_a_block_together(ara, kind):
    """Four layers and more over 65 blocks of 6.3M occurrences, where a block's
    workgroups may be dealt to its layers: every row is, bit for bit, that of
    its layer alone (the sums are exact), with and without hit counts and over
    part of the trials."""
    import torch
    n, per, C = 530_000, 770, 1_000_000
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    print(f"[gpu-evfwd] {kind}: {n} x {per}", flush=True)
    off = torch.arange(n + 1, dtype=torch.int64, device="cuda") * per
    ids = torch.randint(0, C, (n * per,), generator=g, dtype=torch.int32, device="cuda")
    sizes = {"uneven": [3, 9, 14, 20], "even": [9, 9, 9, 9], "few": [1, 1, 2, 2], "five": [1, 4, 8, 16, 20]}[kind]
    rec = 12_000
    K = sum(sizes)
    ro = torch.arange(K + 1, dtype=torch.int64, device="cuda") * rec
    ri = torch.cat([torch.randperm(C, generator=g, device="cuda", dtype=torch.int32)[:rec] for _ in range(K)])
    rl = torch.exp(12.0 + 1.5 * torch.randn(K * rec, generator=g, device="cuda"))
    tables = ara.EltTables(ro, ri, rl, C)
    yet = ara.PreparedYet(off, ids, C, transposed=False)
    del ids
    eo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    et = torch.tensor([[1.0, 5e4, 5e6]] * K, dtype=torch.float64, device="cuda")
    lt = torch.tensor([[1e4 * 4 ** j, 1e8, 1e6, 1e9] for j in range(len(sizes))], dtype=torch.float64, device="cuda")
    layers = ara.Layers(eo, np.arange(K, dtype=np.int32))
    y, s, _ = ara.ylt_forward(tables, yet, layers, et, lt, check=True)
    yh, sh, h = ara.ylt_forward(tables, yet, layers, et, lt, want_hits=True, check=True)
    yr, sr, _ = ara.ylt_forward(tables, yet, layers, et, lt, 1234, n - 777, check=True)
    assert torch.equal(y, yh) and torch.equal(s, sh)
    assert torch.equal(yr, y[:, 1234:n - 777]) and torch.equal(sr, s[:, 1234:n - 777])
    for j, J in enumerate(sizes):
        one = ara.Layers(np.array([0, J], np.int32), np.arange(eo[j], eo[j + 1], dtype=np.int32))
        y1, s1, h1 = ara.ylt_forward(tables, yet, one, et, lt[j:j + 1].contiguous(), want_hits=True, check=True)
        assert torch.equal(y1[0], y[j]) and torch.equal(s1[0], s[j]) and torch.equal(h1[0], h[j]), j


def frequent(n, mean, catalog, freq, seed):
    """A workload whose YET has events of the given numbers of occurrences
    (all held by both ELTs) among ordinary ones."""
    w = workload("frequent", n, mean, catalog, [catalog // 8, catalog // 5], [[0, 1], [1]], TERMS[:2], seed)
    g = np.random.default_rng(seed)
    hot = np.intersect1d(w.elts.rec_ids[:catalog // 8], w.elts.rec_ids[catalog // 8:])[:len(freq)]
    assert len(hot) == len(freq) and sum(freq) < 0.7 * w.yet.nnz
    at = g.permutation(w.yet.nnz)[:sum(freq)]
    w.yet.ids[at] = np.repeat(hot, freq)
    return w


FREQUENCIES = [
    [47, 48, 49, 50, 127, 128, 129, 130, 1023, 1024, 1025, 2047, 2048, 2049, 2050, 16_383, 16_384, 16_385],
    [60] * 40 + [140] * 30,                   # more than a few lanes with lists of either length
    [1100] * 50,
    [2100] * 100,                             # more pieces than wait for the workgroup
    [100_000, 40_000, 3000, 3000],
]


@pytest.mark.parametrize("catalog", [40_000, 10_000])
@pytest.mark.parametrize("freq", FREQUENCIES)
def test_lists_of_frequent_events(ara, catalog, freq):
    """Lists around the lengths from which a wavefront, or the workgroup, adds
    them together, few and many to a unit, in both header forms."""
    check(ara, frequent(7000, 60, catalog, freq, 7 + catalog))


def best_of(f, n=8):
    import torch
    import time
    f()
    t = []
    for _ in range(n):
        torch.cuda.synchronize()
        a = time.perf_counter()
        f()
        torch.cuda.synchronize()
        t.append(time.perf_counter() - a)
    return min(t)


@pytest.mark.parametrize("power", [3.0, 6.0])
def test_frequent_events_cost_no_more_than_the_stream(ara, power):
    """Event frequencies as a power of a uniform variable: the most frequent of
    500,000 events occur in every tenth occurrence and less.  The event-ordered
    forward took 1.4 to 3.6 times the stream's time when a wavefront added such
    an event's list alone, two bytes a lane at a time."""
    import torch
    n, per, C = 100_000, 1000, 500_000
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    off = torch.arange(n + 1, dtype=torch.int64, device="cuda") * per
    u = torch.rand(n * per, generator=g, device="cuda", dtype=torch.float64)
    ids = (u ** power * C).to(torch.int32).clamp_(0, C - 1)
    del u
    K, rec = 12, 10_000
    ri = torch.cat([torch.randperm(C, generator=g, device="cuda", dtype=torch.int32)[:rec] for _ in range(K)])
    ri[:64] = torch.arange(64, device="cuda", dtype=torch.int32)   # the most frequent among them
    first = ri[:rec]
    first[64:][first[64:] < 64] += 64
    ri[:rec] = torch.unique(torch.cat([first, torch.randperm(C, generator=g, device="cuda", dtype=torch.int32)]),
                            sorted=True)[:rec]
    rl = torch.exp(12.0 + 1.5 * torch.randn(K * rec, generator=g, device="cuda"))
    tables = ara.EltTables(torch.arange(K + 1, dtype=torch.int64, device="cuda") * rec, ri, rl, C)
    yets = [ara.PreparedYet(off, ids, C, transposed=False) for _ in range(2)]
    yets[1].handle.reserved = 0
    layers = ara.Layers(np.array([0, K], np.int32), np.arange(K, dtype=np.int32))
    et = torch.tensor([[1.0, 5e4, 5e6]] * K, dtype=torch.float64, device="cuda")
    lt = torch.tensor([[1e5, 1e8, 1e6, 1e10]], dtype=torch.float64, device="cuda")
    ev, stream = (best_of(lambda: ara.ylt_forward(tables, y, layers, et, lt)) for y in yets)
    _say(f"frequencies u^{power}: blocks {ev * 1e6:.0f} us, stream {stream * 1e6:.0f} us")
    assert ev < 1.2 * stream
