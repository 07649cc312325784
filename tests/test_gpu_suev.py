"""Secondary uncertainty over the event-ordered blocks against the stream of
the codes and the oracle.

Both paths make the same draws; the event-ordered one adds a trial's
occurrence losses in integers and rounds once.  Two sums of n of the same
values then differ by at most the stream's n roundings (2^-53 of the total
each), the one rounding, and what the integers leave out: 2^-95 of the power
of two above the largest loss the terms allow, per occurrence.  The oracle's
own logarithms and exponentials keep the 1e-9 of the stream's tests.  A layer
without a finite limit takes the stream, bit for bit, as does a YET whose mark
of the event-ordered blocks is cleared."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

OPEN = [0.0, np.inf, 0.0, np.inf]
TERMS = [[1e4, 5e6, 1e4, 5e8], OPEN, [2e4, np.inf, 0.0, 1e7]]


@pytest.fixture(scope="module")
def ara():
    import torch
    assert torch.cuda.is_available()
    import paper_1308_2572_amd as ara
    ara.library()
    return ara


def workload(name, n, mean, catalog, sizes, lists, terms, seed, elt_limit=5e6):
    g = np.random.default_rng(seed)
    lens = g.poisson(mean, size=n)
    lens[::13] = 0
    off = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    ids = g.integers(0, catalog, size=int(off[-1]), dtype=np.int32)
    elts = synth.lognormal_elts(seed, sizes, catalog, mu=11.0, sigma=1.5)
    elts.terms = np.array([[1.0, 1e3 * k, elt_limit] for k in range(len(sizes))])
    elt_off = np.zeros(len(lists) + 1, np.int32)
    np.cumsum([len(x) for x in lists], out=elt_off[1:])
    layers = synth.Layers(elt_off, np.concatenate([np.asarray(x, np.int32) for x in lists]).astype(np.int32),
                          np.asarray(terms, np.float64))
    return synth.Workload(name, synth.Yet(catalog, off, ids), elts, layers, 0.9)


def check(ara, w, seed, streamed=()):
    import torch
    print(f"[gpu-suev] {w.name}: {w.yet.n_trials} trials, {w.yet.nnz} occurrences, catalogue {w.yet.catalog}", flush=True)
    sys.stdout.flush()
    sg = synth.record_sigmas(seed, w.elts, zero_frac=0.2)
    tables = ara.EltTables.from_numpy(w.elts)
    sigma = ara.SigmaTables.from_numpy(tables, sg)
    layers = ara.Layers(w.layers.elt_off, w.layers.elt_ids)
    yet, stream = (ara.PreparedYet.from_numpy(w.yet, transposed=False, positions=True) for _ in range(2))
    stream.handle.reserved = 0
    et = torch.tensor(w.elts.terms, dtype=torch.float64, device="cuda")
    lt = torch.tensor(w.layers.terms, dtype=torch.float64, device="cuda")

    def run(y, t0=0, t1=None):
        return [x.cpu().numpy() for x in ara.ylt_forward_su(tables, sigma, y, layers, et, lt, seed, t0, t1, check=True)]

    y, s = run(yet)
    ys, ss = run(stream)
    n = int(np.diff(w.yet.offsets).max(initial=0))
    for j in range(w.layers.n_layers):
        a, z = w.layers.elt_off[j], w.layers.elt_off[j + 1]
        most = min(float(w.elts.terms[w.layers.elt_ids[a:z], 2].sum()), float(w.layers.terms[j][1]))
        if j in streamed:
            assert np.array_equal(s[j], ss[j]) and np.array_equal(y[j], ys[j])
        else:
            left_out = n * 2.0 ** (int(np.frexp(most)[1]) - 95)
            assert np.all(np.abs(s[j] - ss[j]) <= (2 * n + 1) * 2.0 ** -53 * ss[j] + left_out)
    ref = oracle.forward_su(oracle.build_tables(w.elts), oracle.build_sigma_tables(w.elts, sg), w.yet, w.layers, w.elts.terms,
                            w.layers.terms, seed, n_threads=8)
    assert np.all(np.abs(s - ref["s_pre"]) <= 1e-9 * ref["s_pre"])
    assert np.all(np.abs(y - ref["ylt"]) <= 1e-9 * np.maximum(np.abs(ref["ylt"]), ref["s_pre"]))
    N = w.yet.n_trials
    for t0, t1 in [(0, 1), (N // 3, N // 3 + 1), (N // 2, N), (1, max(1, N - 1))]:
        if t0 < t1:
            yr, sr = run(yet, t0, t1)
            assert np.array_equal(sr, s[:, t0:t1]) and np.array_equal(yr, y[:, t0:t1])
    return s


@pytest.mark.parametrize("n", [1, 15, 8191, 8192, 8193, 17_000])
@pytest.mark.parametrize("mean,catalog", [(30, 40_000), (60, 6_000)])
def test_block_edges_and_header_forms(ara, n, mean, catalog):
    """One trial to three blocks of trials; short lists and long ones; events
    of one ELT and of three."""
    check(ara, workload("edges", n, mean, catalog, [catalog // 20, catalog // 9, catalog // 30], [[0, 1, 2], [2], [1, 0]],
                        TERMS, n + mean), n)


def test_lists_of_a_whole_wavefront(ara):
    """Events that occur thousands of times in one block of trials (lists
    queued by a whole wavefront) among short ones, in both header forms."""
    for catalog in (50_000, 700):
        w = workload("crowded", 6000, 40, catalog, [catalog // 10, catalog // 3], [[0, 1], [1]], TERMS[:2], catalog)
        g = np.random.default_rng(catalog)
        hot = w.elts.rec_ids[:3]
        u = g.random(w.yet.nnz)
        for k, p in enumerate((0.1, 0.02, 0.0004)):
            w.yet.ids[(u >= k * 0.2) & (u < k * 0.2 + p)] = hot[k]
        check(ara, w, catalog)


def test_layers_without_a_finite_limit(ara):
    """No limit on the ELTs: layers with an occurrence limit are added in
    integers, the others streamed; and a layer one of whose ELTs is scaled far
    below its limit is streamed."""
    w = workload("open", 9000, 30, 30_000, [3000, 2000], [[0], [1], [0, 1]], TERMS, 5, elt_limit=np.inf)
    check(ara, w, 5, streamed=(1, 2))
    w.elts.terms[0, 0] = 2.0 ** -40
    check(ara, w, 6, streamed=(0, 1, 2))


def test_layers_without_events(ara):
    """A layer with an empty ELT beside an ordinary one."""
    s = check(ara, workload("empty", 700, 30, 9_000, [0, 900], [[0], [0, 1], []], TERMS, 3), 3)
    assert np.all(s[0] == 0.0) and np.all(s[2] == 0.0)


@pytest.mark.parametrize("catalog", [(1 << 24) + 1, 1 << 26])
def test_largest_tiles_with_positions(ara, catalog):
    """Catalogues of more than 2^24 events, whose blocks are sorted by tiles of
    16,384 events, with positions: one tile of more records than are held in
    registers (19,456 with positions), the others nearly empty."""
    g = np.random.default_rng(catalog)
    lens = g.poisson(100, size=600)
    off = np.zeros(601, np.int64)
    np.cumsum(lens, out=off[1:])
    ids = g.integers(0, catalog, size=int(off[-1]), dtype=np.int64)
    u = g.random(ids.shape[0])
    ids[u < 0.4] = g.integers(3 << 14, 4 << 14, size=int((u < 0.4).sum()))
    ids[u > 0.98] = catalog - 1
    assert 19 * 1024 < ((ids >> 14) == 3).sum()
    ids = ids.astype(np.int32)
    seen = np.unique(ids)
    recs = [np.sort(g.choice(seen, size=k, replace=False)) for k in (9000, 4000)]
    rec_off = np.array([0, 9000, 13_000], np.int64)
    rec_ids = np.concatenate(recs).astype(np.int32)
    rec_loss = np.exp(g.normal(11.0, 1.5, size=13_000)).astype(np.float32)
    elts = synth.Elts(catalog, rec_off, rec_ids, rec_loss, np.array([[1.0, 1e3, 5e6], [1.5, 1e4, 2e6]]))
    layers = synth.Layers(np.array([0, 2, 3], np.int32), np.array([0, 1, 1], np.int32), np.asarray([TERMS[0], OPEN]))
    check(ara, synth.Workload("largest tiles", synth.Yet(catalog, off, ids), elts, layers, 0.9), 11)


@pytest.mark.parametrize("kind", ["wide", "narrow", "limit"])
def test_small_totals_keep_their_bits(ara, kind):
    """Years of an occurrence or two whose losses lie far below the limits:
    coefficients of variation of a hundred (draws 2^-40 below their mean and
    less) under a limit 2^23 above the mean, of one under a limit 2^21 above,
    and an ELT whose limit is 2^-60 of another's.  The totals of both paths
    differ by their own roundings alone, relative to the total itself."""
    import torch
    w = workload(kind, 20_000, 1, 4_000, [1500, 1500], [[0], [0, 1], [1]], [OPEN] * 3, 21)
    w.elts.rec_loss[:] = np.exp(np.random.default_rng(3).normal(11.0, 0.1, 3000)).astype(np.float32)
    most = 2.0 ** {"wide": 23, "narrow": 21, "limit": 10}[kind] * 6e4
    w.elts.terms = np.array([[1.0, 0.0, most], [1.0, 0.0, most * 2.0 ** -60 / 3 if kind == "limit" else most]])
    sg = (w.elts.rec_loss * {"wide": 100.0, "narrow": 1.0, "limit": 0.5}[kind]).astype(np.float32)
    print(f"[gpu-suev] small totals, {kind}", flush=True)
    tables = ara.EltTables.from_numpy(w.elts)
    sigma = ara.SigmaTables.from_numpy(tables, sg)
    layers = ara.Layers(w.layers.elt_off, w.layers.elt_ids)
    yet, stream = (ara.PreparedYet.from_numpy(w.yet, transposed=False, positions=True) for _ in range(2))
    stream.handle.reserved = 0
    et = torch.tensor(w.elts.terms, dtype=torch.float64, device="cuda")
    lt = torch.tensor(w.layers.terms, dtype=torch.float64, device="cuda")
    s, ss = (ara.ylt_forward_su(tables, sigma, y, layers, et, lt, 77, check=True)[1].cpu().numpy() for y in (yet, stream))
    n = int(np.diff(w.yet.offsets).max())
    assert ss[ss > 0].min() < 2.0 ** -15 * np.median(ss[ss > 0]) or kind == "narrow"
    assert np.all(np.abs(s - ss) <= (2 * n + 1) * 2.0 ** -53 * ss)
