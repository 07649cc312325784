"""Which way the binary64 forward takes, and how the event-ordered one adds.

The preparation marks a YET whose forward takes the event-ordered blocks; small
catalogues with few occurrences, lists of thousands of entries and many short
years keep the stream of the codes.  The tests of the blocks' kernels are small
in just these ways, so they are run here with the mark set.

The blocks' integers come in two widths and give the exact sum of a trial's
occurrence losses, rounded once: math.fsum, bit for bit.  A layer that fits
neither is streamed, bit for bit as the stream."""
import math

import numpy as np
import pytest

import synth
import test_gpu_evfwd as T
from test_gpu_evfwd import OPEN, TERMS, ara, best_of, frequent, workload  # noqa: F401 (ara: fixture)

pytestmark = pytest.mark.gpu

FORWARD = 0x200   # of ara_yet.reserved: the forward takes the blocks


class Forced(T.Case):
    def __init__(self, ara, w):
        super().__init__(ara, w)
        self.yet.handle.reserved |= FORWARD


@pytest.fixture(autouse=True)
def forced(monkeypatch):
    monkeypatch.setattr(T, "Case", Forced)


@pytest.mark.parametrize("n", [1, 15, 8127, 8128, 8129, 17_000])
@pytest.mark.parametrize("mean,catalog", [(30, 40_000), (60, 6_000)])
def test_block_edges_and_header_forms(ara, n, mean, catalog):
    T.check(ara, workload("edges", n, mean, catalog, [catalog // 20, catalog // 9, catalog // 30], [[0, 1, 2], [2], [1, 0]],
                          TERMS, n + mean))


@pytest.mark.parametrize("share", [0.45, 0.55, 0.95])
def test_layers_around_half_the_catalogue(ara, share):
    T.test_layers_around_half_the_catalogue(ara, share)


def test_lists_of_a_whole_wavefront(ara):
    T.test_lists_of_a_whole_wavefront(ara)


@pytest.mark.parametrize("catalog", [40_000, 10_000])
@pytest.mark.parametrize("freq", T.FREQUENCIES)
def test_lists_of_frequent_events(ara, catalog, freq):
    T.test_lists_of_frequent_events(ara, catalog, freq)


@pytest.mark.parametrize("kind", ["spread", "infinite", "subnormal"])
def test_values_beyond_the_integers(ara, kind):
    T.test_values_beyond_the_integers(ara, kind)


def test_scaled_to_the_subnormal_range(ara):
    T.test_scaled_to_the_subnormal_range(ara)


def test_many_layers(ara):
    T.test_many_layers(ara)


@pytest.mark.parametrize("longest,b", [(1, 0), (1024, 10), (1025, 11), (4097, 13)])
@pytest.mark.parametrize("form", ["plain", "carry", "carry_all", "stream"])
def test_forms_at_their_bounds(ara, longest, b, form):
    """The lowest bit of a layer's values at the last place of either width and
    one below it, with the longest trial just at a power of two and beyond."""
    E = 20
    low = {"plain": E - 93 + 2 * b, "carry": E - 94 + 2 * b, "carry_all": E - 95 + b, "stream": E - 96 + b}[form]
    if form == "carry" and low < E - 95 + b:
        pytest.skip("no place between the widths")
    g = np.random.default_rng(100 * b + len(form))
    n, catalog, rec = 9000, 30_000, 3000
    w = workload(form, n, 0 if longest == 1 else 20, catalog, [rec], [[0]], [OPEN], b, elt_terms=[[1.0, 0.0, np.inf]])
    lens = np.minimum(np.diff(w.yet.offsets), longest) if longest > 1 else g.integers(0, 2, size=n)
    lens[n // 2] = longest
    off = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    ids = g.integers(0, catalog, size=int(off[-1]), dtype=np.int32)
    some = g.random(ids.shape[0]) < 0.8
    ids[some] = w.elts.rec_ids[g.integers(0, rec, size=int(some.sum()))]
    w.yet = synth.Yet(catalog, off, ids)
    # odd multiples of 2^low, of 24 bits, between there and 2^(E + 1); the first the largest there can be
    shift = np.where(g.random(rec) < 0.5, 0, g.integers(0, E - 23 - low + 1, size=rec))
    w.elts.rec_loss[:] = ((2 * g.integers(0, 1 << 23, size=rec) + 1).astype(np.float64) * np.exp2(low + shift)).astype(np.float32)
    w.elts.rec_loss[0] = np.float32((2.0 ** 24 - 1) * 2.0 ** (E - 23))
    w.elts.rec_loss[1] = np.float32(2.0 ** low)
    T._say(f"{form}: longest {longest}, lowest bit 2^{low}")
    c = Forced(ara, w)
    loss = np.zeros(catalog)
    loss[w.elts.rec_ids] = w.elts.rec_loss.astype(np.float64)
    v = loss[ids]
    exact = np.array([math.fsum(v[a:z]) for a, z in zip(off, off[1:])])
    _, s, _ = c.run(c.yet, False)
    _, sh, _ = c.run(c.yet, True)
    _, ss, _ = c.run(c.stream, False)
    assert np.array_equal(s, sh)
    assert np.array_equal(s[0], ss[0] if form == "stream" else exact)


def test_wide_values_beside_ordinary_ones(ara):
    """Layers of each form in one call, in blocks that several parts share."""
    w = workload("forms", 9000, 30, 30_000, [3000, 2000, 4000], [[0], [1], [2], [1, 2]], [OPEN, OPEN, OPEN, TERMS[0]], 12,
                 elt_terms=[[1.0, 0.0, np.inf]] * 3)
    g = np.random.default_rng(8)
    w.elts.rec_loss[:3000] = np.exp2(g.uniform(-60, 60, 3000)).astype(np.float32)
    w.elts.rec_loss[3000:5000] = np.exp2(g.uniform(-40, 10, 2000)).astype(np.float32)
    c, s = T.check(ara, w)
    _, ss, _ = c.run(c.stream, False)
    assert np.array_equal(s[0], ss[0])


@pytest.mark.parametrize("n,mean,catalog,blocks", [
    (2000, 1000, 200_000, True), (20_000, 100, 98_305, True),
    (2000, 1000, 98_304, False), (10, 5, 100, False), (20_000, 1000, 30_000, False),
    (1_240_000, 1, 200_000, False), (1_200_000, 1, 200_000, True), (1_240_000, 150, 200_000, True),
])
def test_way_of_a_yet(ara, n, mean, catalog, blocks):
    """The mark for small calls, few ranges, many short years; and an event in
    more than 10,000 places of a block on average."""
    import torch
    off = torch.arange(n + 1, dtype=torch.int64, device="cuda") * mean
    ids = torch.randint(0, catalog, (n * mean,), dtype=torch.int32, device="cuda")
    T._say(f"way: {n} x {mean} over {catalog}")
    assert bool(ara.PreparedYet(off, ids, catalog, transposed=False).handle.reserved & FORWARD) == blocks
    if blocks and n <= 20_000 and mean >= 100:
        k = 10_000 * -(-n // 8128)
        ids[ids == 7] = 8
        ids[:k] = 7
        assert ara.PreparedYet(off, ids, catalog, transposed=False).handle.reserved & FORWARD
        ids[k] = 7
        assert not ara.PreparedYet(off, ids, catalog, transposed=False).handle.reserved & FORWARD


@pytest.mark.parametrize("mean,blocks", [(7850, True), (7900, False)])
def test_way_of_a_small_crowded_catalogue(ara, mean, blocks):
    """8000 trials over 21,000 events: lists just under and over 3000 entries."""
    import torch
    off = torch.arange(8001, dtype=torch.int64, device="cuda") * mean
    ids = torch.randint(0, 21_000, (8000 * mean,), dtype=torch.int32, device="cuda")
    assert bool(ara.PreparedYet(off, ids, 21_000, transposed=False).handle.reserved & FORWARD) == blocks


@pytest.mark.parametrize("spread", [1.5, 9.0])
def test_ground_up_layers_cost_no_more_than_the_stream(ara, spread):
    """Four layers without retentions and limits, as a book has them (lognormal
    losses), and of values too far apart for the integers."""
    import torch
    n, C, sizes, rec = 150_000, 1_000_000, [8, 12, 16, 20], 9000
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    lens = torch.poisson(torch.full((n,), 1000.0, device="cuda"), generator=g).long()
    lens[n // 2] = 1100
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=off[1:])
    ids = torch.randint(0, C, (int(off[-1]),), generator=g, dtype=torch.int32, device="cuda")
    K = sum(sizes)
    ri = torch.cat([torch.randperm(C, generator=g, device="cuda", dtype=torch.int32)[:rec] for _ in range(K)])
    rl = torch.exp(12.0 + spread * torch.randn(K * rec, generator=g, device="cuda")).clamp_(1e-35, 1e35)
    tables = ara.EltTables(torch.arange(K + 1, dtype=torch.int64, device="cuda") * rec, ri, rl, C)
    yets = [ara.PreparedYet(off, ids, C, transposed=False) for _ in range(2)]
    yets[1].handle.reserved = 0
    eo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    layers = ara.Layers(eo, np.arange(K, dtype=np.int32))
    h = np.random.default_rng(1)
    et = torch.tensor(np.stack([h.uniform(0.97, 1.03, K), np.zeros(K), np.full(K, np.inf)], 1), device="cuda")
    lt = torch.tensor([OPEN] * 4, dtype=torch.float64, device="cuda")
    ev, stream = (best_of(lambda: ara.ylt_forward(tables, y, layers, et, lt)) for y in yets)
    T._say(f"ground-up, lognormal(12, {spread}): blocks {ev * 1e6:.0f} us, stream {stream * 1e6:.0f} us")
    y, ys = (ara.ylt_forward(tables, y, layers, et, lt)[0] for y in yets)
    assert float(((y - ys).abs() / ys.clamp(min=1e-300)).max()) < 1e-12
    assert ev < 1.1 * stream
