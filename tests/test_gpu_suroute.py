"""Which way secondary uncertainty takes over a YET that has event-ordered blocks.

Small catalogues with few occurrences, frequent events, dense layers and many
short years take the stream of the codes: bit for bit, and in its time.  The
tests of the blocks' kernel are small in just these ways, so they are run here
with the mark that sends every layer through the blocks."""
import numpy as np
import pytest

import synth
import test_gpu_suev as T
from test_gpu_evfwd import best_of
from test_gpu_suev import TERMS, ara, check, workload  # noqa: F401 (ara: fixture)

pytestmark = pytest.mark.gpu

ALWAYS = 0x800   # of ara_yet.reserved: every layer takes the blocks


@pytest.fixture
def forced(ara, monkeypatch):
    prepare = ara.PreparedYet.from_numpy

    def marked(*args, **kw):
        yet = prepare(*args, **kw)
        yet.handle.reserved |= ALWAYS
        return yet

    monkeypatch.setattr(ara.PreparedYet, "from_numpy", staticmethod(marked))


@pytest.mark.parametrize("n", [1, 15, 8127, 8128, 8129, 17_000])
@pytest.mark.parametrize("mean,catalog", [(30, 40_000), (60, 6_000)])
def test_block_edges_and_header_forms(ara, forced, n, mean, catalog):
    T.test_block_edges_and_header_forms(ara, n, mean, catalog)


def test_lists_of_a_whole_wavefront(ara, forced):
    T.test_lists_of_a_whole_wavefront(ara)


def test_layers_without_a_finite_limit(ara, forced):
    T.test_layers_without_a_finite_limit(ara)


def test_layers_without_events(ara, forced):
    T.test_layers_without_events(ara)


def both(ara, n, mean, catalog, sizes, lists, power=1.0, seed=3):
    """A call, its results over the blocks as the rule has it and over the stream."""
    import torch
    w = workload("route", n, mean, catalog, sizes, lists, [[1e4, 5e6, 1e4, 5e8]] * len(lists), seed)
    if power != 1.0:
        g = np.random.default_rng(seed)
        w.yet.ids[:] = np.minimum(catalog * g.random(w.yet.nnz) ** power, catalog - 1).astype(np.int32)
    tables = ara.EltTables.from_numpy(w.elts)
    sigma = ara.SigmaTables.from_numpy(tables, synth.record_sigmas(seed, w.elts, zero_frac=0.2))
    layers = ara.Layers(w.layers.elt_off, w.layers.elt_ids)
    yet = ara.PreparedYet.from_numpy(w.yet, transposed=False, positions=True)
    et = torch.tensor(w.elts.terms, dtype=torch.float64, device="cuda")
    lt = torch.tensor(w.layers.terms, dtype=torch.float64, device="cuda")
    kept = yet.handle.reserved

    def run(rule):
        yet.handle.reserved = kept if rule else 0
        return ara.ylt_forward_su(tables, sigma, yet, layers, et, lt, seed)

    return run, [[x.cpu().numpy() for x in run(rule)] for rule in (True, False)]


TEN = [list(range(10))]


@pytest.mark.parametrize("name,n,mean,catalog,records,power", [
    ("few_events", 10_000, 1000, 1000, 50, 1.0),
    ("small_catalogue", 10_000, 1000, 20_000, 300, 1.0),
    ("frequent", 20_000, 500, 500_000, 8000, 2.0),
    ("dense", 50_000, 300, 450_000, 45_000, 1.0),
    ("short_years", 1_500_000, 10, 400_000, 6000, 1.0),
])
def test_streamed(ara, name, n, mean, catalog, records, power):
    """As before the blocks: the stream's own results, in its time."""
    run, ((y, s), (ys, ss)) = both(ara, n, mean, catalog, [records] * 10, TEN, power)
    assert np.array_equal(s, ss) and np.array_equal(y, ys)
    rule, stream = best_of(lambda: run(True)), best_of(lambda: run(False))
    print(f"[gpu-suroute] {name}: {1e6 * rule:.0f} us, over the stream {1e6 * stream:.0f} us", flush=True)
    assert rule <= 1.15 * stream


def test_dense_layer_beside_a_sparse_one(ara):
    """The dense layer is streamed, the sparse one is not; each as alone."""
    sizes, C = [3000] * 4 + [80_000] * 3, 500_000
    lists = [[0, 1, 2, 3], [4, 5, 6]]
    _, ((_, s), (_, ss)) = both(ara, 20_000, 300, C, sizes, lists)
    assert np.array_equal(s[1], ss[1]) and not np.array_equal(s[0], ss[0])
    for j, x in enumerate(lists):
        _, ((_, one), _) = both(ara, 20_000, 300, C, sizes, [x])
        assert np.array_equal(one[0], s[j])
