"""Which way the binary64 forward takes, and how the event-ordered one adds.

The preparation marks a YET whose forward takes the event-ordered blocks; small
catalogues with few occurrences, lists of thousands of entries and many short
years keep the stream of the codes.  The tests of the blocks' kernels are small
in just these ways, so they are run here with the mark set."""
import pytest

import test_gpu_evfwd as T
from test_gpu_evfwd import TERMS, ara, workload  # noqa: F401 (ara: fixture)

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
