"""The event-major copy of the YET that the backward reads (an index
transposition: exact).  For every trial slice x and event e the list of
slice-local trial indices must hold exactly the occurrences of e in the
slice's trials, with multiplicity; the list offsets are the running counts.
Checked against a numpy construction from the raw trials.
"""
import sys

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu-prepare] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ara():
    import torch
    assert torch.cuda.is_available()
    import paper_1308_2572_amd as ara
    ara.library()
    return ara


def read_dev(yet, ptr, count, dtype):
    import torch
    itemsize = torch.tensor([], dtype=dtype).element_size()
    off = ptr - yet.buf.data_ptr()
    assert 0 <= off and off + count * itemsize <= yet.buf.numel()
    return yet.buf[off: off + count * itemsize].view(dtype).cpu().numpy()


def expected(yet_np, slice_trials, n_slices):
    n = yet_np.n_trials
    lens = np.diff(yet_np.offsets)
    t = np.repeat(np.arange(n, dtype=np.int64), lens)
    x = t // slice_trials
    key = x * yet_np.catalog + yet_np.ids.astype(np.int64)
    local = t - x * slice_trials
    counts = np.bincount(key, minlength=n_slices * yet_np.catalog)
    off = np.zeros(n_slices * yet_np.catalog + 1, np.int64)
    np.cumsum(counts, out=off[1:])
    order = np.lexsort((local, key))
    return off, key[order], local[order]


def check_codes(py, yet_np):
    """Decode every segment of the 16-bit code stream on the host and compare
    it with the raw trials: same (trial, offset) sequence, in trial order and
    storage order inside a trial; with positions, each occurrence's position
    in its trial beside its code and 0xFFFF beside the other codes."""
    import torch
    h = py.handle
    G, groups, tg, tb = h.n_ranges, h.groups, h.trials_per_group, h.trials_per_block
    nseg = h.n_blocks * G * groups
    codes = read_dev(py, h.code, max(h.n_codes, 1), torch.int16).view(np.uint16).astype(np.int64)
    base = read_dev(py, h.seg_base, max(nseg, 1), torch.int64)
    run = read_dev(py, h.seg_run, max(nseg, 1), torch.int32).astype(np.int64)
    start = read_dev(py, h.lane_start, max(nseg * 64, 1), torch.uint8).astype(np.int64)
    n = yet_np.n_trials
    t = np.repeat(np.arange(n, dtype=np.int64), np.diff(yet_np.offsets))
    ids = yet_np.ids.astype(np.int64)
    key = ((t // tb) * G + (ids >> 15)) * groups + (t % tb) // tg
    order = np.argsort(key, kind="stable")
    key_s, trial_s, local_s = key[order], (t % tb % tg)[order], (ids & 0x7FFF)[order]
    pos_s = (np.arange(yet_np.nnz, dtype=np.int64) - yet_np.offsets[t])[order]
    pos = read_dev(py, h.pos, max(h.n_codes, 1), torch.int16).view(np.uint16).astype(np.int64) if h.pos else None
    bounds = np.searchsorted(key_s, np.arange(nseg + 1))
    lanes = np.arange(64)
    for si in range(nseg):
        R = int(run[si])
        a, b = bounds[si], bounds[si + 1]
        if R == 0:
            assert a == b, f"segment {si}: events but no codes"
            continue
        assert R % 4 == 0
        s = np.arange(R)
        slot = base[si] + (s[None, :] // 4) * 256 + 4 * lanes[:, None] + s[None, :] % 4   # [64, R]
        c = codes[slot]
        tr = start[si * 64: si * 64 + 64][:, None] + np.cumsum(c >> 15, axis=1)
        valid = c != 0xFFFF
        got_t, got_l = tr[valid], (c & 0x7FFF)[valid]      # row-major: lane by lane, in order
        assert np.array_equal(got_t, trial_s[a:b]), f"segment {si}: trials differ"
        assert np.array_equal(got_l, local_s[a:b]), f"segment {si}: offsets differ"
        if pos is not None:
            p = pos[slot]
            assert np.array_equal(p[valid], pos_s[a:b]), f"segment {si}: positions differ"
            assert np.all(p[~valid] == 0xFFFF), f"segment {si}: a gap or padding code has a position"
    assert h.n_codes >= yet_np.nnz


def check(ara, yet_np):
    import torch
    _say(f"trials {yet_np.n_trials} nnz {yet_np.nnz} catalog {yet_np.catalog}")
    py = ara.PreparedYet.from_numpy(yet_np, "cuda", positions=True)
    h = py.handle
    torch.cuda.synchronize()
    check_codes(py, yet_np)
    assert h.n_slices == 8
    assert h.slice_trials % h.trials_per_block == 0 and h.slice_trials * h.n_slices >= yet_np.n_trials
    off_ref, key_ref, loc_ref = expected(yet_np, h.slice_trials, h.n_slices)
    off = read_dev(py, h.tr_off, h.n_slices * yet_np.catalog + 1, torch.int64)
    assert np.array_equal(off, off_ref)
    # the trial-major copy and every event's occurrence count
    assert np.array_equal(read_dev(py, h.t_off, yet_np.n_trials + 1, torch.int64), yet_np.offsets)
    cnt = read_dev(py, h.t_cnt, yet_np.catalog, torch.int32)
    assert np.array_equal(cnt, np.bincount(yet_np.ids, minlength=yet_np.catalog))
    assert h.max_occ == (cnt.max() if yet_np.nnz else 0)
    if yet_np.nnz == 0:
        return
    assert np.array_equal(read_dev(py, h.t_ids, yet_np.nnz, torch.int32), yet_np.ids)
    ent = read_dev(py, h.tr_ent, yet_np.nnz, torch.int32).astype(np.int64)
    key = np.repeat(np.arange(h.n_slices * yet_np.catalog, dtype=np.int64), np.diff(off))
    order = np.lexsort((ent, key))
    assert np.array_equal(key[order], key_ref)
    assert np.array_equal(ent[order], loc_ref)


@pytest.mark.parametrize("seed", range(4))
def test_tiny_random(ara, seed):
    w = synth.tiny_random(seed)
    check(ara, w.yet)


def test_many_ranges_ragged_and_empty_trials(ara):
    g = np.random.default_rng(11)
    lens = g.integers(0, 300, size=5000)
    lens[::7] = 0
    off = np.zeros(5001, np.int64)
    np.cumsum(lens, out=off[1:])
    ids = g.integers(0, 300_000, size=int(off[-1]), dtype=np.int32)
    ids[:40] = 299_999                     # last event of a ragged last range
    ids[40:90] = 7                         # one event many times in one trial
    check(ara, synth.Yet(300_000, off, ids))


def test_fewer_blocks_than_slices(ara):
    g = np.random.default_rng(3)
    off = np.array([0, 3, 3, 10], np.int64)
    ids = g.integers(0, 70_000, size=10, dtype=np.int32)
    check(ara, synth.Yet(70_000, off, ids))


def test_no_trials_and_no_occurrences(ara):
    check(ara, synth.Yet(1000, np.zeros(1, np.int64), np.zeros(0, np.int32)))
    check(ara, synth.Yet(1000, np.zeros(50, np.int64), np.zeros(0, np.int32)))


def test_config0_layout(ara):
    check(ara, synth.config(0, n_trials=20_000).yet)


def test_gap_and_edge_offset_codes(ara):
    """Trials with no event in a range between trials that have some (gap
    codes), events at offset 0x7FFF opening a trial (their advance cannot sit
    on the code), a trial of 300 events in one range (several 64-ID chunks)."""
    g = np.random.default_rng(17)
    trials = []
    for k in range(40_000):   # 10 trials per group, so gaps occur inside segments
        kind = k % 7
        if kind == 0:
            trials.append([])
        elif kind == 1:
            trials.append([32767, 32767 + 32768, 5])
        elif kind == 2:
            trials.append(list(g.integers(0, 100_000, size=300)))
        elif kind == 3:
            trials.append([32767] * 3 + [0])
        else:
            trials.append(list(g.integers(0, 100_000, size=int(g.integers(1, 6)))))
    off = np.zeros(len(trials) + 1, np.int64)
    np.cumsum([len(x) for x in trials], out=off[1:])
    ids = np.array([e for x in trials for e in x], np.int32)
    check(ara, synth.Yet(100_000, off, ids))


def test_forward_only_prepare_and_backward_refusal(ara):
    import torch
    w = synth.tiny_random(1)
    yet = ara.PreparedYet.from_numpy(w.yet, "cuda", transposed=False)
    assert yet.handle.n_slices == 0 and not yet.handle.tr_off
    assert not yet.handle.t_off and not yet.handle.t_ids and not yet.handle.t_cnt
    tables = ara.EltTables.from_numpy(w.elts, "cuda")
    layers = ara.Layers(w.layers.elt_off, w.layers.elt_ids)
    et = torch.tensor(w.elts.terms, dtype=torch.float64, device="cuda")
    lt = torch.tensor(w.layers.terms, dtype=torch.float64, device="cuda")
    ylt, s_pre, _ = ara.ylt_forward(tables, yet, layers, et, lt, want_s_pre=True)
    cot = torch.ones((1,) + tuple(ylt.shape), dtype=torch.float64, device="cuda")
    with pytest.raises(ara.AraError, match="TRANSPOSED"):
        ara.ylt_backward(tables, yet, layers, et, lt, s_pre, cot)


@pytest.mark.parametrize("lens", [(8191, 8192, 8193), (20_000, 1, 0, 3000), (70_000,)])
def test_trials_beyond_one_sorted_chunk(ara, lens):
    """Trials around and beyond the 8192 occurrences sorted at once, among
    short ones, crowded into one range (segments beyond the codes staged in
    LDS: 48 and 128 per lane) and spread over several.  The longest trial
    exceeds the positions' limit of 65536, so it is checked without them."""
    g = np.random.default_rng(sum(lens))
    for crowd in (True, False):
        trials = []
        for k in range(400):
            n = lens[(k // 20) % len(lens)] if k % 20 == 0 else int(g.integers(0, 30))
            hi = 3000 if crowd and n > 1000 else 200_000
            trials.append(g.integers(0, hi, size=n))
        off = np.zeros(len(trials) + 1, np.int64)
        np.cumsum([len(x) for x in trials], out=off[1:])
        yet_np = synth.Yet(200_000, off, np.concatenate(trials).astype(np.int32))
        if max(lens) <= 65536:
            check(ara, yet_np)
        else:
            with pytest.raises(ara.AraError) as ex:
                ara.PreparedYet.from_numpy(yet_np, "cuda", positions=True)
            assert ex.value.status == 6
            check_codes(ara.PreparedYet.from_numpy(yet_np, "cuda"), yet_np)


def test_decreasing_offsets_are_refused(ara):
    off = np.arange(0, 5001, 5, dtype=np.int64)
    off[400], off[401] = off[401], off[400]
    with pytest.raises(ara.AraError) as ex:
        ara.PreparedYet.from_numpy(synth.Yet(1000, off, np.zeros(5000, np.int32)), "cuda")
    assert ex.value.status == 2


@pytest.mark.parametrize("n,mean,catalog", [
    (9000, 40, 30_000),      # blocks of 4500 trials that the slices cut, sparse headers
    (20_000, 12, 5_000),     # 7 blocks of trials, lists of about 7 occurrences: dense headers
    (8193, 3, 64),           # two blocks, one tile of the smallest size class
    (300, 200, 9),           # crowded events: tiles read twice (more records than held in registers)
    (70_000, 5, 3_000_000),  # many empty lists
])
def test_event_blocks(ara, n, mean, catalog):
    """The event-ordered blocks, through what is derived from them: the
    event-major lists, every event's count and the largest one (check), with
    block sizes that the slices do and do not cut, both header forms, counts
    of fifteen and more among short lists, and tiles beyond the registers."""
    g = np.random.default_rng(n)
    lens = g.poisson(mean, size=n)
    lens[::11] = 0
    off = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    ids = g.integers(0, catalog, size=int(off[-1]), dtype=np.int32)
    ids[g.random(ids.shape[0]) < 0.02] = catalog - 1       # a long list in the last group
    ids[g.random(ids.shape[0]) < 0.01] = catalog // 2
    check(ara, synth.Yet(catalog, off, ids))


def test_more_sorted_tiles_than_one_grid_row(ara):
    """9 million trials, all but a few empty, over 2^24 events: 1099 blocks of
    4096 tiles, 4.6e9 threads of the sort, more than a launch holds in one
    dimension.  Year losses of the trials that have occurrences."""
    import torch
    n, catalog = 9_000_000, 1 << 24
    g = np.random.default_rng(2)
    trials = np.sort(g.choice(n, size=4000, replace=False))
    trials[0], trials[-1] = 0, n - 1
    lens = np.zeros(n, np.int64)
    lens[trials] = g.integers(1, 20, size=4000)
    off = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    rec = np.sort(g.choice(catalog, size=50_000, replace=False)).astype(np.int32)
    rec[-1] = catalog - 1
    ids = rec[g.integers(0, 50_000, size=int(off[-1]))]
    loss = np.round(np.exp(g.normal(8.0, 1.0, size=50_000))).astype(np.float32)   # whole numbers: exact sums
    _say(f"trials {n} catalog {catalog}")
    yet = ara.PreparedYet.from_numpy(synth.Yet(catalog, off, ids), "cuda", transposed=False)
    tables = ara.EltTables.from_numpy(synth.Elts(catalog, np.array([0, 50_000], np.int64), rec, loss, None))
    terms = [torch.tensor([x], dtype=torch.float64, device="cuda") for x in ([1.0, 0.0, np.inf], [0.0, np.inf, 0.0, np.inf])]
    y, _, _ = ara.ylt_forward(tables, yet, ara.Layers([0, 1], [0]), *terms, check=True)
    want = np.bincount(np.repeat(np.arange(n), lens), weights=loss.astype(np.float64)[np.searchsorted(rec, ids)], minlength=n)
    assert np.array_equal(y[0].cpu().numpy(), want)


@pytest.mark.parametrize("flags", [0, 3, 4, 7])
def test_scratch_is_free_after_the_call(ara, flags):
    """One buffer and two give the same prepared YET, and what lies behind its
    kept bytes, or in the scratch, may be written over afterwards."""
    import ctypes
    import torch
    w = synth.config(0, n_trials=3000)
    off = torch.from_numpy(w.yet.offsets).cuda()
    ids = torch.from_numpy(w.yet.ids).cuda()
    n, nnz, catalog = w.yet.n_trials, w.yet.nnz, int(w.yet.catalog)
    lib = ara.library()
    nb, keep, scr = (ctypes.c_size_t() for _ in range(3))
    assert lib.ara_yet_prepare_bytes(n, nnz, catalog, flags, ctypes.byref(nb)) == 0
    assert lib.ara_yet_prepare_split_bytes(n, nnz, catalog, flags, ctypes.byref(keep), ctypes.byref(scr)) == 0
    _say(f"flags {flags}: {nb.value} bytes, {keep.value} kept")
    one = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
    two, scratch = (torch.empty(b.value, dtype=torch.uint8, device="cuda") for b in (keep, scr))
    yets = []
    for buf, s in ((one, None), (two, scratch)):
        y = object.__new__(ara.PreparedYet)
        y.handle, y.buf, y.device, y.n_trials, y.catalog = ara.ara_yet(), buf, buf.device, n, catalog
        args = (off.data_ptr(), ids.data_ptr(), n, catalog, flags, buf.data_ptr(), buf.numel())
        if s is None:
            assert lib.ara_yet_prepare(*args, None, ctypes.byref(y.handle)) == 0
        else:
            assert lib.ara_yet_prepare_split(*args, s.data_ptr(), scr.value - 1, None, ctypes.byref(y.handle)) == 4
            assert lib.ara_yet_prepare_split(*args, s.data_ptr(), s.numel(), None, ctypes.byref(y.handle)) == 0
        yets.append(y)
    one[keep.value:] = 0xA5
    scratch[:] = 0x5A
    check_codes(yets[1], w.yet)
    tables = ara.EltTables.from_numpy(w.elts)
    layers = ara.Layers(w.layers.elt_off, w.layers.elt_ids)
    et = torch.tensor(w.elts.terms, dtype=torch.float64, device="cuda")
    lt = torch.tensor(w.layers.terms, dtype=torch.float64, device="cuda")
    out = [ara.ylt_forward(tables, y, layers, et, lt, want_hits=True, check=True) for y in yets]
    assert all(torch.equal(a, b) for a, b in zip(*out))
    if flags & ara.PREP_TRANSPOSED:
        cot = torch.rand((1,) + tuple(out[0][0].shape), dtype=torch.float64, device="cuda")
        g = [ara.ylt_backward(tables, y, layers, et, lt, out[0][1], cot) for y in yets]
        assert all(torch.equal(a, b) for a, b in zip(*g))
    if flags & ara.PREP_POSITIONS:
        sigma = ara.SigmaTables.from_numpy(tables, synth.record_sigmas(1, w.elts))
        s = [ara.ylt_forward_su(tables, sigma, y, layers, et, lt, 9, check=True) for y in yets]
        assert all(torch.equal(a, b) for a, b in zip(*s))


@pytest.mark.parametrize("n,mean,catalog,freq", [
    (9000, 60, 30_000, [7, 8, 9, 126, 127, 128, 129, 130, 135, 136, 137, 519, 520, 521, 5000, 60_000]),   # blocks the slices cut
    (70_000, 10, 3_000, [200, 40_000, 200_000]),          # blocks inside slices too
    (500, 300, 12, []),                                    # nothing but long lists, one block in eight slices
    (40, 3000, 70, [20_000]),
])
def test_event_major_lists_of_frequent_events(ara, n, mean, catalog, freq):
    """Lists, and groups of eight events' entries, around and far beyond those
    that a wavefront takes together."""
    g = np.random.default_rng(catalog)
    lens = g.poisson(mean, size=n)
    lens[::17] = 0
    off = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    ids = g.integers(0, catalog, size=int(off[-1]), dtype=np.int32)
    at = g.permutation(len(ids))[:sum(freq)]
    ids[at] = np.repeat(g.choice(catalog, size=len(freq), replace=False), freq) if freq else 0
    check(ara, synth.Yet(catalog, off, ids))


@pytest.mark.parametrize("n,per,catalog,power", [(100_000, 500, 500_000, 6.0), (100_000, 500, 500_000, 3.0), (100_000, 500, 200, 1.0)])
def test_frequent_events_are_laid_out_in_time(ara, n, per, catalog, power):
    """The event-major copy of events of very unequal frequency, and of a small
    catalogue, in at most fifteen times the time of a YET as large with uniform
    frequencies over 500,000 events: one CU lays the most frequent event's lists
    of a slice out, a lane took over a hundred times as long."""
    import time
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    off = torch.arange(n + 1, dtype=torch.int64, device="cuda") * per
    u = torch.rand(n * per, generator=g, device="cuda", dtype=torch.float64)
    times = []
    for c, p in ((500_000, 1.0), (catalog, power)):
        ids = (u ** p * c).to(torch.int32).clamp_(0, c - 1)
        t = []
        for _ in range(4):
            torch.cuda.synchronize()
            a = time.perf_counter()
            ara.PreparedYet(off, ids, c)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - a)
        times.append(min(t))
    _say(f"{n} x {per} over {catalog}, u^{power}: {times[1] * 1e3:.2f} ms, uniform over 500,000 {times[0] * 1e3:.2f} ms")
    assert times[1] < 15.0 * times[0]


@pytest.mark.parametrize("n,mean,catalog", [(30, 1_500_000, 300_000), (9000, 9000, 40_000)])
def test_blocks_of_many_chunks_and_tiles(ara, n, mean, catalog):
    """Thousands of chunks of a block, over thousands of tiles: their sums are
    made by several workgroups.  The blocks through the year losses."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    lens = torch.randint(0, 2 * mean + 1, (n,), generator=g, device="cuda")
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=off[1:])
    ids = torch.randint(0, catalog, (int(off[-1]),), generator=g, dtype=torch.int32, device="cuda")
    rec = torch.randperm(catalog, generator=g, device="cuda", dtype=torch.int32)[:catalog // 3].contiguous()
    loss = torch.randint(1, 1000, (rec.numel(),), generator=g, device="cuda").float()   # whole numbers: exact sums
    _say(f"{n} x {mean} over {catalog}: {ids.numel()} occurrences")
    yet = ara.PreparedYet(off, ids, catalog, transposed=False)
    yet.handle.reserved |= 0x200   # the forward takes the blocks
    tables = ara.EltTables(torch.tensor([0, rec.numel()], device="cuda"), rec, loss, catalog)
    terms = [torch.tensor([x], dtype=torch.float64, device="cuda") for x in ([1.0, 0.0, np.inf], [0.0, np.inf, 0.0, np.inf])]
    y, _, _ = ara.ylt_forward(tables, yet, ara.Layers([0, 1], [0]), *terms, check=True)
    by_event = torch.zeros(catalog, dtype=torch.float64, device="cuda")
    by_event[rec.long()] = loss.double()
    want = torch.segment_reduce(by_event[ids.long()], "sum", offsets=off, initial=0.0)
    assert torch.equal(y[0], want)
