"""Parity of the HIP forward (prepare, tables, occurrence table, stream) and
of the metrics kernels against the CPU oracle, through the C ABI.

Tolerances (the method reaches an exact result; only the order of the
per-trial summation differs between the two sides):
  hits            bit-exact
  year loss Y     |Y_gpu - Y_ref| <= 1e-9 * max(Y_ref, S_ref)   (S = total
                  before aggregate terms; near the aggregate retention a
                  plain relative error is ill-conditioned)
  S               1e-9 relative
  AAL             1e-9 relative
  PML             1e-9 * max(PML, S) over the trials whose oracle year loss
                  is the PML (the same rule as Y, at the selected trials)
  TVaR            1e-9 * mean of max(Y, S) over the oracle's r largest
                  year losses
  (PML exact, AAL and TVaR 1e-9 relative when computed from the same YLT)
"""
import sys

import numpy as np
import pytest

import oracle
import synth
from _indep import load_hand_example

pytestmark = pytest.mark.gpu
TOL = 1e-9


def _say(msg):
    print(f"[gpu-forward] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ara():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a device"
    import paper_1308_2572_amd as ara
    ara.library()
    return ara


class Engine:
    def __init__(self, ara, w, device="cuda"):
        import torch
        self.ara = ara
        self.w = w
        self.tables = ara.EltTables.from_numpy(w.elts, device)
        self.yet = ara.PreparedYet.from_numpy(w.yet, device)
        self.layers = ara.Layers(w.layers.elt_off, w.layers.elt_ids)
        self.et = torch.tensor(w.elts.terms, dtype=torch.float64, device=device)
        self.lt = torch.tensor(w.layers.terms, dtype=torch.float64, device=device)

    def forward(self, t0=0, t1=None, hits=True, et=None, lt=None):
        y, s, h = self.ara.ylt_forward(self.tables, self.yet, self.layers, self.et if et is None else et,
                                       self.lt if lt is None else lt, t0, t1, want_s_pre=True, want_hits=hits,
                                       check=True)
        return (y.cpu().numpy(), s.cpu().numpy(), None if h is None else h.cpu().numpy())


def assert_ylt(y, s, ref):
    bound = TOL * np.maximum(np.abs(ref["ylt"]), ref["s_pre"])
    bad = np.abs(y - ref["ylt"]) > bound
    assert not bad.any(), f"{bad.sum()} year losses off; worst {np.abs(y - ref['ylt'])[bad].max()}"
    sb = np.abs(s - ref["s_pre"]) > TOL * ref["s_pre"]
    assert not sb.any(), f"{sb.sum()} totals off"


def metric_bounds(ref, p):
    """Tolerance of (AAL, PML, TVaR) per layer of a forward: AAL plain
    relative; PML and TVaR by the year-loss rule at the trials the metric
    selects (the PML's trials, the r largest)."""
    y, s = ref["ylt"], ref["s_pre"]
    n = y.shape[1]
    r = oracle.tail_count(n, p)
    out = np.zeros((y.shape[0], 3))
    for j in range(y.shape[0]):
        order = np.argsort(-y[j], kind="stable")
        top = order[:r]
        pml = y[j, order[r - 1]]
        out[j, 0] = TOL * abs(y[j].mean())
        out[j, 1] = TOL * max(pml, s[j, y[j] == pml].max())
        out[j, 2] = TOL * np.maximum(y[j, top], s[j, top]).mean()
    return out


def oracle_ref(w, t0=0, t1=None, threads=1):
    tb = oracle.build_tables(w.elts)
    return oracle.forward(tb, w.yet, w.layers, w.elts.terms, w.layers.terms, t0, t1, n_threads=threads)


# ------------------------------------------------------------------ small cases
def test_hand_example_exact(ara):
    w, g = load_hand_example()
    e = Engine(ara, w)
    y, s, h = e.forward()
    assert y[0].tolist() == g["ylt"]
    assert s[0].tolist() == g["s_pre"]
    assert h[0].tolist() == g["hits"]
    import torch
    for p, m in g["metrics"].items():
        out, _ = ara.metrics(torch.tensor(y, device="cuda"), float(p))
        assert out.cpu().numpy()[0].tolist() == [m["aal"], m["pml"], m["tvar"]]


@pytest.mark.parametrize("seed", range(12))
def test_tiny_random_vs_oracle(ara, seed):
    w = synth.tiny_random(seed, n_trials=37 + 13 * seed, max_events=30, catalog=48 + 40 * seed, n_layers=3)
    _say(f"tiny seed {seed}")
    e = Engine(ara, w)
    ref = oracle_ref(w)
    y, s, h = e.forward()
    assert np.array_equal(h, ref["hits"])
    assert_ylt(y, s, ref)
    # without hits the (smaller) hot-only table must give the same totals
    y2, s2, _ = e.forward(hits=False)
    assert np.array_equal(y2, y) or np.allclose(y2, y, rtol=1e-13, atol=0)
    assert_ylt(y2, s2, ref)


def test_catalogue_spanning_many_ranges(ara):
    """Catalogue of 300,000 events (5 occurrence-table super-ranges, a ragged
    last one), 3000 trials with lengths 0..400."""
    g = np.random.default_rng(5)
    lens = g.integers(0, 401, size=3000)
    lens[::97] = 0
    off = np.zeros(3001, np.int64)
    np.cumsum(lens, out=off[1:])
    ids = g.integers(0, 300_000, size=int(off[-1]), dtype=np.int32)
    ids[:50] = 299_999
    ids[50:100] = 0
    elts = synth.lognormal_elts(77, [30_000, 5_000, 60_000, 1], 300_000, mu=11.0)
    elts.rec_ids[elts.rec_off[3]] = 299_999
    layers = synth.Layers(np.array([0, 4, 6, 6], np.int32), np.array([2, 0, 1, 3, 3, 2], np.int32),
                          np.array([[1e4, 5e6, 1e5, 5e7], [0.0, np.inf, 0.0, np.inf], [1e4, 1e6, 0, 1e7]]))
    w = synth.Workload("ranges", synth.Yet(300_000, off, ids), elts, layers, 0.9)
    e = Engine(ara, w)
    ref = oracle_ref(w)
    y, s, h = e.forward()
    assert np.array_equal(h, ref["hits"])
    assert_ylt(y, s, ref)
    assert np.all(y[2] == 0.0) and np.all(h[2] == 0)          # a layer with no ELTs


def test_trial_subsets_match_full_run(ara):
    w = synth.config(2, n_trials=9000)
    e = Engine(ara, w)
    y, s, h = e.forward()
    for t0, t1 in [(0, 1), (17, 4099), (4096, 4097), (8000, 9000), (123, 123)]:
        ys, ss, hs = e.forward(t0, t1)
        assert np.array_equal(ys, y[:, t0:t1]) and np.array_equal(ss, s[:, t0:t1]) and np.array_equal(hs, h[:, t0:t1])


@pytest.mark.parametrize("hits", [True, False])
def test_one_occurrence_trials_bit_exact(ara, hits):
    """Binary64: when every trial holds one occurrence, its total S is that
    event's occurrence loss O(e) (steps one to three of Algorithm 1: the
    lookups, each ELT's terms, the sum over the layer's ELTs in listed order,
    the occurrence terms), and the year loss is the aggregate terms of it.
    Both sides evaluate these in the same operations and order, so S, Y and
    the hit counts must be equal (==) for every event of a 200,000-event
    catalogue (each once, in shuffled order, then 20,000 repeats, with empty
    trials between), in three layers: scaled ELTs with mixed terms, three
    ELTs in a scrambled order, two without terms."""
    w0 = synth.config(0, n_trials=1)
    C = w0.elts.catalog
    g = np.random.default_rng(20)
    ev = np.concatenate([g.permutation(C), g.integers(0, C, 20_000)]).astype(np.int32)
    lens = np.ones(ev.shape[0] + 3000, np.int64)
    lens[g.choice(lens.shape[0], 3000, replace=False)] = 0          # empty trials
    off = np.zeros(lens.shape[0] + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    et = w0.elts.terms.copy()
    et[:, 0] = g.uniform(0.3, 3.0, 15)                              # products s*l round
    et[:, 1] = g.uniform(0.0, 2e5, 15)
    et[:, 2] = g.uniform(1e5, 5e6, 15)
    et[4] = [1.0, 0.0, np.inf]
    elts = synth.Elts(C, w0.elts.rec_off, w0.elts.rec_ids, w0.elts.rec_loss, et)
    layers = synth.Layers(np.array([0, 15, 18, 20], np.int32),
                          np.array(list(range(15)) + [9, 2, 13] + [4, 0], np.int32),
                          np.array([[1e5, 2e7, 1e5, 1e7], [3.3e4, 9e5, 0.0, np.inf], [0.0, np.inf, 0.0, np.inf]]))
    w = synth.Workload("one-occurrence", synth.Yet(C, off, ev), elts, layers, 0.9)
    e = Engine(ara, w)
    ref = oracle_ref(w, threads=8)
    y, s, h = e.forward(hits=hits)
    assert np.array_equal(s, ref["s_pre"]), f"{np.count_nonzero(s != ref['s_pre'])} totals differ"
    assert np.array_equal(y, ref["ylt"]), f"{np.count_nonzero(y != ref['ylt'])} year losses differ"
    if hits:
        assert np.array_equal(h, ref["hits"])
    assert np.count_nonzero(s[0]) > 10_000 and np.count_nonzero(s[1]) > 1000


def test_run_twice_bitwise_identical(ara):
    w = synth.config(0, n_trials=3000)
    e = Engine(ara, w)
    a = e.forward()
    b = e.forward()
    for x, z in zip(a, b):
        assert np.array_equal(x, z)


def test_empty_yet_and_empty_trials(ara):
    w = synth.tiny_random(1, n_trials=5)
    w.yet = synth.Yet(w.yet.catalog, np.zeros(6, np.int64), np.zeros(0, np.int32))
    e = Engine(ara, w)
    y, s, h = e.forward()
    assert np.all(y == 0) and np.all(s == 0) and np.all(h == 0)


# ------------------------------------------------------------------ errors
def test_invalid_inputs_are_rejected(ara):
    import torch
    w = synth.tiny_random(2)
    ids = w.yet.ids.copy()
    ids[3] = w.yet.catalog
    with pytest.raises(ara.AraError) as ex:
        ara.PreparedYet.from_numpy(synth.Yet(w.yet.catalog, w.yet.offsets, ids))
    assert ex.value.status == 2
    el = w.elts
    dup = el.rec_ids.copy()
    k = int(np.argmax(np.diff(el.rec_off) >= 2))
    dup[el.rec_off[k] + 1] = dup[el.rec_off[k]]
    with pytest.raises(ara.AraError) as ex:
        ara.EltTables.from_numpy(synth.Elts(el.catalog, el.rec_off, dup, el.rec_loss, el.terms))
    assert ex.value.status == 3
    e = Engine(ara, w)
    lt = e.lt.clone()
    lt[0, 0] = -1.0
    with pytest.raises(ara.AraError) as ex:
        e.forward(lt=lt)
    assert ex.value.status == 1
    et = e.et.clone()
    et[0, 0] = float("nan")
    with pytest.raises(ara.AraError):
        e.forward(et=et)


# ------------------------------------------------------------------ metrics
@pytest.mark.parametrize("seed", range(6))
def test_metrics_vs_oracle(ara, seed):
    import torch
    g = np.random.default_rng(seed)
    n = [1, 7, 1000, 10_000, 123_457, 400_000][seed]
    L = 1 + seed % 3
    y = g.lognormal(15, 2, size=(L, n))
    if seed % 2:
        y = np.round(y / 1e5) * 1e5             # many ties
    y[:, : n // 10] = 0.0
    for p in [0.5, 0.9, 0.99, 0.999]:
        out, wts = ara.metrics(torch.tensor(y, device="cuda"), p, want_weights=True)
        out, wts = out.cpu().numpy(), wts.cpu().numpy()
        ref = oracle.metrics(y, p)
        assert np.array_equal(out[:, 1], ref[:, 1])
        np.testing.assert_allclose(out[:, [0, 2]], ref[:, [0, 2]], rtol=TOL, atol=0)
        np.testing.assert_array_equal(wts, oracle.metric_weights(y, p))


@pytest.mark.parametrize("n_crowd,ties", [(16_000, 0), (16_385, 0), (60_000, 0), (60_000, 25_000), (200_000, 199_000)])
def test_metrics_crowded_prefix_bin(ara, n_crowd, ties):
    """Values crowded into one 23-bit prefix bin (the window [999936, 1000192)
    shares exponent and 11 leading mantissa bits): distinct values spaced
    1e-5 apart, some of them repeated, the rest of the row below the window.
    Below and above the 16384 values selected inside LDS."""
    import torch
    g = np.random.default_rng(n_crowd + ties)
    n = 250_000
    y = g.uniform(0.0, 9.9e5, size=(1, n))
    crowd = 1e6 + np.arange(n_crowd, dtype=np.float64) * 1e-5
    crowd[:ties] = crowd[ties]                       # the first `ties` values equal one value
    y[0, g.permutation(n)[:n_crowd]] = crowd
    for p in [0.5, 0.8, 0.95, 0.9999]:
        out, wts = ara.metrics(torch.tensor(y, device="cuda"), p, want_weights=True)
        out, wts = out.cpu().numpy(), wts.cpu().numpy()
        ref = oracle.metrics(y, p)
        assert np.array_equal(out[:, 1], ref[:, 1]), (p, out[:, 1], ref[:, 1])
        np.testing.assert_allclose(out[:, [0, 2]], ref[:, [0, 2]], rtol=TOL, atol=0)
        np.testing.assert_array_equal(wts, oracle.metric_weights(y, p))


@pytest.mark.parametrize("n_crowd,n_top", [(5_000, 4_000), (20_000, 12_000), (60_000, 40_000), (200_000, 150_000)])
def test_metrics_tied_at_the_top_of_the_bin(ara, n_crowd, n_top):
    """Year losses capped at one limit: the largest value of the crowded
    prefix bin repeated n_top times, the rest of the crowd distinct below it.
    Ranks inside the tied block (the PML is that value, found from the tie
    count alone), at its edge, just past it and past the whole crowd, below
    and above the 16384 values selected inside LDS."""
    import torch
    g = np.random.default_rng(n_crowd + n_top)
    n = 250_000
    y = g.uniform(0.0, 9.9e5, size=(1, n))
    crowd = 1e6 + np.arange(n_crowd, dtype=np.float64) * 1e-5
    crowd[n_crowd - n_top:] = crowd[-1]
    y[0, g.permutation(n)[:n_crowd]] = crowd
    for r in [1, n_top // 2, n_top, n_top + 1, n_crowd, n_crowd + 3]:
        p = (n - r) / n
        out, wts = ara.metrics(torch.tensor(y, device="cuda"), p, want_weights=True)
        out, wts = out.cpu().numpy(), wts.cpu().numpy()
        ref = oracle.metrics(y, p)
        assert np.array_equal(out[:, 1], ref[:, 1]), (r, out[:, 1], ref[:, 1])
        np.testing.assert_allclose(out[:, [0, 2]], ref[:, [0, 2]], rtol=TOL, atol=0)
        np.testing.assert_array_equal(wts, oracle.metric_weights(y, p))


def test_metrics_subnormal_and_zero_bins(ara):
    """PML and TVaR among subnormal year losses (exponent field 0: the
    gathered values' significands carry no implicit bit), among zeros, and
    just above them, against the oracle."""
    import torch
    g = np.random.default_rng(17)
    n = 50_000
    y = np.zeros((3, n))
    tiny = np.ldexp(g.integers(1, 1 << 40, size=n).astype(np.float64), -1074)   # subnormals
    y[0] = np.where(g.random(n) < 0.7, tiny, 0.0)
    y[1, : n // 3] = tiny[: n // 3]
    y[1, n // 3: n // 2] = g.lognormal(0.0, 1.0, size=n // 2 - n // 3)          # a few normal values above
    y[2] = 0.0
    y[2, :5] = [1e-300, 2e-310, 5e-320, 1.0, 0.0]
    for p in [0.01, 0.3, 0.5, 0.9, 0.99, 0.9999]:
        out, wts = ara.metrics(torch.tensor(y, device="cuda"), p, want_weights=True)
        out, wts = out.cpu().numpy(), wts.cpu().numpy()
        ref = oracle.metrics(y, p)
        assert np.array_equal(out[:, 1], ref[:, 1]), (p, out[:, 1], ref[:, 1])
        np.testing.assert_allclose(out[:, [0, 2]], ref[:, [0, 2]], rtol=TOL, atol=0)
        np.testing.assert_array_equal(wts, oracle.metric_weights(y, p))


@pytest.mark.parametrize("n", [4_000, 250_000])
@pytest.mark.parametrize("n_crowd,ties", [(1, 0), (2, 0), (255, 0), (256, 0), (257, 0), (256, 256), (256, 100), (257, 256)])
def test_metrics_few_keys_left(ara, n, n_crowd, ties):
    """Around the 256 keys of one prefix bin up to which the rank is found by
    counting, and its ties, in one workgroup's rows and in longer ones."""
    import torch
    g = np.random.default_rng(n_crowd + ties)
    y = g.uniform(0.0, 9.9e5, size=(1, n))
    crowd = 1e6 + np.arange(n_crowd, dtype=np.float64) * 1e-5
    crowd[:ties] = crowd[ties - 1]
    y[0, g.permutation(n)[:n_crowd]] = crowd
    for r in sorted({1, max(1, n_crowd // 2), n_crowd, n_crowd + 1}):
        p = (n - r) / n
        out, wts = ara.metrics(torch.tensor(y, device="cuda"), p, want_weights=True)
        out, wts = out.cpu().numpy(), wts.cpu().numpy()
        ref = oracle.metrics(y, p)
        assert np.array_equal(out[:, 1], ref[:, 1]), (r, out[:, 1], ref[:, 1])
        np.testing.assert_allclose(out[:, [0, 2]], ref[:, [0, 2]], rtol=TOL, atol=0)
        np.testing.assert_array_equal(wts, oracle.metric_weights(y, p))


@pytest.mark.parametrize("n", [1, 2, 1025, 8191, 8192, 8193])
@pytest.mark.parametrize("kind", ["spread", "tied", "zero", "subnormal"])
def test_metrics_around_one_workgroup(ara, n, kind):
    """Rows of up to 8192 values are selected by one workgroup in one kernel,
    longer ones by passes over the row."""
    import torch
    g = np.random.default_rng(n)
    y = g.lognormal(15, 2, size=(2, n))
    if kind == "tied":
        y = np.minimum(y, np.quantile(y, 0.7))
    elif kind == "zero":
        y[:, g.random(n) < 0.97] = 0.0
    elif kind == "subnormal":
        y[0] = np.ldexp(g.integers(0, 1 << 50, size=n).astype(np.float64), -1074)
    for p in [0.01, 0.5, 0.99]:
        out, wts = ara.metrics(torch.tensor(y, device="cuda"), p, want_weights=True)
        out, wts = out.cpu().numpy(), wts.cpu().numpy()
        ref = oracle.metrics(y, p)
        assert np.array_equal(out[:, 1], ref[:, 1])
        np.testing.assert_allclose(out[:, [0, 2]], ref[:, [0, 2]], rtol=TOL, atol=0)
        np.testing.assert_array_equal(wts, oracle.metric_weights(y, p))


def test_metrics_repeatable_and_layers_independent(ara):
    """Same answer twice (order-free gathering) and each layer as if alone."""
    import torch
    g = np.random.default_rng(11)
    y = g.lognormal(14, 1.5, size=(3, 70_000))
    y[1] = np.round(y[1] / 1e6) * 1e6
    y[2, :40_000] = 5e7
    t = torch.tensor(y, device="cuda")
    a, _ = ara.metrics(t, 0.99)
    b, _ = ara.metrics(t, 0.99)
    assert torch.equal(a, b)
    for l in range(3):
        one, _ = ara.metrics(t[l:l + 1].contiguous(), 0.99)
        assert torch.equal(one[0], a[l])


def test_metrics_constant_and_vjp(ara):
    import torch
    y = torch.full((2, 50_000), 1e8, dtype=torch.float64, device="cuda")
    out, _ = ara.metrics(y, 0.99)
    assert np.all(out.cpu().numpy() == 1e8)
    yr = torch.tensor(np.random.default_rng(0).exponential(10.0, (2, 1000)), device="cuda", requires_grad=True)
    m = ara.Metrics.apply(yr, 0.9)
    gout = torch.tensor([[1.0, 2.0, 3.0], [0.5, -1.0, 0.25]], dtype=torch.float64, device="cuda")
    (m * gout).sum().backward()
    wref = oracle.metric_weights(yr.detach().cpu().numpy(), 0.9)
    expect = np.einsum("lm,mlt->lt", gout.cpu().numpy(), wref)
    np.testing.assert_allclose(yr.grad.cpu().numpy(), expect, rtol=1e-15, atol=1e-18)


# ------------------------------------------------------------------ named workloads
def test_config0_full(ara):
    _say("workload 0 (10k x 1000, 15 ELTs)")
    w = synth.config(0)
    e = Engine(ara, w)
    ref = oracle_ref(w, threads=4)
    y, s, h = e.forward()
    assert np.array_equal(h, ref["hits"])
    assert_ylt(y, s, ref)
    import torch
    out, _ = ara.metrics(torch.tensor(y, device="cuda"), w.p)
    np.testing.assert_allclose(out.cpu().numpy(), oracle.metrics(ref["ylt"], w.p), rtol=TOL)


def test_config2_prefix_four_layers(ara):
    _say("workload 2 prefix (20k x Poisson(1000), 4 layers)")
    w = synth.config(2, n_trials=20_000)
    e = Engine(ara, w)
    ref = oracle_ref(w, threads=8)
    y, s, h = e.forward()
    assert np.array_equal(h, ref["hits"])
    assert_ylt(y, s, ref)


def test_config1_full_size_sampled(ara):
    """1,000,000 trials x 1,000 events, 15 ELTs over a 2,000,000-event
    catalogue, in the configuration the benchmark times: every year loss
    from the GPU; a random sample recomputed by the oracle one trial at a
    time; metrics checked on the full GPU YLT."""
    import torch
    _say("workload 1: generating 1M x 1000")
    w = synth.config(1)
    e = Engine(ara, w)
    _say("workload 1: forward")
    y, s, _ = e.forward(hits=False)
    g = np.random.default_rng(1)
    sample = np.unique(np.concatenate([g.integers(0, w.yet.n_trials, 300), [0, 1, w.yet.n_trials - 1]]))
    tb = oracle.build_tables(w.elts)
    for t in sample:
        ref = oracle.forward(tb, w.yet, w.layers, w.elts.terms, w.layers.terms, int(t), int(t) + 1)
        assert abs(y[0, t] - ref["ylt"][0, 0]) <= TOL * max(ref["ylt"][0, 0], ref["s_pre"][0, 0])
        assert abs(s[0, t] - ref["s_pre"][0, 0]) <= TOL * ref["s_pre"][0, 0]
    # hits on the sample through the hit-count path, over a trial sub-range
    yh, sh, hh = e.forward(int(sample[1]), int(sample[1]) + 1, hits=True)
    refh = oracle.forward(tb, w.yet, w.layers, w.elts.terms, w.layers.terms, int(sample[1]), int(sample[1]) + 1)
    assert np.array_equal(hh, refh["hits"])
    _say("workload 1: metrics")
    out, _ = ara.metrics(torch.tensor(y, device="cuda"), w.p)
    np.testing.assert_allclose(out.cpu().numpy(), oracle.metrics(y, w.p), rtol=TOL)
    assert np.all(y >= 0) and np.all(y <= w.layers.terms[0, 3])


def _full_parity(ara, w, label):
    """Every trial of a full-size workload against the oracle (all host
    threads): YLT and S to the tolerance, hit counts bit-exact, through both
    the plain path and the hit-count path (whose larger tables spill out of
    LDS on the uneven workload); AAL, PML and TVaR of the device YLT against
    those of the oracle's YLT (metric_bounds)."""
    import torch
    _say(f"{label}: oracle over every trial")
    ref = oracle_ref(w, threads=oracle.num_threads_available())
    e = Engine(ara, w)
    _say(f"{label}: forward")
    y, s, _ = e.forward(hits=False)
    assert_ylt(y, s, ref)
    yh, sh, hh = e.forward(hits=True)
    assert np.array_equal(hh, ref["hits"])
    assert np.array_equal(yh, y) and np.array_equal(sh, s)
    _say(f"{label}: metrics against the oracle's")
    out, _ = ara.metrics(torch.tensor(y, device="cuda"), w.p)
    out = out.cpu().numpy()
    want = oracle.metrics(ref["ylt"], w.p)
    bound = metric_bounds(ref, w.p)
    assert np.all(np.abs(out - want) <= bound), (out, want, bound)


def test_config1_full_size_every_trial(ara):
    _say("workload 1: generating 1M x 1000")
    _full_parity(ara, synth.config(1), "workload 1")


def test_config2_full_size_every_trial(ara):
    _say("workload 2: generating 1M x Poisson(1000), 4 layers over 55 ELTs")
    _full_parity(ara, synth.config(2), "workload 2")


def test_largest_catalogue(ara):
    """A catalogue of ARA_MAX_CATALOG = 2^26 events: 2048 ranges, so the YET
    preparation walks its per-range state in two windows and the forward's
    range table is at its largest; events crowd the first and last ranges and
    one in the middle, the rest are spread out."""
    cat = 1 << 26
    g = np.random.default_rng(31)
    n = 6000
    lens = g.integers(0, 120, size=n)
    off = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    ids = g.integers(0, cat, size=int(off[-1]), dtype=np.int64)
    pick = g.random(ids.shape[0])
    ids[pick < 0.2] = g.integers(0, 40_000, size=int((pick < 0.2).sum()))
    ids[(pick >= 0.2) & (pick < 0.4)] = g.integers(cat - 40_000, cat, size=int(((pick >= 0.2) & (pick < 0.4)).sum()))
    ids[(pick >= 0.4) & (pick < 0.5)] = g.integers(1 << 25, (1 << 25) + 30_000, size=int(((pick >= 0.4) & (pick < 0.5)).sum()))
    ids = ids.astype(np.int32)
    # ELTs drawn from the same crowded places so that many occurrences hit
    hot = np.unique(ids)
    recs = [np.sort(g.choice(hot, size=min(len(hot), k), replace=False)) for k in (20_000, 8_000, 30_000)]
    rec_off = np.zeros(4, np.int64)
    np.cumsum([len(r) for r in recs], out=rec_off[1:])
    rec_ids = np.concatenate(recs).astype(np.int32)
    rec_loss = np.exp(g.normal(11.0, 1.5, size=rec_ids.shape[0])).astype(np.float32)
    elts = synth.Elts(cat, rec_off, rec_ids, rec_loss, np.array([[1.0, 5e4, 5e6], [1.5, 1e4, 2e6], [0.8, 0.0, np.inf]]))
    layers = synth.Layers(np.array([0, 3, 4], np.int32), np.array([0, 1, 2, 1], np.int32),
                          np.array([[1e4, 2e7, 1e5, 1e8], [0.0, np.inf, 0.0, np.inf]]))
    w = synth.Workload("max-catalogue", synth.Yet(cat, off, ids), elts, layers, 0.95)
    _say("largest catalogue: prepare and forward")
    e = Engine(ara, w)
    assert e.yet.handle.n_ranges == 2048
    ref = oracle_ref(w, threads=oracle.num_threads_available())
    y, s, h = e.forward()
    assert np.array_equal(h, ref["hits"])
    assert_ylt(y, s, ref)
