"""The work that a user of the library has it do, as cases that can be timed and
checked: pricing layers over a resident Year Event Table (YET), the gradients of
the tail metrics, event-level losses, secondary uncertainty, bringing in a new
portfolio or a new YET, and a burst of quotes.

A case is a dict of plain values.  `path` names the work (see PATHS), the other
fields the sizes:
  trials, mean    trials of the YET and their mean number of occurrences
  lengths         "fixed", "poisson" or "ragged" (uniform on 0..2*mean)
  catalog         events of the catalogue (IDs are uniform over it)
  layers          layers priced in one call
  elts            ELTs of each layer ("elts_step" more for each next layer)
  rec_lo, rec_hi  records of an ELT, uniform between the two
  p               tail probability of PML and TVaR
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1308_2572_amd as ara

DEV = "cuda"
PATHS = ("price", "hits", "fp32", "grad", "grad_dense", "event_losses", "uncertain", "book", "new_yet", "serve")


def listed():
    """The sizes are those of the repository's benchmark (1M x 1000 over 2M
    events, 15 ELTs of 20k; 1M x Poisson(1000) with four uneven layers; 200
    resident ELTs behind the quote server) and of its smoke run (2000 x 1000
    over 200k events), with ordinary and ragged sizes between."""
    return [
        # a what-if on a small book: the smallest call, latency and launches count
        dict(name="price_small", path="price", trials=2_000, mean=1000, lengths="fixed", catalog=200_000, layers=1,
             elts=15, elts_step=0, rec_lo=10_000, rec_hi=10_000, p=0.99),
        # the headline: one layer over a full YET, year losses and tail metrics
        dict(name="price_paper", path="price", trials=1_000_000, mean=1000, lengths="fixed", catalog=2_000_000, layers=1,
             elts=15, elts_step=0, rec_lo=20_000, rec_hi=20_000, p=0.99),
        # a programme of four layers of different sizes over uneven years
        dict(name="price_uneven4", path="price", trials=1_000_000, mean=1000, lengths="poisson", catalog=2_000_000,
             layers=4, elts=8, elts_step=4, rec_lo=5_000, rec_hi=30_000, p=0.99),
        # pricing with hit counts, ragged years, two layers, an odd number of trials
        dict(name="price_hits", path="hits", trials=200_003, mean=1000, lengths="ragged", catalog=2_000_000, layers=2,
             elts=10, elts_step=5, rec_lo=10_000, rec_hi=30_000, p=0.99),
        # the binary32 option at an ordinary size
        dict(name="price_fp32", path="fp32", trials=100_000, mean=1000, lengths="poisson", catalog=2_000_000, layers=1,
             elts=15, elts_step=0, rec_lo=20_000, rec_hi=20_000, p=0.99),
        # one optimisation step on the terms: forward, metrics and their gradients through autograd
        dict(name="grad_metrics", path="grad", trials=1_000_000, mean=1000, lengths="fixed", catalog=2_000_000, layers=1,
             elts=15, elts_step=0, rec_lo=20_000, rec_hi=20_000, p=0.99),
        # a caller's own objective on every year loss: a cotangent that differs from trial to trial
        dict(name="grad_own_objective", path="grad_dense", trials=300_001, mean=800, lengths="poisson", catalog=2_000_000,
             layers=2, elts=10, elts_step=5, rec_lo=10_000, rec_hi=30_000, p=0.99),
        # event-level year losses and yearly maxima for occurrence-exceedance metrics
        dict(name="event_losses", path="event_losses", trials=250_000, mean=1000, lengths="poisson", catalog=2_000_000,
             layers=1, elts=15, elts_step=0, rec_lo=20_000, rec_hi=20_000, p=0.99),
        # pricing with secondary uncertainty
        dict(name="price_uncertain", path="uncertain", trials=250_000, mean=1000, lengths="poisson", catalog=2_000_000,
             layers=1, elts=15, elts_step=0, rec_lo=20_000, rec_hi=20_000, p=0.99),
        # a new portfolio arrives as records: its tables, then its layers over a resident YET
        dict(name="new_book", path="book", trials=50_000, mean=1000, lengths="poisson", catalog=2_000_000, layers=4,
             elts=8, elts_step=4, rec_lo=5_000, rec_hi=30_000, p=0.99),
        # a new simulation of the years arrives: laid out, then a layer priced over it with gradients
        dict(name="new_yet", path="new_yet", trials=400_000, mean=1000, lengths="poisson", catalog=2_000_000, layers=1,
             elts=15, elts_step=0, rec_lo=20_000, rec_hi=20_000, p=0.99),
        # quotes arriving together at the server, half of them with gradients
        dict(name="quote_burst", path="serve", trials=1_000_000, mean=1000, lengths="poisson", catalog=2_000_000, layers=48,
             elts=200, elts_step=0, rec_lo=10_000, rec_hi=30_000, p=0.99),
    ]


#: most occurrences of a drawn case's YET, and most layers, by path
_MOST = {"price": (1_000_000_000, 6), "hits": (400_000_000, 3), "fp32": (400_000_000, 2), "grad": (600_000_000, 2),
         "grad_dense": (400_000_000, 3), "event_losses": (250_000_000, 2), "uncertain": (250_000_000, 2),
         "book": (100_000_000, 5), "new_yet": (400_000_000, 2), "serve": (600_000_000, 40)}


def draw(rng: random.Random) -> dict:
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(PATHS)
    most, most_layers = _MOST[path]
    layers = rng.randint(1, most_layers)
    mean = log_int(200, 2000)
    trials = min(log_int(1_000, 1_000_000), most // mean)
    if path == "price" and layers > 3:
        trials = min(trials, 600_000_000 // mean)
    catalog = log_int(100_000, 3_000_000)
    rec_lo = log_int(max(500, catalog // 300), catalog // 60)
    rec_hi = log_int(rec_lo, max(rec_lo, catalog // 50))
    lengths = rng.choice(("fixed", "poisson", "ragged"))
    p = rng.choice((0.9, 0.95, 0.99, 0.996))
    if path == "serve":
        return dict(path=path, trials=max(trials, 50_000), mean=min(mean, 1000), lengths=lengths, catalog=catalog,
                    layers=max(layers, 4), elts=rng.randint(30, 200), elts_step=0, rec_lo=rec_lo, rec_hi=rec_hi, p=p)
    return dict(path=path, trials=trials, mean=mean, lengths=lengths, catalog=catalog, layers=layers,
                elts=rng.randint(3, 20), elts_step=rng.randint(0, 4), rec_lo=rec_lo, rec_hi=rec_hi, p=p)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

class Inputs:
    """The raw inputs of a case on the GPU, from the seed alone."""

    def __init__(self, case: dict, seed: int):
        g = torch.Generator(device=DEV)
        g.manual_seed(int(seed) * 1_000_003 + 17)
        h = np.random.default_rng([int(seed), 1308])
        n, mean, C = case["trials"], case["mean"], case["catalog"]
        # lengths in pairs x and 2 * mean - x, so that the total is the same for every seed
        if case["lengths"] == "poisson":
            half = torch.poisson(torch.full((n // 2,), float(mean), device=DEV), generator=g).to(torch.int64).clamp_(max=2 * mean)
        elif case["lengths"] == "ragged":
            half = torch.randint(0, 2 * mean + 1, (n // 2,), generator=g, device=DEV)
        else:
            half = torch.full((n // 2,), mean, dtype=torch.int64, device=DEV)
        lens = torch.cat([half, 2 * mean - half, torch.full((n % 2,), mean, dtype=torch.int64, device=DEV)])
        self.catalog, self.n, self.p = C, n, case["p"]
        self.offsets = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
        torch.cumsum(lens, 0, out=self.offsets[1:])
        self.ids = torch.randint(0, C, (int(self.offsets[-1]),), generator=g, dtype=torch.int32, device=DEV)

        # ELT records: distinct events, lognormal(12, 1.5) binary32 losses
        serve = case["path"] == "serve"
        counts = [case["elts"]] if serve else [case["elts"] + j * case["elts_step"] for j in range(case["layers"])]
        n_elts = sum(counts)
        sizes = h.integers(case["rec_lo"], case["rec_hi"] + 1, size=n_elts)
        off = np.zeros(n_elts + 1, np.int64)
        np.cumsum(sizes, out=off[1:])
        self.rec_off = torch.from_numpy(off).to(DEV)
        self.rec_ids = torch.cat([torch.randperm(C, generator=g, device=DEV, dtype=torch.int32)[:int(s)] for s in sizes])
        z = torch.randn(int(off[-1]), generator=g, device=DEV)
        self.rec_loss = torch.exp(12.0 + 1.5 * z)
        cv = torch.rand(int(off[-1]), generator=g, device=DEV) * 1.25 + 0.25
        cv[torch.rand(int(off[-1]), generator=g, device=DEV) < 0.1] = 0.0
        self.rec_sigma = cv * self.rec_loss
        self.elt_terms = torch.tensor(np.array([1.0, 5e4, 5e6]) * h.uniform(0.97, 1.03, size=(n_elts, 3)), device=DEV)
        self.draw_seed = int(h.integers(0, 1 << 62))

        # layer terms in the benchmark's proportions to a year's expected loss
        def terms(n_records):
            year = 3e5 * mean * n_records / C
            r = np.exp(h.uniform(np.log([1e4, 1e6, 2e-3, 0.6]), np.log([1e6, 1e8, 0.2, 8.0])))
            return [r[0], r[1], r[2] * year, r[3] * year]

        self.elt_off = np.zeros(len(counts) + 1, np.int32)
        np.cumsum(counts, out=self.elt_off[1:])
        self.elt_ids = np.arange(n_elts, dtype=np.int32)
        self.quotes = []
        if serve:
            for k in range(case["layers"]):
                ids = h.choice(n_elts, size=5 + 13 * k % 21, replace=False).astype(np.int32)
                size = int(h.integers(max(1, n // 10), n + 1))
                begin = int(h.integers(0, n - size + 1))
                self.quotes.append((ids, terms(int(sizes[ids].sum())), begin, begin + size, k % 2 == 1))
        else:
            lt = [terms(int(sizes[a:b].sum())) for a, b in zip(self.elt_off, self.elt_off[1:])]
            self.layer_terms = torch.tensor(np.array(lt), device=DEV)
            # what the caller's objective asks of every metric, and of every year loss
            self.grad_out = torch.tensor([[1.0, 0.05, 0.1]] * len(lt), dtype=torch.float64, device=DEV)
            if case["path"] == "grad_dense":
                self.grad_ylt = torch.rand((len(lt), n), generator=g, dtype=torch.float64, device=DEV) / n


def prepare(case: dict, seed: int) -> dict:
    path = case["path"]
    i = Inputs(case, seed)
    s = {"path": path, "in": i}
    if path != "serve":
        s["layers"] = ara.Layers(i.elt_off, i.elt_ids)
    if path != "book":
        s["tables"] = ara.EltTables(i.rec_off, i.rec_ids, i.rec_loss, i.catalog)
    if path not in ("new_yet", "event_losses"):
        s["yet"] = ara.PreparedYet(i.offsets, i.ids, i.catalog, transposed=path in ("grad", "grad_dense", "serve"),
                                   positions=path == "uncertain")
    if path == "uncertain":
        s["sigma"] = ara.SigmaTables(s["tables"], i.rec_sigma)
    if path == "grad":
        i.elt_terms.requires_grad_(True)
        i.layer_terms.requires_grad_(True)
    if path == "grad_dense":   # the forward of the step, whose totals the backward reads
        s["s_pre"] = ara.ylt_forward(s["tables"], s["yet"], s["layers"], i.elt_terms, i.layer_terms)[1]
    if path == "serve":
        s["server"] = ara.QuoteServer(s["tables"], s["yet"], i.elt_terms)
    if path not in ("new_yet", "event_losses"):
        i.ids = None   # the program's own copy has gone into the layout
    return s


def run(s: dict):
    path, i = s["path"], s["in"]
    if path in ("price", "hits", "fp32", "book"):
        tables = ara.EltTables(i.rec_off, i.rec_ids, i.rec_loss, i.catalog) if path == "book" else s["tables"]
        ylt, _, hits = ara.ylt_forward(tables, s["yet"], s["layers"], i.elt_terms, i.layer_terms, want_s_pre=False,
                                       want_hits=path == "hits", fp32_accum=path == "fp32")
        out, _ = ara.metrics(ylt, i.p)
        return {"ylt": ylt, "metrics": out, "hits": hits} if path == "hits" else {"ylt": ylt, "metrics": out}
    if path in ("grad", "new_yet"):
        if path == "new_yet":
            yet = ara.PreparedYet(i.offsets, i.ids, i.catalog)
            et, lt = i.elt_terms.detach().requires_grad_(True), i.layer_terms.detach().requires_grad_(True)
        else:
            yet, et, lt = s["yet"], i.elt_terms, i.layer_terms
        ylt = ara.YLT.apply(et, lt, (s["tables"], yet, s["layers"], 0, i.n))
        out = ara.Metrics.apply(ylt, i.p)
        ge, gl = torch.autograd.grad(out, [et, lt], i.grad_out)
        return {"ylt": ylt.detach(), "metrics": out.detach(), "grad_elt": ge, "grad_layer": gl}
    if path == "grad_dense":
        ge, gl = ara.ylt_backward(s["tables"], s["yet"], s["layers"], i.elt_terms, i.layer_terms, s["s_pre"], i.grad_ylt)
        return {"grad_elt": ge, "grad_layer": gl}
    if path == "event_losses":
        yelt, occ_max = ara.yelt_forward(s["tables"], i.offsets, i.ids, s["layers"], i.elt_terms, i.layer_terms)
        return {"yelt": yelt, "occ_max": occ_max}
    if path == "uncertain":
        ylt, _ = ara.ylt_forward_su(s["tables"], s["sigma"], s["yet"], s["layers"], i.elt_terms, i.layer_terms,
                                    i.draw_seed, want_s_pre=False)
        out, _ = ara.metrics(ylt, i.p)
        return {"ylt": ylt, "metrics": out}
    srv = s["server"]
    tickets = [srv.submit(ids, terms, b, e, i.p, want_grad=grad) for ids, terms, b, e, grad in i.quotes]
    res = [srv.wait(t) for t in tickets]
    with_grad = [r for r in res if "grad_elt" in r]
    return {"metrics": np.stack([r["metrics"] for r in res]),
            "grad_layer": np.stack([r["grad_layer"] for r in with_grad]),
            "grad_elt": np.concatenate([r["grad_elt"].transpose(1, 0, 2) for r in with_grad])}


def work(case: dict) -> dict:
    """Each occurrence's event ID (4 bytes) and each trial's boundary (8 bytes)
    read once, each ELT record (8 bytes) once, each output written once.  The
    arithmetic: the look-up and the sum of each occurrence's loss, the draws of
    secondary uncertainty (a generator block and a lognormal, ~250 operations)."""
    path, n, L = case["path"], case["trials"], case["layers"]
    nnz = n * case["mean"]
    rec = (case["rec_lo"] + case["rec_hi"]) / 2
    elts = case["elts"] * L + case["elts_step"] * L * (L - 1) / 2
    held = min(1.0, elts / L * rec / case["catalog"])      # share of occurrences with a loss in a layer
    b, f = 4.0 * nnz + 8.0 * n + 8.0 * elts * rec + 8.0 * n * L, 2.0 * nnz * L * held
    if path == "hits":
        b += 4.0 * n * L
    elif path == "grad":                                  # the backward of the metrics: the tail trials' events again
        b += 4.0 * nnz * (1.0 - case["p"]) + 32.0 * n * L
        f *= 2.0
    elif path == "grad_dense":                            # the occurrences of events with a loss, the cotangents, the totals
        b = 4.0 * nnz * min(1.0, held * L) + 8.0 * elts * rec + 16.0 * n * L
    elif path == "event_losses":
        b += 8.0 * nnz * L
    elif path == "uncertain":
        f = 250.0 * nnz * elts * rec / case["catalog"]
    elif path == "book":
        b += 4.0 * elts * case["catalog"]                 # the direct-access tables, written
    elif path == "new_yet":
        b += 4.0 * nnz * 2.0                              # the layout for the forward and that for the backward, written
    elif path == "serve":                                 # each quote reads its share of the years; 15 ELTs on average
        held = min(1.0, 15 * rec / case["catalog"])
        b = 0.55 * L * (4.0 * nnz + 16.0 * n) + L * 15 * 8.0 * rec
        f = 0.55 * L * 2.0 * nnz * held
    return {"bytes": b, "flops": f}


# --------------------------------------------------------------------------
# the same results in 64 bits, from the definitions, in plain torch
# --------------------------------------------------------------------------

def _clamp(v, r, l):
    """min(max(v - r, 0), l), where it is strictly between (its slope is one), and where the limit holds."""
    y = v - r
    a = torch.where(y > 0, y, torch.zeros_like(y))
    below = a < l
    return torch.where(below, a, torch.full_like(a, float(l))), (y > 0) & below, ~below


def _dense(i: Inputs, k: int, values):
    a, b = int(i.rec_off[k]), int(i.rec_off[k + 1])
    t = torch.zeros(i.catalog, dtype=torch.float64, device=DEV)
    t[i.rec_ids[a:b].long()] = values[a:b].double()
    return t


def _occurrence_losses(i: Inputs, elts, terms):
    """O(e) of a layer over the catalogue, its slope, where its limit holds, and the number of ELTs holding e."""
    x = torch.zeros(i.catalog, dtype=torch.float64, device=DEV)
    held = torch.zeros(i.catalog, dtype=torch.int32, device=DEV)
    et = i.elt_terms.detach().cpu().numpy()
    for k in elts:
        loss = _dense(i, int(k), i.rec_loss)
        x = x + _clamp(loss * et[k, 0], et[k, 1], et[k, 2])[0]
        held += (loss != 0).to(torch.int32)
    return (*_clamp(x, terms[0], terms[1]), held)


def _chunks(i: Inputs, begin, end, most=1 << 27):
    """(first trial, last trial, first occurrence, last occurrence) of runs of whole trials."""
    off = i.offsets.cpu().numpy()
    a = begin
    while a < end:
        b = max(a + 1, min(end, int(np.searchsorted(off, off[a] + most, "right")) - 1))
        yield a, b, int(off[a]), int(off[b])
        a = b


def _totals(i: Inputs, per_event, begin, end):
    out = torch.zeros(end - begin, dtype=torch.float64, device=DEV)
    for a, b, u, v in _chunks(i, begin, end):
        out[a - begin:b - begin] = _sum_by_trial(i, per_event[i.ids[u:v]].double(), a, b)
    return out


def _sum_by_trial(i: Inputs, values, a, b):
    return torch.segment_reduce(values, "sum", offsets=i.offsets[a:b + 1] - i.offsets[a], initial=0.0)


def _metrics(ylt, p):
    """AAL, PML and TVaR of one row, and their derivatives by each year loss."""
    n = ylt.numel()
    r = max(1, min(n, n - math.floor(p * n + 1e-9)))
    top = torch.topk(ylt, r).values
    pml = top[-1]
    above, tied = ylt > pml, ylt == pml
    n_above, n_tied = int(above.sum()), int(tied.sum())
    w = torch.stack([torch.full_like(ylt, 1.0 / n), tied.double() / n_tied,
                     above.double() / r + tied.double() * ((r - n_above) / (r * n_tied))])
    return torch.stack([ylt.mean(), pml, top.mean()]), w


def _gradients(i: Inputs, elts, terms, totals, cotangents, begin, end):
    """Of sum_t c_t * year loss_t for each row c: [rows, elts, 3] by the ELTs' terms, [rows, 4] by the layer's."""
    occ, slope, capped, _ = _occurrence_losses(i, elts, terms)
    _, in_agg, at_agg = _clamp(totals, terms[2], terms[3])
    rows = cotangents.shape[0]
    W = torch.zeros((rows, i.catalog), dtype=torch.float64, device=DEV)
    hot = occ != 0
    lens = i.offsets[1:] - i.offsets[:-1]
    for a, b, u, v in _chunks(i, begin, end, 1 << 26):
        ids = i.ids[u:v]
        at = hot[ids].nonzero()[:, 0]
        trial = torch.repeat_interleave(torch.arange(a - begin, b - begin, device=DEV), lens[a:b], output_size=v - u)[at]
        for c in range(rows):
            W[c].index_add_(0, ids[at].long(), (cotangents[c] * in_agg)[trial])
    et = i.elt_terms.detach().cpu().numpy()
    ge = []
    for k in elts:
        loss = _dense(i, int(k), i.rec_loss)
        _, s, at = _clamp(loss * et[k, 0], et[k, 1], et[k, 2])
        through = W * slope
        ge.append(torch.stack([(through * (loss * s)).sum(1), -(through * s).sum(1), (through * at).sum(1)], 1))
    gl = torch.stack([-(W * slope).sum(1), (W * capped).sum(1), -(cotangents * in_agg).sum(1),
                      (cotangents * at_agg).sum(1)], 1)
    return torch.stack(ge, 1), gl


_LOW = 0xFFFFFFFF


def _philox(counter, k, key):
    """Philox4x32-10 of the counter words (i mod 2^32, i div 2^32, k, 0), as int64 words below 2^32."""
    c = [counter & _LOW, counter >> 32, torch.full_like(counter, k), torch.zeros_like(counter)]
    k0, k1 = key & _LOW, key >> 32
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & _LOW) ^ c[1] ^ k0, p1 & _LOW, ((p0 >> 32) & _LOW) ^ c[3] ^ k1, p0 & _LOW]
        k0, k1 = (k0 + 0x9E3779B9) & _LOW, (k1 + 0xBB67AE85) & _LOW
    return c


def _drawn_totals(i: Inputs, elts, terms):
    """Trial totals where every (occurrence, ELT) pair draws its loss."""
    et = i.elt_terms.detach().cpu().numpy()
    mean = {int(k): _dense(i, int(k), i.rec_loss) for k in elts}
    dev = {int(k): _dense(i, int(k), i.rec_sigma) for k in elts}
    union = torch.stack(list(mean.values())).ne(0).any(0)
    out = torch.zeros(i.n, dtype=torch.float64, device=DEV)
    for a, b, u, v in _chunks(i, 0, i.n, 1 << 25):
        ids = i.ids[u:v]
        at = union[ids].nonzero()[:, 0]
        ev = ids[at].long()
        x = torch.zeros(at.numel(), dtype=torch.float64, device=DEV)
        for k in map(int, elts):
            sub = (mean[k][ev] != 0).nonzero()[:, 0]
            mu, sd = mean[k][ev[sub]], dev[k][ev[sub]]
            w = _philox(at[sub] + u, k, i.draw_seed)
            u1, u2 = (((w[h + 1] << 20 | w[h] >> 12).double() + 0.5) * 2.0 ** -52 for h in (0, 2))
            s2 = torch.log1p((sd / mu) ** 2)
            z = torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(2.0 * math.pi * u2)
            loss = torch.where(sd == 0, mu, torch.exp(torch.log(mu) - 0.5 * s2 + torch.sqrt(s2) * z))
            x[sub] += _clamp(loss * et[k, 0], et[k, 1], et[k, 2])[0]
        occ = torch.zeros(v - u, dtype=torch.float64, device=DEV)
        occ[at] = _clamp(x, terms[0], terms[1])[0]
        out[a:b] = _sum_by_trial(i, occ, a, b)
    return out


def _event_losses(i: Inputs, per_event, terms, out, occ_max):
    for a, b, u, v in _chunks(i, 0, i.n, 1 << 24):
        lens = i.offsets[a + 1:b + 1] - i.offsets[a:b]
        inside = torch.arange(max(1, int(lens.max())), device=DEV)[None, :] < lens[:, None]
        occ = torch.zeros(inside.shape, dtype=torch.float64, device=DEV)
        occ[inside] = per_event[i.ids[u:v]]
        after = _clamp(torch.cumsum(occ, 1), terms[2], terms[3])[0]
        loss = torch.diff(after, dim=1, prepend=torch.zeros_like(after[:, :1])) * inside
        out[u:v] = loss[inside]
        occ_max[a:b] = loss.max(1).values


def exact(case: dict, seed: int):
    path = case["path"]
    i = Inputs(case, seed)
    if path == "serve":
        met, gls, ges = [], [], []
        for ids, terms, begin, end, grad in i.quotes:
            totals = _totals(i, _occurrence_losses(i, ids, terms)[0], begin, end)
            m, w = _metrics(_clamp(totals, terms[2], terms[3])[0], i.p)
            met.append(m)
            if grad:
                ge, gl = _gradients(i, ids, terms, totals, w, begin, end)
                ges.append(ge.transpose(0, 1))
                gls.append(gl)
        return {"metrics": torch.stack(met), "grad_layer": torch.stack(gls), "grad_elt": torch.cat(ges)}
    lists = [i.elt_ids[a:b] for a, b in zip(i.elt_off, i.elt_off[1:])]
    all_terms = i.layer_terms.cpu().numpy()
    L, nnz = len(lists), i.ids.numel()
    if path == "event_losses":
        yelt = torch.empty((L, nnz), dtype=torch.float64, device=DEV)
        occ_max = torch.zeros((L, i.n), dtype=torch.float64, device=DEV)
        for j, (ids, terms) in enumerate(zip(lists, all_terms)):
            _event_losses(i, _occurrence_losses(i, ids, terms)[0], terms, yelt[j], occ_max[j])
        return {"yelt": yelt, "occ_max": occ_max}
    ylt, met, hits, gls = [], [], [], []
    grad_elt = torch.zeros((int(i.elt_off[-1]), 3), dtype=torch.float64, device=DEV)
    for j, (ids, terms) in enumerate(zip(lists, all_terms)):
        if path == "uncertain":
            totals = _drawn_totals(i, ids, terms)
        else:
            occ, _, _, held = _occurrence_losses(i, ids, terms)
            totals = _totals(i, occ, 0, i.n)
            if path == "hits":
                hits.append(_totals(i, held, 0, i.n).to(torch.int32))
        year = _clamp(totals, terms[2], terms[3])[0]
        m, w = _metrics(year, i.p)
        ylt.append(year)
        met.append(m)
        if path in ("grad", "new_yet", "grad_dense"):
            c = i.grad_ylt[j:j + 1] if path == "grad_dense" else (i.grad_out[j][:, None] * w).sum(0, keepdim=True)
            ge, gl = _gradients(i, ids, terms, totals, c, 0, i.n)
            grad_elt[torch.from_numpy(ids.astype(np.int64)).to(DEV)] += ge[0]
            gls.append(gl[0])
    if path == "grad_dense":
        return {"grad_elt": grad_elt, "grad_layer": torch.stack(gls)}
    got = {"ylt": torch.stack(ylt), "metrics": torch.stack(met)}
    if path == "hits":
        got["hits"] = torch.stack(hits)
    if path in ("grad", "new_yet"):
        got.update(grad_elt=grad_elt, grad_layer=torch.stack(gls))
    return got
