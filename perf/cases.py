"""The work a user has this library do, as cases that can be prepared, run and checked one by one.

Five kinds of pass, each through the public entry points:

  train    sweeps over one resident matrix (same_lda_sweep, _sweep_poisson or _sweep_sampled), then the state read back
  stream   one sweep over the resident minibatch while the next one is staged from pinned host memory, then committed
  heldout  the per-word log-likelihood of held-out documents (theta fitted by fold-in sweeps)
  sddmm    the normaliser at every nonzero
  vb       exp E[log beta] of a topic-word state, then the variational E-step of all documents

Corpora are drawn from the LDA generative process with the shapes of the presets in synth.py: a news collection (log-normal
lengths around 330 tokens, Zipf-skewed words), abstracts (Poisson 90) and the two small presets.
"""
from __future__ import annotations

import functools

import numpy as np
import torch

from paper_1409_5402_amd import binding, schedule, synth

BETA = 0.01


def _case(name, kind, D, V, K, length, mean_len, zipf, **more):
    c = {"kind": kind, "D": D, "V": V, "K": K, "length": length, "mean_len": mean_len, "zipf": zipf}
    c.update(more)
    if name:
        c = {"name": name, **c}
    return c


def listed():
    news = dict(length="lognormal", mean_len=330.0, zipf=1.1)
    formed = dict(start="formed", burn=100, settle=30)
    return [
        # a toy corpus fitted in one go: ten sweeps, then the parameters; every launch counts
        _case("tiny_fit", "train", 1_000, 2_000, 16, "poisson", 100.0, 0.0,
              form="multinomial", m_first=10, m_last=10, sweeps=10, start="formed", burn=0, settle=0),
        # a few thousand documents with the usual fifty topics (not a multiple of four), odd sizes, a quick look at a topic model
        _case("small_fit_k50", "train", 4_001, 15_013, 50, "lognormal", 150.3, 1.1,
              form="multinomial", m_first=5, m_last=5, sweeps=5, start="formed", burn=40, settle=20),
        # a mid-sized collection annealed from one copy to twenty
        _case("medium_annealed", "train", 50_000, 20_000, 64, "poisson", 200.0, 1.1,
              form="multinomial", m_first=1, m_last=20, sweeps=20, start="formed", burn=40, settle=0),
        # the headline: one sweep at m = 100 over the news collection with topics formed
        _case("news_sweep", "train", 270_000, 100_000, 256, form="multinomial", m_first=100, m_last=100, sweeps=1, **formed, **news),
        # the first sweeps of a run at m = 100 from the random start: a flat posterior, many topics per word
        _case("news_first_sweeps", "train", 27_000, 100_000, 256, form="multinomial", m_first=100, m_last=100, sweeps=2,
              start="random", burn=0, settle=0, **news),
        # many topics
        _case("news_k1024", "train", 27_000, 100_000, 1024, form="multinomial", m_first=100, m_last=100, sweeps=1, **formed, **news),
        # the Poisson form with a real number of copies
        _case("poisson_sweep", "train", 27_000, 100_000, 256, form="poisson", m_first=100.0, m_last=100.0, sweeps=1, **formed, **news),
        # uncollapsed Gibbs: one copy per token, theta and phi drawn instead of averaged
        _case("sampled_gibbs_k200", "train", 60_000, 50_021, 200, form="sampled", m_first=1, m_last=1, sweeps=2, **formed, **news),
        # one step of a stream of minibatches of 100k abstracts
        _case("stream_abstracts", "stream", 100_000, 140_000, 256, "poisson", 90.0, 1.05, m=30, rho=0.2),
        # held-out likelihood of a tenth of the news collection, as an evaluation between sweeps calls it
        _case("heldout_news", "heldout", 30_000, 100_000, 256, foldin=3, m=100, train_docs=10_000, **news),
        # the normaliser alone, as a diagnostic or another method's building block takes it
        _case("sddmm_news", "sddmm", 100_000, 100_000, 256, **news),
        # variational E-step, five iterations
        _case("vb_estep", "vb", 60_000, 100_000, 256, iters=5, **news),
    ]


def _log_uniform(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def draw(rng):
    """One more case: kinds by how often they are called, topics between the usual round numbers and any number, sizes over
    their logarithm, at most a tenth of the work of the largest listed case."""
    kind = rng.choice(["train"] * 6 + ["stream", "heldout", "sddmm", "vb"])
    K = rng.choice([20, 50, 64, 100, 128, 150, 200, 256, 300, 500, 512, 1000, 1024, int(_log_uniform(rng, 8, 1200)), int(_log_uniform(rng, 8, 1200))])
    length = rng.choice(["poisson", "lognormal"])
    mean_len = round(_log_uniform(rng, 40, 400), 1)
    V = int(_log_uniform(rng, 1_000, 120_000))
    most = min(60_000.0, 2.0e9 / (mean_len * K))
    D = int(_log_uniform(rng, 600, max(700.0, most)))
    zipf = rng.choice([0.0, 1.05, 1.1])
    if kind == "train":
        form = rng.choice(["multinomial"] * 4 + ["poisson", "sampled"])
        m = rng.choice([1, 2, 5, 10, 30, 100])
        if form == "poisson":
            m = round(m * (0.5 + rng.random()), 3)
        if rng.random() < 0.2:
            return _case(None, kind, D, V, K, length, mean_len, zipf, form=form, m_first=m, m_last=m, sweeps=2, start="random", burn=0, settle=0)
        return _case(None, kind, D, V, K, length, mean_len, zipf, form=form, m_first=m, m_last=m, sweeps=rng.choice([1, 2, 4]),
                     start="formed", burn=40, settle=20)
    if kind == "stream":
        return _case(None, kind, D, V, K, length, mean_len, zipf, m=rng.choice([1, 10, 30, 100]), rho=round(0.05 + 0.9 * rng.random(), 3))
    if kind == "heldout":
        return _case(None, kind, D, V, K, length, mean_len, zipf, foldin=rng.choice([1, 3, 5]), m=rng.choice([10, 100]), train_docs=max(600, D // 3))
    if kind == "vb":
        return _case(None, kind, D, V, K, length, mean_len, zipf, iters=rng.choice([1, 5, 10]))
    return _case(None, kind, D, V, K, length, mean_len, zipf)


def _room(case):
    """Entries of a buffer that takes one value per nonzero: their number differs a little from corpus to corpus, a program
    that goes through several allocates for the largest.  What lies behind the last nonzero stays zero."""
    return int(1.2 * case["D"] * case["mean_len"]) + 8_192


def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _alpha(case):
    return 50.0 / case["K"] if case["length"] == "lognormal" and case["K"] >= 100 else 0.1


def _corpus(case, seed, D=None):
    return synth.generate(D or case["D"], case["V"], min(case["K"], 256), _alpha(case), BETA, seed, length=case["length"],
                          mean_len=case["mean_len"], zipf_s=case["zipf"], device=_device())


def _state(corpus, case, seed):
    return synth.state(corpus, case["K"], _alpha(case), BETA, seed, zipf_s=case["zipf"])


def _lambda(corpus, case, seed):
    """A concentrated topic-word state of the variational method: the prior plus the tokens each topic holds of each word."""
    _, phi = synth.state(corpus.slice_docs(0, 1), case["K"], _alpha(case), BETA, seed, zipf_s=case["zipf"])
    return (BETA + phi * (float(corpus.tokens) / case["K"])).contiguous()


def _model(corpus, case, seed):
    return binding.SameLDA(corpus.D, corpus.V, corpus.colptr, corpus.rowidx, corpus.val, case["K"], _alpha(case), BETA, seed, 1)


_TYPES = {binding.THETA: torch.float32, binding.PHI: torch.float32, binding.NDK: torch.int32, binding.NWK: torch.int32}


def _buffers(g, which):
    """Device tensors the state is read into (the 32-bit counts as int32)."""
    shape = {binding.THETA: (g.D, g.K), binding.NDK: (g.D, g.K), binding.PHI: (g.V, g.K), binding.NWK: (g.V, g.K)}
    return {w: torch.empty(shape[w], dtype=_TYPES[w], device=_device()) for w in which}


def _read(g, buffers):
    """same_lda_get into device memory."""
    lib = binding.load()
    for which, t in buffers.items():
        rc = lib.same_lda_get(g._h, which, t.data_ptr(), t.numel() * 4, 1)
        if rc != 0:
            raise binding.SameLdaError(rc, lib.same_lda_last_error(g._h).decode())


def _copies(case):
    n, a, b = case["sweeps"], case["m_first"], case["m_last"]
    if a == b:
        return [a] * n
    return schedule.linear((a + b) / 2.0, n)


def prepare(case, seed):
    torch.manual_seed(seed)
    s = {"case": case}
    kind = case["kind"]
    if kind == "train":
        X = _corpus(case, seed)
        g = s["g"] = _model(X, case, seed)
        for _ in range(case["burn"]):
            g.sweep(1)
        for _ in range(case["settle"]):
            _sweep(g, case["form"], case["m_first"])
        g.synchronize()
        s["copies"] = _copies(case)
        s["out"] = _buffers(g, (binding.THETA, binding.PHI, binding.NDK, binding.NWK))
        if case["start"] == "random":                      # a run starts over from the checkpoint of its random start
            s["checkpoint"] = _buffers(g, (binding.THETA, binding.PHI))
            _read(g, s["checkpoint"])
            s["pass"] = g.pass_index
    elif kind == "stream":
        s["batches"] = []
        for i in range(2):
            c = _corpus(case, seed + 7919 * i)
            s["batches"].append((c.D,) + tuple(t.cpu().pin_memory() for t in (c.colptr, c.rowidx, c.val)))
        D, colptr, rowidx, val = s["batches"][0]
        g = s["g"] = binding.SameLDA(D, case["V"], colptr, rowidx, val, case["K"], _alpha(case), BETA, seed, 1)
        s["at"] = 0
        s["out"] = _buffers(g, (binding.PHI, binding.THETA))
        for _ in range(4):                                 # into the stream: phi has seen several minibatches
            _step(s)
        g.synchronize()
    elif kind == "heldout":
        g = s["g"] = _model(_corpus(case, seed, case["train_docs"]), case, seed)
        for _ in range(20):
            g.sweep(1)
        g.synchronize()
        s["test"] = _corpus(case, seed + 1)
    elif kind == "sddmm":
        X = _corpus(case, seed)
        g = s["g"] = _model(X, case, seed)
        theta, phi = _state(X, case, seed)
        g.set(binding.THETA, theta)
        g.set(binding.PHI, phi)
        s["mu"] = torch.zeros(_room(case), dtype=torch.float32, device=_device())
    elif kind == "vb":
        X = _corpus(case, seed)
        g = s["g"] = _model(X, case, seed)
        lam = s["lam"] = _lambda(X, case, seed)
        s["b"] = torch.empty_like(lam)
        s["shift"] = torch.empty(X.V, dtype=torch.float32, device=_device())
        s["gamma"] = torch.empty((X.D, case["K"]), dtype=torch.float32, device=_device())
        s["log_mu"] = torch.zeros(_room(case), dtype=torch.float32, device=_device())
    else:
        raise ValueError(kind)
    return s


def _sweep(g, form, m):
    if form == "poisson":
        g.sweep_poisson(m)
    elif form == "sampled":
        g.sweep_sampled(m)
    else:
        g.sweep(m)


def _step(s):
    g, case = s["g"], s["case"]
    g.sweep(case["m"], case["rho"])
    s["at"] ^= 1
    D, colptr, rowidx, val = s["batches"][s["at"]]
    g.stage_batch(D, colptr, rowidx, val, 1, 0)
    g.commit_batch()


def run(s):
    g, case = s["g"], s["case"]
    kind = case["kind"]
    if kind == "train":
        if "checkpoint" in s:
            for which, t in s["checkpoint"].items():
                g.set(which, t)
            g.pass_index = s["pass"]
        for m in s["copies"]:
            _sweep(g, case["form"], m)
        _read(g, s["out"])
        o = s["out"]
        return {"theta": o[binding.THETA], "phi": o[binding.PHI], "ndk": o[binding.NDK], "nwk": o[binding.NWK]}
    if kind == "stream":
        _step(s)
        _read(g, s["out"])
        return {"theta": s["out"][binding.THETA], "phi": s["out"][binding.PHI]}
    if kind == "heldout":
        t = s["test"]
        return {"ll": g.loglik(t.D, t.colptr, t.rowidx, t.val, case["foldin"], case["m"])}
    if kind == "sddmm":
        return {"mu": g.sddmm(s["mu"])}
    s["gamma"].fill_(1.0)
    g.vb_exp_elog_beta(s["lam"], s["b"], s["shift"])
    g.vb_estep(s["b"], s["shift"], 0.1, case["iters"], s["gamma"], s["log_mu"])
    return {"b": s["b"], "shift": s["shift"], "gamma": s["gamma"], "log_mu": s["log_mu"]}


@functools.lru_cache(maxsize=64)
def _nonzeros_per_document(V, K, alpha, length, mean_len, zipf):
    """From a sample of documents: the number of different words of a document has no closed form here."""
    c = synth.generate(2_000, V, min(K, 256), alpha, BETA, 0, length=length, mean_len=mean_len, zipf_s=zipf, device=_device())
    return c.nnz / c.D


def work(case):
    """Compulsory bytes and operations: ids and counts, theta and phi read once, the new counts and parameters written once;
    two operations per topic and nonzero for the normaliser (four per iteration for the variational step)."""
    D, V, K = case["D"], case["V"], case["K"]
    nnz = D * _nonzeros_per_document(V, K, _alpha(case), case["length"], case["mean_len"], case["zipf"])
    kind = case["kind"]
    sweep = {"bytes": 8 * nnz + D * (4 + 12 * K) + 12 * V * K, "flops": 2.0 * nnz * K}
    if kind == "train":
        return {k: case["sweeps"] * v for k, v in sweep.items()}
    if kind == "stream":                                   # and the next minibatch, its theta written
        return {"bytes": sweep["bytes"] + 16 * nnz + 4 * D * K, "flops": sweep["flops"]}
    if kind == "heldout":                                  # theta in and out per fold-in sweep, phi, and the final sums
        n = case["foldin"] + 1
        return {"bytes": n * (8 * nnz + D * (4 + 8 * K) + 4 * V * K), "flops": 2.0 * n * nnz * K}
    if kind == "sddmm":
        return {"bytes": 12 * nnz + 4 * K * (D + V), "flops": 2.0 * nnz * K}
    return {"bytes": 12 * nnz + 8 * K * (D + V), "flops": 4.0 * case["iters"] * nnz * K}


def tolerance(case):
    """Counts are whole numbers and the same.  theta and phi come from them by a division or two in binary32 (sampled: by
    binary32 sequences of a few dozen operations).  The normaliser adds K products of one sign (5e-8 from 64 bits at K = 256);
    the variational step feeds such sums back once per iteration (5e-8 after five, more after ten).  The log-likelihood adds logarithms in double of binary32 sums."""
    return {
        "train": {"rel": 1e-6, "max": 1e-5},
        "stream": {"rel": 1e-6, "max": 1e-5},
        "heldout": {"rel": 1e-6},
        "sddmm": {"rel": 4e-7, "max": 4e-6},
        "vb": {"rel": 2e-6, "max": 5e-5},
    }[case["kind"]]


def _chunks(n, size):
    return ((i, min(n, i + size)) for i in range(0, n, size))


def exact(case, seed):
    """What has a value in 64 bits: the normaliser and the variational step.  Sampled counts have none."""
    kind, K = case["kind"], case["K"]
    if kind not in ("sddmm", "vb"):
        return None
    X = _corpus(case, seed)
    doc = torch.repeat_interleave(torch.arange(X.D, device=_device()), (X.colptr[1:] - X.colptr[:-1]).long())
    word = X.rowidx.long()
    rows = max(1, int(2.0e8) // K)
    if kind == "sddmm":
        theta, phi = _state(X, case, seed)
        mu = torch.zeros(_room(case), dtype=torch.float64, device=_device())
        for lo, hi in _chunks(X.nnz, rows):
            mu[lo:hi] = (theta[doc[lo:hi]].double() * phi[word[lo:hi]].double()).sum(1)
        return {"mu": mu}
    lam = _lambda(X, case, seed).double()
    elog = torch.special.digamma(lam) - torch.special.digamma(lam.sum(0))
    shift = elog.max(dim=1).values
    b = torch.exp(elog - shift[:, None])
    del lam, elog
    cnt = X.val.double()
    alpha = float(np.float32(0.1))
    gamma = torch.ones((X.D, K), dtype=torch.float64, device=_device())
    log_mu = torch.zeros(_room(case), dtype=torch.float64, device=_device())
    for _ in range(case["iters"]):
        a = torch.exp(torch.special.digamma(gamma) - torch.special.digamma(gamma.sum(1))[:, None])
        acc = torch.zeros_like(gamma)
        for lo, hi in _chunks(X.nnz, rows):
            bw = b[word[lo:hi]]
            mu = (a[doc[lo:hi]] * bw).sum(1)
            acc.index_add_(0, doc[lo:hi], bw * (cnt[lo:hi] / mu)[:, None])
            log_mu[lo:hi] = torch.log(mu) + shift[word[lo:hi]]
        gamma = alpha + a * acc
    return {"b": b, "shift": shift, "gamma": gamma, "log_mu": log_mu}
