"""The work whose speed this library is judged by: what a program that trains
students (and makes their targets) has it do, through the public entry points.

A case is a dict of plain values; its "kind" says which part of the library it
exercises:

  train    one training step (trainer.StudentStep.step): forward, soft-target
           CE, BPTT, then threshold compression and the decoded update ("gtc")
           or plain local SGD
  score    lstm_am_forward of one chunk with the state carried in and out
           (validation, streaming)
  teacher  blstm_teacher_forward of a batch whose targets are to be stored
  targets  the k best teacher logits, their posteriors, and the CE of student
           logits against them
  gtc      threshold encode of a whole gradient with its residual, and decode
  workers  aggregate of several workers' compressed updates, and the SGD step
  bmuf     the block update that ends a block of local SGD
  inputs   frame stacking with causal mean and normalisation, delayed targets

`exact` evaluates each kind in 64 bits with plain torch.
"""

import math

import numpy as np
import torch

from paper_1904_10584_amd import binding as am
from paper_1904_10584_amd import synth
from paper_1904_10584_amd.trainer import StudentStep

DEV = "cuda"
LR, MASS, ZIPF = 0.01, 0.98, 1.1
PAPER_PARAMS = 24_145_848  # 5 x 768, 192 inputs, 3000 classes


# ------------------------------------------------------------------ cases --

def _train(name, layers, input_dim, hidden, classes, T, B, K, len_lo=0, dtype="bf16", gtc=True,
           tau=1e-4):
    c = dict(kind="train", layers=layers, input_dim=input_dim, hidden=hidden, classes=classes, T=T,
             B=B, K=K, len_lo=len_lo, dtype=dtype, gtc=gtc, tau=tau)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest model of the workloads, fp32 throughout: a developer's
        # quick run, made of launches
        _train("step tiny f32", 2, 64, 64, 500, T=50, B=16, K=5, dtype="f32", tau=1e-3),
        # the paper's student on its chunked batch: what the framework is for
        _train("step paper", 5, 192, 768, 3000, T=64, B=256, K=20),
        # the wide student
        _train("step wide", 5, 192, 1536, 6000, T=64, B=512, K=20),
        # whole utterances instead of chunks (200 to 1500 frames)
        _train("step varlen", 5, 192, 768, 3000, T=1500, B=128, K=20, len_lo=200),
        # a smaller student on a small worker batch of ragged chunks, local
        # SGD between BMUF blocks
        _train("step small", 3, 120, 512, 2000, T=40, B=48, K=10, len_lo=13, gtc=False),
        # scoring a few streams chunk by chunk, the state carried
        dict(kind="score", name="score chunk", layers=5, input_dim=192, hidden=768, classes=3000,
             T=32, B=12),
        # teacher logits of one chunked batch
        dict(kind="teacher", name="teacher", layers=5, input_dim=192, hidden=768, classes=3000,
             T=64, B=256, len_lo=0),
        # stored k-best targets of the same batch, and the CE against them with
        # the first frames of each chunk masked (three-frame look-ahead)
        dict(kind="targets", name="targets and ce", N=16384, classes=3000, K=20, masked=True,
             dtype="bf16"),
        # the paper model's gradient at a running trainer's send rate (about 1 %)
        dict(kind="gtc", name="gtc", n=PAPER_PARAMS, ratio=0.0125, noalloc=False),
        # eight workers' updates
        dict(kind="workers", name="workers", n=PAPER_PARAMS, streams=8, rate=0.01),
        # eight local models into the global one, with the restart copies
        dict(kind="bmuf", name="bmuf", n=PAPER_PARAMS, count=8),
        # raw 10 ms frames of whole utterances to packed model inputs
        dict(kind="inputs", name="inputs", B=128, T=1500, len_lo=200, raw_dim=64, K=20,
             dtype="bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(rng, lo, hi, m):
    """A multiple of m in [lo, hi], spread over the logarithm."""
    return min(hi // m, max(-(-lo // m), round(_log(rng, lo, hi) / m))) * m


def _hidden(rng, lo, hi):
    """Layer widths are multiples of 64 as a rule, of 16 now and then."""
    return _mult(rng, lo, hi, 16 if rng.random() < 0.15 else 64)


def draw(rng):
    kind = rng.choice(["train"] * 5 + ["score", "score", "teacher", "targets", "gtc", "workers",
                                       "bmuf", "inputs"])
    if kind == "train":
        if rng.random() < 0.15:
            T = rng.randint(5, 64)
            return _train(None, rng.randint(1, 3), _mult(rng, 16, 128, 4), _mult(rng, 16, 256, 16),
                          _mult(rng, 64, 1000, 4), T, _log(rng, 2, 64), rng.randint(1, 10),
                          len_lo=rng.choice([0, 1 + T // 4]), dtype="f32", tau=1e-3)
        while True:
            layers, hidden = rng.randint(1, 5), _hidden(rng, 64, 1536)
            whole = hidden <= 768 and rng.random() < 0.3
            T = _log(rng, 100, 600) if whole else _log(rng, 8, 100)
            B = _log(rng, 4, 128) if whole else _log(rng, 4, 512)
            c = _train(None, layers, _mult(rng, 40, 240, 8), hidden, _mult(rng, 500, 6000, 8), T, B,
                       rng.randint(1, 32), len_lo=1 + T // 7 if whole or rng.random() < 0.3 else 0,
                       gtc=rng.random() < 0.6)
            if work(c)["flops"] <= 1.0e13 and layers * T <= 1200:
                return c
    if kind == "score":
        return dict(kind=kind, layers=rng.randint(1, 5), input_dim=_mult(rng, 40, 240, 8),
                    hidden=_hidden(rng, 64, 1536), classes=_mult(rng, 500, 6000, 8),
                    T=_log(rng, 1, 64), B=_log(rng, 1, 128))
    if kind == "teacher":
        T = _log(rng, 8, 200)
        return dict(kind=kind, layers=rng.randint(1, 5), input_dim=_mult(rng, 40, 240, 8),
                    hidden=_hidden(rng, 64, 768), classes=_mult(rng, 500, 6000, 8), T=T,
                    B=_log(rng, 4, 256), len_lo=rng.choice([0, 1 + T // 7]))
    if kind == "targets":
        return dict(kind=kind, N=_log(rng, 100, 40000), classes=_mult(rng, 100, 8192, 4),
                    K=rng.randint(1, 64), masked=rng.random() < 0.5,
                    dtype=rng.choice(["bf16", "bf16", "f32"]))
    if kind == "gtc":
        n = _log(rng, 20_000, 60_000_000)
        return dict(kind=kind, n=n, ratio=rng.choice([0.002, 0.01, 0.05, 0.5]),
                    noalloc=n <= am.ENCODE_NOALLOC_MAX_N and rng.random() < 0.5)
    if kind == "workers":
        return dict(kind=kind, n=_log(rng, 20_000, 60_000_000), streams=_log(rng, 2, 32),
                    rate=rng.choice([0.002, 0.01, 0.03]))
    if kind == "bmuf":
        return dict(kind=kind, n=_log(rng, 20_000, 60_000_000), count=rng.randint(1, 16))
    T = _log(rng, 20, 1500)
    return dict(kind=kind, B=_log(rng, 4, 512 if T <= 300 else 128), T=T,
                len_lo=rng.choice([0, 1 + T // 7]), raw_dim=rng.choice([40, 64, 80]),
                K=rng.randint(1, 32), dtype=rng.choice(["bf16", "bf16", "f32"]))


# ----------------------------------------------------------------- inputs --

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(n, bound, g):
    return (torch.rand(n, generator=g, device=DEV) * 2.0 - 1.0) * bound


def _lengths(case):
    """Lengths U{len_lo..T}, longest first and the longest of T frames (a
    batch is cut to its longest utterance), the same for every seed (outputs
    keep their shapes); None: every sequence has T."""
    if not case["len_lo"]:
        return None
    lens = synth.utterance_lengths(case["B"], case["len_lo"], case["T"]).tolist()
    lens[0] = case["T"]
    return lens


def _frames(case, lengths):
    return case["T"] * case["B"] if lengths is None else sum(lengths)


def _teacher_targets(N, C, K, mass, g, seed):
    """K classes per frame, Zipf-distributed without replacement, with
    Dirichlet(0.3) probabilities of the given mass."""
    logp = -ZIPF * torch.log(torch.arange(1, C + 1, device=DEV, dtype=torch.float32))
    idx = torch.empty((N, K), dtype=torch.int32, device=DEV)
    for s in range(0, N, 16384):
        e = min(N, s + 16384)
        u = torch.rand((e - s, C), generator=g, device=DEV).clamp_(1e-30, 1.0)
        idx[s:e] = torch.topk(logp - torch.log(-torch.log(u).clamp_min_(1e-30)), K, dim=1).indices
    w = np.random.default_rng(seed).gamma(0.3, size=(N, K)).astype(np.float32) + 1e-6
    return idx, torch.from_numpy(mass * w / w.sum(1, keepdims=True)).to(DEV)


def _model(case, dtype):
    return am.Model(case["layers"], case["input_dim"], case["hidden"], case["classes"],
                    am.BF16 if dtype == "bf16" else am.F32)


def _train_inputs(case, seed):
    g = _gen(seed)
    lengths = _lengths(case)
    N = _frames(case, lengths)
    n = am.param_count(_model(case, case["dtype"]))
    master = _uniform(n, 1.0 / math.sqrt(case["hidden"]), g)
    x = torch.randn((N, case["input_dim"]), generator=g, device=DEV)
    idx, prob = _teacher_targets(N, case["classes"], min(case["K"], case["classes"]), MASS, g, seed)
    return lengths, master, x, idx, prob


def _score_inputs(case, seed):
    g = _gen(seed)
    n = am.param_count(_model(case, "bf16"))
    L, B, H = case["layers"], case["B"], case["hidden"]
    params = _uniform(n, 1.0 / math.sqrt(H), g).bfloat16()
    x = torch.randn((case["T"] * B, case["input_dim"]), generator=g, device=DEV).bfloat16()
    h0 = 0.2 * torch.randn((L, B, H), generator=g, device=DEV)
    c0 = 0.4 * torch.randn((L, B, H), generator=g, device=DEV)
    return params, x, h0.clamp_(-1.0, 1.0), c0


def _teacher_inputs(case, seed):
    g = _gen(seed)
    lengths = _lengths(case)
    N = _frames(case, lengths)
    n = am.teacher_param_count(_model(case, "bf16"))
    params = _uniform(n, 1.0 / math.sqrt(case["hidden"]), g).bfloat16()
    x = torch.randn((N, case["input_dim"]), generator=g, device=DEV).bfloat16()
    return lengths, params, x


def _target_inputs(case, seed):
    g = _gen(seed)
    N, C = case["N"], case["classes"]
    zt = 2.5 * torch.randn((N, C), generator=g, device=DEV)
    zs = 0.5 * zt + torch.randn((N, C), generator=g, device=DEV)
    mask = (torch.rand(N, generator=g, device=DEV) > 3.0 / 64).to(torch.uint8) if case["masked"] else None
    return zt, zs, mask


def _gtc_inputs(case, seed):
    """A gradient of standard deviation ratio x tau, and the residual of a
    running trainer."""
    g = _gen(seed)
    grad = torch.randn(case["n"], generator=g, device=DEV) * (1e-4 * case["ratio"])
    return grad, _uniform(case["n"], 0.99e-4, g)


def _worker_inputs(case, seed):
    g = _gen(seed)
    n, S = case["n"], case["streams"]
    rows = []
    for _ in range(S):
        at = torch.nonzero(torch.rand(n, generator=g, device=DEV) < case["rate"]).view(-1)
        sign = torch.randint(0, 2, at.shape, generator=g, device=DEV)
        rows.append(((at << 1) | sign).to(torch.int32))
    words = torch.zeros((S, max(16, max(r.numel() for r in rows))), dtype=torch.int32, device=DEV)
    for s, r in enumerate(rows):
        words[s, :r.numel()] = r
    counts = torch.tensor([r.numel() for r in rows], dtype=torch.int64, device=DEV)
    return words, counts, _uniform(n, 1.0 / math.sqrt(768), g)


def _bmuf_inputs(case, seed):
    g = _gen(seed)
    n, N = case["n"], case["count"]
    wg = _uniform(n, 1.0 / math.sqrt(768), g)
    delta = 1e-3 * torch.randn(n, generator=g, device=DEV)
    models = torch.empty((N, n), device=DEV)
    for i in range(N):
        models[i] = wg + 1e-3 * torch.randn(n, generator=g, device=DEV)
    return models, wg, delta


def _raw_inputs(case, seed):
    """Raw log mel frames around a per-dimension level, longest first."""
    g = _gen(seed)
    lengths = _lengths(case) or [case["T"]] * case["B"]
    raw_lengths = [3 * t + (i % 3) for i, t in enumerate(lengths)]  # incomplete last stacks too
    D = case["raw_dim"]
    raw = 2.0 + 3.0 * torch.randn((1, D), generator=g, device=DEV)
    raw = raw + torch.randn((sum(raw_lengths), D), generator=g, device=DEV)
    mean = 0.1 * torch.randn(3 * D, generator=g, device=DEV)
    std = 0.5 + torch.rand(3 * D, generator=g, device=DEV)
    N, K = sum(lengths), case["K"]
    idx = torch.randint(0, 3000, (N, K), generator=g, device=DEV, dtype=torch.int32)
    prob = torch.rand((N, K), generator=g, device=DEV)
    return lengths, raw_lengths, raw, mean, std, idx, prob


# ---------------------------------------------------------- prepare and run --

class _State:
    def __init__(self, **kw):
        self.__dict__.update(kw)


def _bytes(n):
    return torch.zeros(max(256, n), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        lengths, master, x, idx, prob = _train_inputs(case, seed)
        step = StudentStep(_model(case, case["dtype"]), case["T"], case["B"], idx.shape[1],
                           lengths=lengths, lr=LR, tau=case["tau"], gtc=case["gtc"], device=DEV)
        step.load_params(master)
        step.load_batch(x, idx, prob)
        return _State(kind=kind, step=step)
    if kind == "score":
        params, x, h0, c0 = _score_inputs(case, seed)
        m = _model(case, "bf16")
        N = case["T"] * case["B"]
        return _State(kind=kind, m=m, T=case["T"], B=case["B"], params=params, x=x, h0=h0, c0=c0,
                      hT=torch.zeros_like(h0), cT=torch.zeros_like(c0),
                      logits=torch.zeros((N, m.classes), device=DEV),
                      ws=_bytes(am.workspace_bytes(m, case["T"], case["B"], N)))
    if kind == "teacher":
        lengths, params, x = _teacher_inputs(case, seed)
        m = _model(case, "bf16")
        N = x.shape[0]
        return _State(kind=kind, m=m, T=case["T"], B=case["B"], lengths=lengths, params=params, x=x,
                      logits=torch.zeros((N, m.classes), device=DEV),
                      ws=_bytes(am.teacher_workspace_bytes(m, case["T"], case["B"], N)))
    if kind == "targets":
        zt, zs, mask = _target_inputs(case, seed)
        N, K = case["N"], case["K"]
        dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        return _State(kind=kind, zt=zt, zs=zs, mask=mask,
                      idx=torch.zeros((N, K), dtype=torch.int32, device=DEV),
                      val=torch.zeros((N, K), device=DEV), prob=torch.zeros((N, K), device=DEV),
                      loss=torch.zeros(1, device=DEV),
                      dz=torch.zeros((N, case["classes"]), dtype=dt, device=DEV),
                      ws=_bytes(am.ce_workspace_bytes(N)))
    if kind == "gtc":
        grad, residual = _gtc_inputs(case, seed)
        n = case["n"]
        return _State(kind=kind, noalloc=case["noalloc"], grad=grad, residual=residual,
                      words=torch.zeros(n, dtype=torch.int32, device=DEV),
                      count=torch.zeros(1, dtype=torch.int64, device=DEV),
                      dense=torch.zeros(n, device=DEV), ws=_bytes(am.encode_workspace_bytes(n)))
    if kind == "workers":
        words, counts, master = _worker_inputs(case, seed)
        n = case["n"]
        return _State(kind=kind, words=words, counts=counts, master=master,
                      weights=master.bfloat16(), dense=torch.zeros(n, device=DEV),
                      ws=_bytes(am.decode_multi_workspace_bytes(case["streams"], n)))
    if kind == "bmuf":
        models, wg, delta = _bmuf_inputs(case, seed)
        return _State(kind=kind, models=models, wg=wg, delta=delta, local=torch.zeros_like(wg),
                      local16=torch.zeros(case["n"], dtype=torch.bfloat16, device=DEV))
    lengths, raw_lengths, raw, mean, std, idx, prob = _raw_inputs(case, seed)
    N = sum(lengths)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    return _State(kind=kind, T=max(lengths), B=case["B"], lengths=lengths, raw_lengths=raw_lengths,
                  raw=raw, mean=mean, std=std, idx=idx, prob=prob,
                  x=torch.zeros((N, 3 * case["raw_dim"]), dtype=dt, device=DEV),
                  idx_out=torch.zeros_like(idx), prob_out=torch.zeros_like(prob),
                  mask=torch.zeros(N, dtype=torch.uint8, device=DEV))


def _bmuf_rates(count):
    eta = 1.0 - 1.0 / max(2, count)
    return eta, eta, 1.0 * count * (1.0 - eta)  # eta, eta_next, zeta = C N (1 - eta), C = 1


def run(s):
    if s.kind == "train":
        s.step.step()
        return {"loss": s.step.loss, "logits": s.step.logits, "grads": s.step.grads,
                "master": s.step.master}
    if s.kind == "score":
        am.lstm_am_forward(s.m, s.params, s.x, s.T, s.B, s.logits, s.ws, h0=s.h0, c0=s.c0, hT=s.hT,
                           cT=s.cT)
        return {"logits": s.logits, "hT": s.hT, "cT": s.cT}
    if s.kind == "teacher":
        am.blstm_teacher_forward(s.m, s.params, s.x, s.T, s.B, s.logits, s.ws, lengths=s.lengths)
        return s.logits
    if s.kind == "targets":
        am.kbest_logits(s.zt, s.idx, s.val)
        am.kbest_posteriors(s.val, s.prob)
        am.sparse_soft_ce(s.zs, s.idx, s.prob, s.loss, s.dz, s.ws, mask=s.mask)
        return {"idx": s.idx, "val": s.val, "prob": s.prob, "loss": s.loss, "dlogits": s.dz}
    if s.kind == "gtc":
        if s.noalloc:
            am.grad_threshold_encode_noalloc(s.grad, s.residual, 1e-4, s.words, s.count)
        else:
            am.grad_threshold_encode(s.grad, s.residual, 1e-4, s.words, s.count, s.ws)
        am.grad_threshold_decode(s.words, s.count, 1e-4, s.dense)
        return {"words": s.words, "count": s.count, "residual": s.residual, "update": s.dense}
    if s.kind == "workers":
        am.grad_threshold_decode_multi(s.words, s.counts, 1e-4, s.dense, s.ws)
        am.sgd_apply(s.master, s.dense, LR, s.weights)
        return {"update": s.dense, "master": s.master, "weights": s.weights}
    if s.kind == "bmuf":
        eta, eta_next, zeta = _bmuf_rates(s.models.shape[0])
        am.bmuf_block_update(s.models, s.models.shape[0], s.wg, s.delta, eta, eta_next, zeta,
                             s.local, s.local16)
        return {"model": s.wg, "delta": s.delta, "local": s.local, "local16": s.local16}
    am.lfr_features(s.raw_lengths, s.raw, s.mean, s.std, s.x)
    am.delay_targets(s.T, s.B, s.idx, s.prob, s.idx_out, s.prob_out, s.mask, 3, lengths=s.lengths)
    return {"x": s.x, "idx": s.idx_out, "prob": s.prob_out, "mask": s.mask}


# ------------------------------------------------------------------- work --

def _num_frames(case):
    return float(_frames(case, _lengths(case) if case.get("len_lo") else None))


def _layer_weights(case, k=1):
    """Weights per frame of k directions (k = 2: the teacher) and the senone layer."""
    H, D = case["hidden"], case["input_dim"]
    first = k * 4 * H * (D + H)
    return first + (case["layers"] - 1) * k * 4 * H * (k * H + H) + case["classes"] * k * H


def work(case):
    kind = case["kind"]
    if kind in ("train", "score", "teacher"):
        k = 2 if kind == "teacher" else 1
        e = 2 if case.get("dtype", "bf16") == "bf16" else 4
        N, W = _num_frames(case), _layer_weights(case, k)
        flops = 2.0 * N * W
        b = N * (case["input_dim"] * e + case["classes"] * 4) + W * e
        if kind == "train":
            flops = 3.0 * flops - 2.0 * N * 4 * case["hidden"] * case["input_dim"]
            # targets; gradient written, master (and residual) read and written, bf16 copy written
            b += N * case["K"] * 8 + W * (4 + 8 + (8 if case["gtc"] else 0) + (2 if e == 2 else 0))
        if kind == "score":
            b += 16.0 * case["layers"] * case["B"] * case["hidden"]
        return {"bytes": b, "flops": flops}
    if kind == "targets":
        e = 2 if case["dtype"] == "bf16" else 4
        return {"bytes": case["N"] * (case["classes"] * (8.0 + e) + case["K"] * 12.0),
                "flops": 6.0 * case["N"] * case["classes"]}
    n = case.get("n", 0)
    if kind == "gtc":
        return {"bytes": n * (12.0 + 4.0 + 4.0 * min(1.0, 0.8 * case["ratio"])), "flops": 3.0 * n}
    if kind == "workers":
        return {"bytes": n * (4.0 + 8.0 + 2.0 + 4.0 * case["rate"] * case["streams"]), "flops": 3.0 * n}
    if kind == "bmuf":
        return {"bytes": n * (4.0 * case["count"] + 16.0 + 6.0), "flops": n * (case["count"] + 7.0)}
    N, D = _num_frames(case), 3 * case["raw_dim"]
    e = 2 if case["dtype"] == "bf16" else 4
    return {"bytes": N * (D * (4.0 + e) + case["K"] * 16.0 + 1), "flops": 5.0 * N * D}


def tolerance(case):
    kind = case["kind"]
    if kind in ("train", "score", "teacher"):
        if case.get("dtype") == "f32":
            # sums in another order differ by 1e-8 to 2e-7; a compressed update
            # that falls the other way moves one weight by lr tau
            return {"rel": 2e-6, "max": 1e-3}
        # a whole model: a bf16 rounding that falls the other way travels
        # through the layers above and the steps after it.  The library's
        # three recurrence paths differ by up to 8e-4 (8e-3 an element).
        return {"rel": 4e-3, "max": 4e-2}
    if kind == "targets":  # bf16 rows: a last-bit difference that moves a rounding
        return {"rel": 5e-4, "max": 2e-2} if case["dtype"] == "bf16" else {"rel": 2e-6, "max": 1e-4}
    return "exact"  # the quantiser, SGD, BMUF and the input frames are defined bit for bit


# ------------------------------------------------------------------ exact --

def _schedule(T, B, lengths):
    lens = [T] * B if lengths is None else list(lengths)
    counts, nb = [], B
    for t in range(T):
        while nb > 0 and lens[nb - 1] <= t:
            nb -= 1
        counts.append(nb)
    offs = [0]
    for c in counts:
        offs.append(offs[-1] + c)
    return lens, counts, offs


def _lstm(x, Wx, Wh, b, counts, offs, h0=None, c0=None):
    """One layer over packed rows, fp64.  Returns the gates [N][4H] (i, f, g,
    o), c and h [N][H], and the shifted h and c (h_{t-1}, c_{t-1} per row)."""
    H = Wh.shape[1]
    A = x @ Wx.t() + b
    N = x.shape[0]
    C, Hh, Hs, Cs = (torch.zeros((N, H), dtype=torch.float64, device=DEV) for _ in range(4))
    h = torch.zeros((counts[0] if counts else 0, H), dtype=torch.float64, device=DEV) if h0 is None else h0
    c = torch.zeros_like(h) if c0 is None else c0
    WhT = Wh.t().contiguous()
    for t, nb in enumerate(counts):
        if nb == 0:
            break
        o = offs[t]
        h, c = h[:nb], c[:nb]
        Hs[o:o + nb], Cs[o:o + nb] = h, c
        a = A[o:o + nb]
        a += h @ WhT
        a[:, :2 * H].sigmoid_()
        a[:, 2 * H:3 * H].tanh_()
        a[:, 3 * H:].sigmoid_()
        c = a[:, H:2 * H] * c + a[:, :H] * a[:, 2 * H:3 * H]
        h = a[:, 3 * H:] * torch.tanh(c)
        C[o:o + nb], Hh[o:o + nb] = c, h
    return A, C, Hh, Hs, Cs


def _lstm_backward(dH, A, C, Cs, Wh, counts, offs):
    """dA [N][4H] of one layer; dH [N][H] the gradient from above, fp64."""
    H = Wh.shape[1]
    dA = torch.empty_like(A)
    T = len(counts)
    dc = da_next = None
    nn = 0
    for t in range(T - 1, -1, -1):
        nb, o = counts[t], offs[t]
        if nb == 0:
            continue
        i, f, g, ou = (A[o:o + nb, q * H:(q + 1) * H] for q in range(4))
        dh = dH[o:o + nb].clone()
        if nn:
            dh[:nn] += da_next @ Wh
        tc = torch.tanh(C[o:o + nb])
        d = dh * ou * (1.0 - tc * tc)
        if nn:
            d[:nn] += dc
        a = dA[o:o + nb]
        a[:, :H] = d * g * i * (1.0 - i)
        a[:, H:2 * H] = d * Cs[o:o + nb] * f * (1.0 - f)
        a[:, 2 * H:3 * H] = d * i * (1.0 - g * g)
        a[:, 3 * H:] = dh * tc * ou * (1.0 - ou)
        dc, da_next, nn = d * f, a, nb
    return dA


def _soft_ce(z, idx, prob, mask):
    """loss and dlogits, mean over the valid rows, fp64."""
    N = z.shape[0]
    m = torch.ones(N, dtype=torch.float64, device=DEV) if mask is None else mask.double()
    s = m / m.sum().clamp_min(1.0)
    p = prob.double()
    lse = torch.logsumexp(z, dim=1)
    zi = torch.gather(z, 1, idx.long())
    loss = (s * -(p * (zi - lse[:, None])).sum(1)).sum()
    d = torch.exp(z - lse[:, None]) * p.sum(1, keepdim=True)
    d.scatter_add_(1, idx.long(), -p)
    return loss.view(1), d * s[:, None]


def _exact_train(case, seed):
    lengths, master, x, idx, prob = _train_inputs(case, seed)
    if case["dtype"] == "bf16":
        W, x = master.bfloat16().double(), x.bfloat16().double()
    else:
        W, x = master.double(), x.double()
    L, D0, H, C = case["layers"], case["input_dim"], case["hidden"], case["classes"]
    G = 4 * H
    _, counts, offs = _schedule(case["T"], case["B"], lengths)
    off = am.param_offsets(_model(case, case["dtype"]))
    par = []
    for l in range(L):
        D = D0 if l == 0 else H
        wx, wh, b = off[3 * l:3 * l + 3]
        par.append((W[wx:wx + G * D].view(G, D), W[wh:wh + G * H].view(G, H), W[b:b + G]))
    Wo, bo = W[off[3 * L]:off[3 * L] + C * H].view(C, H), W[off[3 * L + 1]:off[3 * L + 1] + C]
    kept, X = [], x
    for l in range(L):
        r = _lstm(X, *par[l], counts, offs)
        kept.append((X, *r))
        X = r[2]
    logits = X @ Wo.t() + bo
    loss, dz = _soft_ce(logits, idx, prob, None)
    grads = torch.empty_like(W)
    grads[off[3 * L]:off[3 * L] + C * H] = (dz.t() @ X).view(-1)
    grads[off[3 * L + 1]:off[3 * L + 1] + C] = dz.sum(0)
    dH = dz @ Wo
    del dz
    for l in range(L - 1, -1, -1):
        X, A, Cc, _, Hs, Cs = kept.pop()
        dA = _lstm_backward(dH, A, Cc, Cs, par[l][1], counts, offs)
        wx, wh, b = off[3 * l:3 * l + 3]
        grads[wx:wx + G * X.shape[1]] = (dA.t() @ X).view(-1)
        grads[wh:wh + G * H] = (dA.t() @ Hs).view(-1)
        grads[b:b + G] = dA.sum(0)
        if l > 0:
            dH = dA @ par[l][0]
    if case["gtc"]:
        u = torch.where(grads.abs() > case["tau"], grads.sign() * case["tau"], torch.zeros_like(grads))
    else:
        u = grads
    return {"loss": loss, "logits": logits, "grads": grads, "master": master.double() - LR * u}


def _exact_score(case, seed):
    params, x, h0, c0 = _score_inputs(case, seed)
    W, X = params.double(), x.double()
    L, H, C, G = case["layers"], case["hidden"], case["classes"], 4 * case["hidden"]
    _, counts, offs = _schedule(case["T"], case["B"], None)
    off = am.param_offsets(_model(case, "bf16"))
    hT, cT = [], []
    for l in range(L):
        D = X.shape[1]
        wx, wh, b = off[3 * l:3 * l + 3]
        _, Cc, X, _, _ = _lstm(X, W[wx:wx + G * D].view(G, D), W[wh:wh + G * H].view(G, H),
                               W[b:b + G], counts, offs, h0[l].double(), c0[l].double())
        hT.append(X[-case["B"]:])
        cT.append(Cc[-case["B"]:])
    logits = X @ W[off[3 * L]:off[3 * L] + C * H].view(C, H).t() + W[off[3 * L + 1]:off[3 * L + 1] + C]
    return {"logits": logits, "hT": torch.stack(hT), "cT": torch.stack(cT)}


def _exact_teacher(case, seed):
    lengths, params, x = _teacher_inputs(case, seed)
    W, X = params.double(), x.double()
    L, H, C, G = case["layers"], case["hidden"], case["classes"], 4 * case["hidden"]
    lens, counts, offs = _schedule(case["T"], case["B"], lengths)
    off = am.teacher_param_offsets(_model(case, "bf16"))
    rev = torch.empty(X.shape[0], dtype=torch.int64)  # row of the mirrored frame
    for t, nb in enumerate(counts):
        for b in range(nb):
            rev[offs[t] + b] = offs[lens[b] - 1 - t] + b
    rev = rev.to(DEV)
    for l in range(L):
        D, out = X.shape[1], []
        for d in range(2):
            wx, wh, b = off[6 * l + 3 * d:6 * l + 3 * d + 3]
            h = _lstm(X[rev] if d else X, W[wx:wx + G * D].view(G, D), W[wh:wh + G * H].view(G, H),
                      W[b:b + G], counts, offs)[2]
            out.append(h[rev] if d else h)
        X = torch.cat(out, 1)
    wo, bo = off[6 * L], off[6 * L + 1]
    return X @ W[wo:wo + C * 2 * H].view(C, 2 * H).t() + W[bo:bo + C]


def _exact_targets(case, seed):
    zt, zs, mask = _target_inputs(case, seed)
    val, idx = torch.sort(zt, dim=1, descending=True, stable=True)  # ties: the lower index first
    val, idx = val[:, :case["K"]].double(), idx[:, :case["K"]]
    prob = torch.softmax(val, dim=1)
    loss, dz = _soft_ce(zs.double(), idx, prob, mask)
    return {"idx": None, "val": val, "prob": prob, "loss": loss, "dlogits": dz}


def _exact_workers(case, seed):
    words, counts, master = _worker_inputs(case, seed)
    k = torch.zeros(case["n"], dtype=torch.float64, device=DEV)
    for s in range(case["streams"]):
        w = words[s, :int(counts[s])].long()
        k.index_add_(0, w >> 1, (1 - 2 * (w & 1)).double())
    u = float(np.float32(1e-4)) * k
    m = master.double() - float(np.float32(LR)) * u
    return {"update": u, "master": m, "weights": m}


def _exact_bmuf(case, seed):
    models, wg, delta = _bmuf_inputs(case, seed)
    eta, eta_next, zeta = (float(np.float32(v)) for v in _bmuf_rates(case["count"]))
    bar = torch.zeros(case["n"], dtype=torch.float64, device=DEV)
    for i in range(case["count"]):
        bar += models[i]
    d = eta * delta.double() + zeta * (bar / case["count"] - wg.double())
    w = wg.double() + d + eta_next * d
    return {"model": w, "delta": d, "local": w, "local16": w}


def _exact_inputs(case, seed):
    lengths, raw_lengths, raw, mean, std, _, _ = _raw_inputs(case, seed)
    _, counts, offs = _schedule(max(lengths), case["B"], lengths)
    out = torch.empty((sum(lengths), mean.numel()), dtype=torch.float64, device=DEV)
    at = torch.tensor(offs[:-1], device=DEV)
    pos = 0
    for b, T in enumerate(lengths):
        y = raw[pos:pos + 3 * T].double().view(T, -1)
        pos += raw_lengths[b]
        z = y - torch.cumsum(y, 0) / torch.arange(1, T + 1, device=DEV, dtype=torch.float64)[:, None]
        out[at[:T] + b] = (z - mean.double()) / std.double()
    return {"x": out, "idx": None, "prob": None, "mask": None}


def exact(case, seed):
    f = {"train": _exact_train, "score": _exact_score, "teacher": _exact_teacher,
         "targets": _exact_targets, "workers": _exact_workers, "bmuf": _exact_bmuf,
         "inputs": _exact_inputs}.get(case["kind"])
    if f is None:  # (gtc: words, and single fp32 adds)
        return None
    with torch.no_grad():
        return f(case, seed)
