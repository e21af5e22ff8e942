"""Performance cases of the vocabulary head + Pruned CTC loss.

A case is one call (or one short chain of calls) that a training or decoding program makes:

  kind "loss"     pruned_ctc_fwd_bwd: loss, per-utterance losses and the head's gradients (a
                  training step's head; "frozen" leaves the head weight's gradient out);
  kind "greedy"   greedy_decode: framewise argmax over the vocabulary and the collapsed tokens;
  kind "grouped"  grouped_head and its autograd backward: the export for a stock CTC loss;
  kind "sweep"    beam_sweep: the discarded posterior mass of every utterance at every beam.

Sizes are those of the named workloads, the tests and the benchmark: D = 64 .. 5120,
V = 500 .. 180,000 classes, 1 to 160 utterances of 20 to 1500 frames, bf16 and fp32 heads.
Frame counts depend on the case alone, values on the seed.  Inputs are drawn on the device:
H ~ N(0, 1) (rows of unit RMS for the language-model heads), W ~ N(0, 1/D) (N(0, 0.02^2) for
the language-model heads), Zipf(1.1) targets; "peak" adds that many nats to the logit of one
class per frame along an alignment of the target, as a trained head's posteriors have it.
"""
import math

import numpy as np
import torch

from paper_2609_33645_amd import beam_sweep as bs
from paper_2609_33645_amd import prunedctc as pc

INF = -1.0  # "beam": keep every alignment
BEAMS = (8.0, 10.0, 16.0, 25.0, 32.0, 50.0, 64.0, 75.0, 100.0)
SLACK = 1e-3  # the library keeps arcs up to this many nats beyond the beam


def _case(kind, dtype, D, V, N, t_min, t_max, u_frac, **more):
    c = {"kind": kind, "dtype": dtype, "D": D, "V": V, "N": N, "t_min": t_min, "t_max": t_max, "u_frac": u_frac,
         "beam": INF, "blank": 0, "bias": False, "weights": False, "frozen": False, "llm": False, "repeat": 0.0,
         "peak": 0.0}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: a unit-test sized fp32 head, where launches and host work count
        _case("loss", "f32", 64, 1000, 2, 42, 50, 0.2, name="tiny_f32"),
        # an ordinary subword vocabulary on the encoder benchmark's batch, fp32 head, head bias
        _case("loss", "f32", 512, 5000, 160, 100, 100, 1 / 6, beam=100.0, bias=True, name="encoder_f32_v5k"),
        # the encoder benchmark's memory shape: 160 x 100 frames, 180,000 classes, fp32 head
        _case("loss", "f32", 512, 180_000, 160, 100, 100, 1 / 6, name="encoder_f32_v180k"),
        # one utterance (batch of one: evaluation, adaptation to a speaker)
        _case("loss", "bf16", 512, 180_000, 1, 331, 331, 1 / 6, beam=16.0, peak=8.0, name="one_utterance"),
        # the benchmark's training step
        _case("loss", "bf16", 512, 180_000, 16, 150, 375, 1 / 6, beam=16.0, name="zipformer_m"),
        # the same step for a linear layer with bias, losses normalised per token, no pruning
        _case("loss", "bf16", 512, 180_000, 16, 150, 375, 1 / 6, bias=True, weights=True, name="zipformer_m_bias"),
        # long utterances on the widest language-model head: the lattice is long
        _case("loss", "bf16", 5120, 151_936, 2, 1500, 1500, 4 / 15, beam=16.0, llm=True, repeat=0.1,
              name="qwen3_32b"),
        # the language-model benchmark's memory shape, head frozen (no weight gradient)
        _case("loss", "bf16", 4096, 151_936, 107, 106, 108, 0.25, beam=32.0, llm=True, frozen=True,
              name="qwen3_8b_frozen"),
        # decoding one utterance as it arrives, and a whole batch
        _case("greedy", "bf16", 512, 180_000, 1, 150, 150, 1 / 6, peak=14.0, name="greedy_one"),
        _case("greedy", "bf16", 512, 180_000, 16, 150, 375, 1 / 6, bias=True, peak=14.0, name="greedy_batch"),
        # the export to a stock CTC loss, forward and backward through autograd
        _case("grouped", "bf16", 1024, 151_936, 8, 200, 500, 0.25, bias=True, llm=True, name="grouped"),
        # choosing a beam: the discarded mass at nine beams
        _case("sweep", "bf16", 512, 180_000, 16, 150, 375, 1 / 6, name="beam_sweep"),
    ]


def draw(rng):
    def spread(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    while True:
        kind = rng.choices(["loss", "greedy", "grouped", "sweep"], [6, 2, 1, 1])[0]
        dtype = "f32" if rng.random() < 0.3 else "bf16"
        # widths of real heads are mostly multiples of 64; some are odd multiples of 8
        D = int(spread(64, 5120)) // (8 if rng.random() < 0.3 else 64) * (8 if rng.random() < 0.3 else 64)
        D = min(max(D, 64), 5120)
        V = int(spread(500, 180_001))
        N = int(round(spread(1, 160)))
        t = spread(20, 1500)
        t_min, t_max = int(max(4, t * rng.uniform(0.5, 1.0))), int(t)
        t_min = min(t_min, t_max)
        c = _case(kind, dtype, D, V, N, t_min, t_max, rng.choice([0.1, 1 / 6, 0.25, 0.4]),
                  beam=rng.choice([INF, 16.0, 32.0, 100.0]), blank=rng.choice([0, 0, V - 1]),
                  bias=kind != "sweep" and rng.random() < 0.4, weights=kind == "loss" and rng.random() < 0.3,
                  frozen=kind == "loss" and rng.random() < 0.25, llm=D >= 1024, repeat=rng.choice([0.0, 0.1]),
                  peak=14.0 if kind == "greedy" else rng.choice([0.0, 0.0, 8.0]))
        M = int(_lengths(c)[0].sum())
        # no more work than the largest listed cases: 16,000 frames, and by type the products of
        # the fp32 encoder head and of the widest bf16 head
        if 20 <= M <= 16_000 and M * V * D <= (1.4e12 if dtype == "f32" else 2.3e12):
            return c


# ---- inputs --------------------------------------------------------------------------------

def _lengths(c):
    r = np.random.default_rng([c["N"], c["t_min"], c["t_max"]])
    T = r.integers(c["t_min"], c["t_max"] + 1, size=c["N"]).astype(np.int32)
    return T, np.floor(T * c["u_frac"] + 1e-9).astype(np.int32)


def _inputs(c, seed):
    r = np.random.default_rng(seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    D, V, blank = c["D"], c["V"], c["blank"]
    T, U = _lengths(c)
    M = int(T.sum())
    cdf = np.cumsum(np.arange(1, V, dtype=np.float64) ** -1.1)
    ids = np.searchsorted(cdf, r.random(int(U.sum())) * cdf[-1], side="right")
    ids = np.minimum(ids, V - 2) + 1  # ranks 1 .. V - 1
    ids = np.where(ids == blank, 0, ids).astype(np.int32)
    first = np.zeros(ids.size, bool)
    off = np.concatenate([[0], np.cumsum(U)])
    first[off[:-1][U > 0]] = True
    for i in np.flatnonzero((r.random(ids.size) < c["repeat"]) & ~first):
        ids[i] = ids[i - 1]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    H = torch.randn(M, D, generator=g, device="cuda")
    if c["llm"]:
        H /= H.square().mean(1, keepdim=True).sqrt()
    std = 0.02 if c["llm"] else 1.0 / math.sqrt(D)
    W = torch.randn(V, D, generator=g, device="cuda").mul_(std).to(dt)
    if c["peak"]:
        path = np.full(M, blank, np.int64)
        t0 = 0
        for n in range(c["N"]):
            at = np.sort(r.choice(int(T[n]), size=int(U[n]), replace=False))
            path[t0 + at] = ids[off[n]:off[n + 1]]
            t0 += int(T[n])
        H += W[torch.from_numpy(path).cuda()].float() * (c["peak"] / (D * std * std))
    x = {"H": H.to(dt), "W": W, "y": torch.from_numpy(ids).cuda(), "T": T, "U": U, "bias": None, "weight": None}
    if c["bias"]:
        x["bias"] = torch.randn(V, generator=g, device="cuda") * 0.5
        x["bias"][blank] += 2.0
    if c["weights"]:
        x["weight"] = torch.from_numpy((1.0 / np.maximum(U, 1)).astype(np.float32)).cuda()
    if c["kind"] == "grouped":
        # the blank and the batch's distinct labels; their number is the case's, as its frames are
        # (about six in ten targets are new: the commonest of the others make up the number)
        k = min(int(0.6 * ids.size) + 1, V - 1)
        seen = np.unique(ids, return_index=True)
        seen = seen[0][np.argsort(seen[1])][:k]
        rest = np.setdiff1d(np.arange(min(V, 2 * k + 2)), np.append(seen, blank))
        u = np.sort(np.concatenate([seen, rest[:k - seen.size]]))
        x["u"] = torch.from_numpy(np.concatenate([[blank], u]).astype(np.int32)).cuda()
        # minus the occupancies of the selected classes, a few per frame, as a CTC loss returns them
        occ = torch.softmax(3.0 * torch.randn(M, x["u"].numel(), generator=g, device="cuda"), 1)
        x["dlogp"] = torch.cat([-occ, torch.zeros(M, 1, device="cuda")], 1)
    return x


def _beam(c):
    return math.inf if c["beam"] < 0 else c["beam"]


def prepare(case, seed):
    c = dict(case)
    x = _inputs(c, seed)
    if c["kind"] == "loss":  # a training program keeps its workspace and gradient buffers
        M, D = x["H"].shape
        code = pc.PCTC_BF16 if c["dtype"] == "bf16" else pc.PCTC_F32
        n = pc.workspace_size(code, x["T"], x["U"], D, c["V"], _beam(c), want_dW=not c["frozen"])
        x["ws"] = torch.empty(n + 256, dtype=torch.uint8, device="cuda")
        x["ws"] = x["ws"][(-x["ws"].data_ptr()) % 256:][:n]
        x["dH"] = torch.empty(M, D, device="cuda")
        x["dW"] = None if c["frozen"] else torch.empty(c["V"], D, device="cuda")
    elif c["kind"] == "grouped":
        x["leaves"] = [t.requires_grad_() for t in (x["H"], x["W"], x["bias"]) if t is not None]
    x["case"] = c
    return x


# ---- one pass ------------------------------------------------------------------------------

def run(s):
    c = s["case"]
    if c["kind"] == "loss":
        o = pc.pruned_ctc_fwd_bwd(s["H"], s["W"], s["y"], s["T"], s["U"], blank=c["blank"], beam=_beam(c),
                                  want_dW=not c["frozen"], workspace=s["ws"], dH_out=s["dH"], dW_out=s["dW"],
                                  bias=s["bias"], utt_weight=s["weight"], want_db=c["bias"] and not c["frozen"])
        return {k: o[k] for k in ("loss", "loss_per_utt", "status", "dH", "dW", "db")}
    if c["kind"] == "greedy":
        o = pc.greedy_decode(s["H"], s["W"], s["T"], blank=c["blank"], bias=s["bias"])
        tokens = np.full((c["N"], c["t_max"]), -1, np.int32)  # the batch of hypotheses, padded
        for n, seq in enumerate(o["tokens"]):
            tokens[n, :len(seq)] = seq
        return {"ids": o["ids"], "token_lengths": o["token_lengths"], "tokens": tokens}
    if c["kind"] == "grouped":
        logp = pc.grouped_head(s["H"], s["W"], s["u"], s["bias"])
        return {"logp": logp.detach(), "grads": list(torch.autograd.grad(logp, s["leaves"], s["dlogp"]))}
    return {"delta": bs.beam_sweep(s["H"], s["W"], s["y"], s["T"], s["U"], c["blank"], BEAMS)["delta"]}


# ---- what a pass cannot do without, and how exact it is ------------------------------------------

def work(case):
    c = case
    T, U = _lengths(c)
    M, Y, D, V, e = int(T.sum()), int(U.sum()), c["D"], c["V"], 2 if c["dtype"] == "bf16" else 4
    inputs = (M + V) * D * e + 4 * Y + (4 * V if c["bias"] else 0)
    if c["kind"] == "loss":
        both = not c["frozen"]
        return {"bytes": inputs + 4 * M * D + (4 * V * D if both else 0) + (4 * V if both and c["bias"] else 0),
                "flops": (6.0 if both else 4.0) * M * V * D}
    if c["kind"] == "greedy":
        return {"bytes": inputs + 8 * M, "flops": 2.0 * M * V * D}
    if c["kind"] == "grouped":
        k = min(int(0.6 * Y) + 1, V - 1) + 1
        return {"bytes": inputs + (M + V) * D * e + (4 * V if c["bias"] else 0) + 8 * M * (k + 1),
                "flops": 6.0 * M * V * D}
    return {"bytes": inputs + 8 * len(BEAMS) * c["N"], "flops": 2.0 * M * V * D}


def tolerance(case):
    c = case
    if c["kind"] == "greedy":  # the products' sums may break a near tie the other way
        return {"rel": 0.0, "differ": 0.01}
    if c["kind"] == "sweep":  # alignments at the beam's edge, decided in 32 bits
        return {"rel": 1e-3}
    if c["dtype"] == "bf16":  # gradients from probabilities rounded to bf16 once
        return {"rel": 8e-3, "max": 0.2}
    return {"rel": 1e-5, "max": 1e-3}


# ---- the same in 64 bits ---------------------------------------------------------------------------

def _shift(x, k, fill):
    """Column s of the result is column s - k of x (k > 0) or s + |k| (k < 0)."""
    y = torch.full_like(x, fill)
    if abs(k) < x.shape[-1]:
        if k > 0:
            y[..., k:] = x[..., :-k]
        else:
            y[..., :k] = x[..., -k:]
    return y


class _Lattice:
    """CTC trellis of a padded batch in float64: E [N, T, S] log-probabilities of the extended
    label states (blank, y1, blank, ..), -inf outside."""

    def __init__(self, S, y, T, U):  # S [M, K] log-probabilities, y: columns of the targets, 0 the blank
        N, Tm, Sm = len(T), int(T.max()), 2 * int(U.max()) + 1
        ext = np.zeros((N, Sm), np.int64)
        rows = np.zeros((N, Tm), np.int64)
        valid = np.zeros((N, Sm), bool)
        o = t0 = 0
        for n in range(N):
            ext[n, 1:2 * U[n] + 1:2] = y[o:o + U[n]]
            valid[n, :2 * U[n] + 1] = True
            rows[n, :T[n]] = t0 + np.arange(T[n])
            o += int(U[n])
            t0 += int(T[n])
        dev = S.device
        self.N, self.Tm, self.Sm = N, Tm, Sm
        self.ext, self.rows = torch.from_numpy(ext).to(dev), torch.from_numpy(rows).to(dev)
        self.T = torch.from_numpy(T.astype(np.int64)).to(dev)
        self.valid = torch.from_numpy(valid).to(dev)
        sp = torch.from_numpy(2 * U.astype(np.int64) + 1).to(dev)[:, None]
        s = torch.arange(Sm, device=dev)[None]
        self.skip = self.valid & (s % 2 == 1) & (s >= 3) & (self.ext != _shift(self.ext, 2, -1))
        self.start = self.valid & (s < 2)
        self.final = self.valid & (s >= sp - 2)
        self.live = torch.arange(Tm, device=dev)[None] < self.T[:, None]
        E = S[self.rows[:, :, None], self.ext[:, None, :]]
        self.E = torch.where(self.valid[:, None, :] & self.live[:, :, None], E, -math.inf)

    @staticmethod
    def join(a, viterbi):
        a = torch.stack(a)
        if viterbi:
            return a.amax(0)
        return torch.logsumexp(a, 0)

    def passes(self, viterbi, keep=None):
        """alpha, beta [N, T, S] and the total [N]; keep: arc masks (stay, step, skip, start, final)."""
        no = -math.inf
        k0, k1, k2, ks, kf = keep if keep else (None, None, None, self.start, self.final)
        on = lambda x, m: x if m is None else torch.where(m, x, no)  # noqa: E731
        a = torch.full_like(self.E, no)
        b = torch.full_like(self.E, no)
        a[:, 0] = torch.where(ks, self.E[:, 0], no)
        for t in range(1, self.Tm):
            p = a[:, t - 1]
            m = (lambda k: None if k is None else k[:, t])  # noqa: E731
            a[:, t] = self.E[:, t] + self.join([on(p, m(k0)), on(_shift(p, 1, no), m(k1)),
                                                torch.where(self.skip, on(_shift(p, 2, no), m(k2)), no)], viterbi)
        end = torch.where(kf, 0.0, no).to(self.E)
        for t in range(self.Tm - 1, -1, -1):
            if t + 1 < self.Tm:
                q = self.E[:, t + 1] + b[:, t + 1]
                m = (lambda k: None if k is None else k[:, t + 1])  # noqa: E731
                r = self.join([on(q, m(k0)), _shift(on(q, m(k1)), -1, no),
                               _shift(torch.where(self.skip, on(q, m(k2)), no), -2, no)], viterbi)
                b[:, t] = torch.where((self.T == t + 1)[:, None], end, r)
            else:
                b[:, t] = torch.where((self.T == t + 1)[:, None], end, no)
        last = a[torch.arange(self.N, device=a.device), self.T - 1] + end
        return a, b, self.join(list(last.unbind(1)), viterbi)

    def arcs(self, beam):
        """Arcs whose best alignment scores within the beam of the best one."""
        a, b, best = self.passes(True)
        thr = (best - beam - SLACK)[:, None, None]
        into = self.E + b
        p = torch.cat([torch.full_like(a[:, :1], -math.inf), a[:, :-1]], 1)
        end = a[torch.arange(self.N, device=a.device), self.T - 1]
        return ((p + into >= thr), (_shift(p, 1, -math.inf) + into >= thr), (_shift(p, 2, -math.inf) + into >= thr),
                self.start & (into[:, 0] >= thr[:, 0]), self.final & (end >= thr[:, 0]))


def _blocks(M, V):
    step = max(64, int(2.0e8 // V))
    return [slice(i, min(M, i + step)) for i in range(0, M, step)]


def _union(c, x):
    ids = x["y"].cpu().numpy().astype(np.int64)
    u = np.concatenate([[c["blank"]], np.unique(ids)])
    return torch.from_numpy(u).cuda(), 1 + np.searchsorted(u[1:], ids)


def _selected(c, H, W, bias, u):
    """Log-normaliser, selected log-probabilities and the log-probability of all the others (the
    M x V logits by blocks of frames)."""
    M = H.shape[0]
    lam = torch.empty(M, dtype=torch.float64, device="cuda")
    other = torch.empty(M, dtype=torch.float64, device="cuda")
    S = torch.empty(M, u.numel(), dtype=torch.float64, device="cuda")
    for b in _blocks(M, c["V"]):
        Z = H[b] @ W.T
        if bias is not None:
            Z += bias
        lam[b] = torch.logsumexp(Z, 1)
        S[b] = Z[:, u] - lam[b, None]
        Z[:, u] = -math.inf
        other[b] = torch.logsumexp(Z, 1) - lam[b]
    return lam, S, other


def _head_grads(c, H, W, bias, u, lam, G, g, want_dW):
    """dZ = scatter_u(G) - g p, then dH, dW, db."""
    dH = torch.empty_like(H)
    dW = torch.zeros_like(W) if want_dW else None
    db = torch.zeros(c["V"], dtype=torch.float64, device="cuda")
    for b in _blocks(H.shape[0], c["V"]):
        Z = H[b] @ W.T
        if bias is not None:
            Z += bias
        dZ = Z.sub_(lam[b, None]).exp_().mul_(-g[b, None])
        dZ[:, u] += G[b]
        dH[b] = dZ @ W
        if want_dW:
            dW += dZ.T @ H[b]
        db += dZ.sum(0)
    return dH, dW, db


def exact(case, seed):
    c = dict(case)
    x = _inputs(c, seed)
    with torch.no_grad():
        H, W = x["H"].double(), x["W"].double()
        bias = None if x["bias"] is None else x["bias"].double()
        if c["kind"] == "greedy":
            return None  # whole numbers
        if c["kind"] == "grouped":
            u = x["u"].long()
            lam, S, other = _selected(c, H, W, bias, u)
            logp = torch.cat([S, other[:, None]], 1)
            d = x["dlogp"].double()
            sig, cc = d.sum(1), torch.where(other > -math.inf, d[:, -1] / other.exp(), 0.0)
            G = d[:, :-1] - cc[:, None] * S.exp()
            grads = _head_grads(c, H, W, bias, u, lam, G, sig - cc, True)
            return {"logp": logp, "grads": list(grads[:2 if bias is None else 3])}
        u, y = _union(c, x)
        lam, S, _ = _selected(c, H, W, bias, u)
        lat = _Lattice(S, y, x["T"], x["U"])
        if c["kind"] == "sweep":
            full = lat.passes(False)[2]
            return {"delta": torch.stack([-torch.expm1(lat.passes(False, lat.arcs(b))[2] - full) for b in BEAMS])}
        a, b, total = lat.passes(False, lat.arcs(_beam(c)) if c["beam"] >= 0 else None)
        w = torch.ones(c["N"], dtype=torch.float64, device="cuda") if x["weight"] is None else x["weight"].double()
        fine = torch.isfinite(total)
        gam = torch.where((fine[:, None] & lat.live)[:, :, None], (a + b - total[:, None, None]).exp(), 0.0)
        gam = torch.where(torch.isfinite(gam), gam, 0.0) * w[:, None, None]
        G = torch.zeros_like(S).reshape(-1)
        at = lat.rows[:, :, None] * S.shape[1] + lat.ext[:, None, :]
        G.index_add_(0, at.reshape(-1), -gam.reshape(-1))
        G = G.reshape(S.shape)
        dH, dW, db = _head_grads(c, H, W, bias, u, lam, G, G.sum(1), not c["frozen"])
        loss = torch.where(fine, -total, 0.0)
        return {"loss": (w * loss).sum().reshape(1), "loss_per_utt": loss, "status": None, "dH": dH, "dW": dW,
                "db": db if c["bias"] and not c["frozen"] else None}
