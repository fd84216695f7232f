"""What a user of this library has it do, as cases to be timed.

Three kinds of work, each through the public entry points of ``paper_2603_12617_amd.binding``:

* ``learn``   -- the online-ensemble learner: reset, ``calls`` calls of ``oco_run_rounds`` that
  together cover the horizon T, then the iterates, the Hedge weights, the combined iterate
  (``oco_get_state``) and the regret.  A long simulation is one call (that is how the benchmark
  and the examples run it); a serving loop makes many short ones.
* ``verify``  -- accepted length and next token of a batch of speculative-decoding steps.
* ``accept``  -- the acceptance rate of every draft position of such a batch.

Sizes are those of the benchmark configurations (workloads.py), of the tests, or generic.
"""
import math

import numpy as np
import torch

from paper_2603_12617_amd import binding as B

DEVICE = "cuda:0"


def _learn(name, **kw):
    case = dict(name=name, kind="learn", d=100, K=8, T=1000, R=16, loss="squared", shared=True, nnz=0, seg_len=0,
                optimistic=0, calls=1, host_regret=True, norm=0.5)
    case.update(kw)
    return case


def listed():
    return [
        # a serving loop: a draft's learner is updated after every few verification steps, and the
        # weights and the combined model are read back on the device; many tiny calls
        _learn("serving_calls", d=1000, K=3, T=512, R=1, loss="logistic", shared=False, optimistic=1, calls=64,
               host_regret=False),
        # one learner with a linear loss, the smallest simulation of the benchmark
        _learn("one_learner", d=10, K=1, T=1000, R=1, loss="linear"),
        # independent runs, each with its own stream of rounds (benchmark configuration)
        _learn("per_run_streams", d=100, K=15, T=10000, R=64, shared=False),
        # the same with rows whose length is not a multiple of anything, the two-step update and a
        # logistic loss: what a user's own features look like
        _learn("per_run_ragged", d=777, K=5, T=3000, R=48, loss="logistic", shared=False, optimistic=1, seg_len=700),
        # a step-size sweep over a shared stream: a few hundred learners
        _learn("shared_sweep", d=2048, K=8, T=4000, R=32, loss="logistic", optimistic=2, norm=1.0),
        # few learners of a model too wide for the registers of a wavefront
        _learn("wide_model", d=32768, K=4, T=2000, R=4, norm=0.8),
        # changing environment, comparator redrawn every 1000 rounds (benchmark configuration)
        _learn("piecewise", d=1000, K=17, T=100000, R=256, seg_len=1000, norm=0.8),
        # the largest dense simulation (benchmark configuration)
        _learn("largest_dense", d=4096, K=16, T=20000, R=1024, loss="logistic", norm=1.0),
        # sparse rounds over a state that lives in HBM (benchmark configuration)
        _learn("sparse", d=1 << 20, K=8, T=100000, R=16, nnz=32),
        # the verification step: a small decoding batch, and a large one of a wide vocabulary
        dict(name="verify_few", kind="verify", B=8, k=4, V=32000, sharp=2.5, noise=0.6),
        dict(name="verify_many", kind="verify", B=256, k=4, V=151936, sharp=2.5, noise=0.6),
        # monitoring the draft: acceptance rates of a large batch
        dict(name="acceptance", kind="accept", B=1024, k=4, V=32000, sharp=2.5, noise=0.6),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# no drawn case costs more than the largest listed one: learner updates of a dense case, floats of
# its streams and outputs, entries of the distributions
_MAX_UNITS = 1.3e12
_MAX_FLOATS = 1 << 29


def draw(rng):
    """One more case of the listed ranges."""
    kind = rng.choice(["serving", "per_run", "shared", "shared", "wide", "sparse", "verify", "accept"])
    if kind in ("verify", "accept"):
        V = rng.choice([_log_int(rng, 1000, 200000), 4 * _log_int(rng, 250, 50000)])
        k = rng.randint(1, 8)
        return dict(kind=kind, B=_log_int(rng, 1, max(1, min(1024, 200000000 // (k * V)))), k=k, V=V,
                    sharp=rng.uniform(1.5, 3.5), noise=rng.uniform(0.2, 1.5))
    loss = rng.choice(["squared", "logistic", "squared", "logistic", "linear"])
    over = dict(loss=loss, optimistic=rng.choice([0, 0, 1, 2]), norm=rng.choice([0.5, 0.8, 1.0]))
    if kind == "serving":
        calls = _log_int(rng, 8, 128)
        over.update(d=_log_int(rng, 10, 4096), K=rng.randint(1, 8), R=_log_int(rng, 1, 16), calls=calls,
                    T=calls * _log_int(rng, 1, 64), shared=rng.random() < 0.5, host_regret=False)
    elif kind == "per_run":
        over.update(d=_log_int(rng, 10, 2048), K=rng.randint(1, 24), R=_log_int(rng, 1, 256), T=_log_int(rng, 600, 20000),
                    shared=False)
    elif kind == "shared":
        d = _log_int(rng, 10, 4096)
        over.update(d=d if rng.random() < 0.3 else max(4, d // 4 * 4), K=rng.randint(1, 24), R=_log_int(rng, 1, 1024),
                    T=_log_int(rng, 600, 50000))
    elif kind == "wide":
        over.update(d=4 * _log_int(rng, 1025, 16384), K=rng.randint(1, 16), R=_log_int(rng, 1, 64), T=_log_int(rng, 300, 8000))
    else:
        nnz = rng.choice([8, 16, 32, 64])
        over.update(d=_log_int(rng, 4096, 1 << 20), K=rng.randint(1, 16), R=_log_int(rng, 1, 64), T=_log_int(rng, 2000, 100000),
                    nnz=nnz, loss=rng.choice(["squared", "logistic"]))
    case = _learn("", **over)
    del case["name"]
    streams = (1 if case["shared"] else case["R"]) * (case["nnz"] * 2 if case["nnz"] else case["d"])
    per_round = max(1.0, streams + case["R"] * (case["K"] + 2))
    case["T"] = min(case["T"], int(_MAX_FLOATS / per_round))
    if not case["nnz"]:
        case["T"] = min(case["T"], int(_MAX_UNITS / (case["R"] * case["K"] * case["d"])))
    else:
        # (the state of a sparse case is R K d floats)
        case["R"] = min(case["R"], max(1, (1 << 28) // (case["K"] * case["d"])))
        case["T"] = min(case["T"], int(5e8 / (case["R"] * case["K"] * case["nnz"])))
    case["T"] = max(case["calls"], case["T"])
    if not case["nnz"] and rng.random() < 0.3:
        case["seg_len"] = max(100, case["T"] // rng.randint(2, 60))
    return case


# ---------------------------------------------------------------- preparation ----
class _Learner:
    """The handle of a simulation with its inputs, workspace and outputs on the GPU."""

    def __init__(self, case, seed):
        d, K, T, R, nnz = (case[n] for n in ("d", "K", "T", "R", "nnz"))
        g = torch.Generator(device=DEVICE).manual_seed(seed)

        def randn(*shape):
            return torch.randn(shape, generator=g, device=DEVICE, dtype=torch.float32)

        self.case = case
        S = 1 if case["seg_len"] <= 0 else -(-T // case["seg_len"])
        seg = np.arange(S, dtype=np.int64) * max(case["seg_len"], 0)
        bounds = list(seg) + [T]
        self.x = self.col = self.val = self.y = None
        # the parameter behind the labels of every run and segment is also the comparator
        if nnz:
            keep = min(d, 1024)
            u = torch.zeros((R, S, d), device=DEVICE)
            # (one coordinate of each of `keep` equal stretches: distinct, so the same u every time)
            where = torch.randint(0, d // keep, (R, S, keep), generator=g, device=DEVICE)
            where += torch.arange(keep, device=DEVICE) * (d // keep)
            u.scatter_(2, where, randn(R, S, keep))
        else:
            u = randn(R, S, d)
        u *= case["norm"] / u.norm(dim=2, keepdim=True)
        if nnz:
            # ascending distinct columns: a random offset in each of nnz equal stretches of the coordinates
            width = d // nnz
            off = torch.randint(0, width, (T, nnz), generator=g, device=DEVICE, dtype=torch.int32)
            self.col = (off + torch.arange(nnz, device=DEVICE, dtype=torch.int32) * width).contiguous()
            self.val = randn(T, nnz) / math.sqrt(nnz)
        else:
            self.x = randn(T, d) if case["shared"] else randn(R, T, d)
            if case["loss"] == "linear":
                self.x /= self.x.norm(dim=-1, keepdim=True)          # a stream of gradients of norm G = 1
            else:
                self.x *= 1.0 / math.sqrt(d)
        if case["loss"] == "linear":
            # comparator: the best fixed point in hindsight
            tot = self.x.double().sum(dim=-2).expand(R, d)
            u = (-tot / tot.norm(dim=1, keepdim=True)).float()[:, None, :].expand(R, S, d).contiguous()
        else:
            clean = torch.empty((R, T), device=DEVICE)
            for s in range(S):
                a, b = int(bounds[s]), int(bounds[s + 1])
                for r0 in range(0, R, 16 if nnz else R):
                    r1 = min(R, r0 + 16) if nnz else R
                    us = u[r0:r1, s]
                    if nnz:
                        for t0 in range(a, b, 8192):
                            t1 = min(b, t0 + 8192)
                            clean[r0:r1, t0:t1] = (us[:, self.col[t0:t1].long()] * self.val[t0:t1]).sum(dim=2)
                    elif case["shared"]:
                        clean[r0:r1, a:b] = us @ self.x[a:b].t()
                    else:
                        for r in range(r0, r1):
                            clean[r, a:b] = self.x[r, a:b] @ us[r - r0]
            if case["loss"] == "squared":
                self.y = clean + 0.1 * randn(R, T)
            else:
                flip = torch.rand((R, T), generator=g, device=DEVICE) < 0.1
                self.y = torch.where((clean >= 0) ^ flip, 1.0, -1.0)
        self.u = u.contiguous()
        eta = B.oco_step_grid(1.0, 1.0, T, K)
        self.eta, self.eps, self.seg = eta, math.sqrt(math.log(K) / T) if K > 1 else 0.0, bounds
        n = T // case["calls"]
        self.cuts = [(i * n, n if i + 1 < case["calls"] else T - i * n) for i in range(case["calls"])]
        self.cfg, self._keep = B.make_config(d=d, K=K, T=T, R=R, D=1.0, G=1.0, eta=eta,
                                             eps=self.eps, loss=case["loss"],
                                             x_shared=case["shared"], nnz=nnz, n_max=max(c[1] for c in self.cuts),
                                             optimistic=case["optimistic"])
        self.ws = torch.empty(B.oco_workspace_bytes(self.cfg), dtype=torch.uint8, device=DEVICE)
        self.h = B.oco_create(self.cfg, self.ws)
        B.oco_set_comparator(self.h, self.u, seg)
        self.W = torch.empty((R, K, d), device=DEVICE)
        self.p = torch.empty((R, K), device=DEVICE)
        self.wbar = torch.empty((R, d), device=DEVICE)
        self.bounds = torch.empty((R, 4), dtype=torch.float64, device=DEVICE)

    def __del__(self):
        if getattr(self, "h", None):
            torch.cuda.synchronize()
            B.oco_destroy(self.h)
            self.h = None

    def rounds(self, t0, n):
        """Rounds t0 .. t0 + n - 1, by their addresses in the resident streams."""
        case = self.case
        kw = {}
        if case["nnz"]:
            kw.update(col_ptr=self.col.data_ptr() + 4 * t0 * case["nnz"], val_ptr=self.val.data_ptr() + 4 * t0 * case["nnz"])
        else:
            kw.update(x_ptr=self.x.data_ptr() + 4 * t0 * case["d"],
                      x_run_stride=0 if case["shared"] else case["T"] * case["d"])
        if self.y is not None:
            kw.update(y_ptr=self.y.data_ptr() + 4 * t0, y_run_stride=case["T"])
        B.oco_run_rounds(self.h, t0, n, **kw)

    def run(self):
        B.oco_reset(self.h)
        if self.case["host_regret"]:
            for t0, n in self.cuts:
                self.rounds(t0, n)
            B.oco_get_state(self.h, self.W, self.p, self.wbar)
            return {"regret": B.oco_regret(self.h, self.case["R"]), "W": self.W, "p": self.p, "wbar": self.wbar}
        # serving: the combined model is needed after every call
        for t0, n in self.cuts:
            self.rounds(t0, n)
            B.oco_get_state(self.h, None, self.p, self.wbar)
        B.oco_get_state(self.h, self.W, None, None)
        B.oco_accel_bounds(self.h, 4, 0.05, self.bounds)
        return {"W": self.W, "p": self.p, "wbar": self.wbar, "bounds": self.bounds}


class _Steps:
    """A batch of draft / target distributions: softmax of target logits with a few dominant tokens
    and of the same logits with noise, and draft tokens drawn from the draft's."""

    def __init__(self, case, seed):
        n, k, V = case["B"], case["k"], case["V"]
        self.case = case
        g = torch.Generator(device=DEVICE).manual_seed(seed)
        self.p = torch.empty((n, k + 1, V), device=DEVICE)
        self.q = torch.empty((n, k, V), device=DEVICE)
        for b in range(n) if n * V > 1 << 24 else [slice(None)]:
            lp = case["sharp"] * torch.randn(self.p[b].shape, generator=g, device=DEVICE)
            lq = lp[..., :k, :] + case["noise"] * torch.randn(self.q[b].shape, generator=g, device=DEVICE)
            self.p[b] = torch.softmax(lp, dim=-1)
            self.q[b] = torch.softmax(lq, dim=-1)
        self.tok = torch.multinomial(self.q.view(n * k, V), 1, generator=g).view(n, k).to(torch.int32)
        self.r = torch.rand((n, k), generator=g, device=DEVICE)
        self.draw = torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device=DEVICE, dtype=torch.int64).to(torch.int32)
        self.length = torch.empty((n,), dtype=torch.int32, device=DEVICE)
        self.next = torch.empty((n,), dtype=torch.int32, device=DEVICE)
        self.rate = torch.empty((n, k), dtype=torch.float64, device=DEVICE)

    def run(self):
        if self.case["kind"] == "verify":
            B.sd_verify(self.p, self.q, self.tok, self.r, self.draw, self.length, self.next)
            return {"length": self.length, "next": self.next}
        B.sd_acceptance(self.p, self.q, self.rate)
        return {"rate": self.rate}


def prepare(case, seed):
    return (_Learner if case["kind"] == "learn" else _Steps)(case, seed)


def run(state):
    return state.run()


def work(case):
    """Learner: the streams, labels and comparators once, the outputs once (a sparse state also has
    its touched coordinates read and written); per learner, round and touched coordinate an inner
    product and a step, per run and round the comparator's inner product.  Verification: the
    rows that decide the next token (a rejected step needs two, an accepted one one: 1.5 on
    average) and the gathered scalars.  Acceptance: both distributions."""
    if case["kind"] == "verify":
        return {"bytes": case["B"] * (6.0 * case["V"] + 20.0 * case["k"] + 12.0), "flops": 2.0 * case["B"] * case["V"]}
    if case["kind"] == "accept":
        return {"bytes": case["B"] * case["k"] * (8.0 * case["V"] + 8.0), "flops": 2.0 * case["B"] * case["k"] * case["V"]}
    d, K, T, R, nnz = (case[n] for n in ("d", "K", "T", "R", "nnz"))
    S = 1 if case["seg_len"] <= 0 else -(-T // case["seg_len"])
    stream = 8.0 * T * nnz if nnz else 4.0 * T * d * (1 if case["shared"] else R)
    labels = 0.0 if case["loss"] == "linear" else 4.0 * R * T
    out = 4.0 * R * (K * d + K + d) + 8.0 * R
    if not case["host_regret"]:
        out += 4.0 * R * (K + d) * (case["calls"] - 1)
    comparator = 4.0 * R * S * (min(1024, d) if nnz else d)
    touched = nnz if nnz else d
    state = 8.0 * R * K * T * nnz if nnz else 0.0
    return {"bytes": stream + labels + out + comparator + state, "flops": R * T * touched * (4.0 * K + 2.0)}


def tolerance(case):
    if case["kind"] == "verify":
        return "exact"               # integer arithmetic: the draw does not depend on the order of a sum
    if case["kind"] == "accept":
        return {"rel": 1e-15}        # float64 sums (2.5e-16 between two orders of summation)
    # float32 iterates and inner products over up to 10^5 rounds.  Against the same recurrences in
    # float64, or between two kernels that group the sums differently, the iterates differ by up to
    # 1.2e-6 and the regret, a difference of two sums of losses, by up to 3.7e-6 at the listed cases
    # (wide_model); a drawn case may have a regret that is smaller against its losses
    return {"rel": 2e-5}


# ---------------------------------------------------------------- the same in float64 ----
def _phi(loss, z, y):
    if loss == "linear":
        return z
    return (z - y) ** 2 if loss == "squared" else torch.nn.functional.softplus(-y * z)


def _exact_learn(s):
    """The definition, round by round, in float64.  An iterate is kept as scale * vector, so that a
    projection is a scalar; scale and squared norm are taken afresh every 16 rounds."""
    case, f64 = s.case, torch.float64
    d, K, T, R, nnz, loss, opt = (case[n] for n in ("d", "K", "T", "R", "nnz", "loss", "optimistic"))
    eta = torch.tensor([float(np.float32(e)) for e in s.eta], dtype=f64, device=DEVICE).expand(R, K).contiguous()
    v = torch.zeros((d, R, K) if nnz else (R, K, d), dtype=f64, device=DEVICE)
    sc, n2 = torch.ones((R, K), dtype=f64, device=DEVICE), torch.zeros((R, K), dtype=f64, device=DEVICE)
    a, h, x2p, xp, cp = torch.zeros_like(n2), torch.zeros_like(n2), 0.0, None, None
    Z = torch.empty((T, R, K), dtype=f64, device=DEVICE)
    y = None if s.y is None else s.y.to(f64).t().contiguous()[:, :, None]
    one = torch.ones((), dtype=f64, device=DEVICE)

    def factor(m):
        return torch.minimum(one, m.clamp_min(1e-300).rsqrt())

    for t in range(T):
        if nnz:
            cols, x = s.col[t].long(), s.val[t].to(f64)
            rows = v[cols]
            q = torch.einsum("j,jrk->rk", x, rows) * sc
            x2 = x.dot(x)
            if opt:
                g01 = 0.0 if xp is None else ((cols[:, None] == cp[None, :]).to(f64) * x[:, None] * xp[None, :]).sum()
        elif case["shared"]:
            x = s.x[t].to(f64)
            q = torch.mv(v.view(R * K, d), x).view(R, K) * sc
            x2 = x.dot(x)
            if opt:
                g01 = 0.0 if xp is None else x.dot(xp)
        else:
            x = s.x[:, t].to(f64)
            q = (v @ x[:, :, None])[..., 0] * sc
            x2 = (x * x).sum(1, keepdim=True)
            if opt:
                g01 = 0.0 if xp is None else (x * xp).sum(1, keepdim=True)
        z = q
        if opt:
            z = factor(n2 - 2.0 * a * h + a * a * x2p) * (q - a * g01)
        Z[t] = z
        if loss == "linear":
            b = eta
        elif loss == "squared":
            b = 2.0 * eta * (z - y[t])
        else:
            b = -eta * y[t] * torch.sigmoid(-y[t] * z)
        if nnz:
            v[cols] = rows - x[:, None, None] * (b / sc)
        elif case["shared"]:
            v.view(R * K, d).addr_((b / sc).view(-1), x, alpha=-1.0)
        else:
            v.sub_((b / sc)[:, :, None] * x[:, None, :])
        n2 = n2 - 2.0 * b * q + b * b * x2
        f = factor(n2)
        sc = sc * f
        n2 = n2 * f * f
        if opt:
            a, h, x2p, xp, cp = b, f * (q - b * x2), x2, x, cols if nnz else None
        if (t % 16 == 15 and not nnz) or t == T - 1 or (nnz and t % 256 == 255):
            v *= sc if nnz else sc[:, :, None]
            sc = torch.ones_like(sc)
            n2 = v.square().sum(0 if nnz else 2)
    if nnz:
        v = v.permute(1, 2, 0)
    if opt:                                # the iterate that would be played next
        if nnz:
            row = torch.zeros(d, dtype=f64, device=DEVICE).index_add_(0, cp, xp)
        else:
            row = xp if case["shared"] else xp[:, None, :]
        v = v - a[:, :, None] * row
        v = v * factor(v.square().sum(2))[:, :, None]
    # the comparator's predictions, the meta learner and the regret, over all rounds at once
    zu = torch.empty((T, R), dtype=f64, device=DEVICE)
    for i, (t0, t1) in enumerate(zip(s.seg[:-1], s.seg[1:])):
        for r in range(R):
            u = s.u[r, i].to(f64)
            if nnz:
                for c in range(int(t0), int(t1), 8192):
                    e = min(int(t1), c + 8192)
                    zu[c:e, r] = (u[s.col[c:e].long()] * s.val[c:e].to(f64)).sum(1)
            else:
                x = s.x[t0:t1] if case["shared"] else s.x[r, t0:t1]
                for c in range(0, len(x), 8192):
                    zu[t0 + c:t0 + c + len(x[c:c + 8192]), r] = x[c:c + 8192].to(f64) @ u
    losses = _phi(loss, Z, y)
    L = torch.cumsum(losses, 0)
    before = torch.cat([torch.zeros_like(L[:1]), L[:-1]])
    if opt == 2:
        before[1:] += losses[:-1]
    p = torch.softmax(-s.eps * before, 2)
    y2 = None if y is None else y[..., 0]
    regret = (_phi(loss, (p * Z).sum(2), y2) - _phi(loss, zu, y2)).sum(0)
    p = torch.softmax(-s.eps * (L[-1] + (losses[-1] if opt == 2 else 0.0)), 1)
    out = {"W": v.contiguous(), "p": p, "wbar": torch.einsum("rk,rkd->rd", p, v)}
    if case["host_regret"]:
        return {"regret": regret, **out}
    top = 5.0 * T
    low = top / (1.0 + 5.0 * (regret.clamp_min(0.0) / (2.0 * T)).sqrt())
    out["bounds"] = torch.stack([low, torch.full_like(low, top), low / (T * 1.2), torch.full_like(low, 5.0 / 1.2)], 1)
    return out


def exact(case, seed):
    """What run() returns, in float64 by plain torch; None where that takes too long."""
    if case["kind"] == "learn":
        state = 8.0 * case["R"] * case["K"] * case["d"]
        per_round = 1.5e-4 + (state / 256 if case["nnz"] else 4.0 * state) / 4e12
        return None if case["T"] * per_round > 16.0 or state > 1.2e9 else _exact_learn(prepare(case, seed))
    if case["kind"] == "verify":
        return None                        # whole numbers
    s = prepare(case, seed)
    rate = torch.empty_like(s.rate)
    for b in range(case["B"]):
        rate[b] = torch.minimum(s.p[b, :case["k"]], s.q[b]).double().sum(1)
    return {"rate": rate}
