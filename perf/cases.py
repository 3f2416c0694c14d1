"""Timed cases of the framework: what a program that uses it calls, at the sizes it is used at.

A case is one pass through the public entry points (`Adpsgd.run`, `run_traced`, `local_steps`,
`step_average`, `average`, `schedule`, `adpsgd_average_noalloc`).  The listed cases follow the six
full-size workloads (65K to 138M parameters, 4 to 32 workers, 1 to 400 tensors), shortened, plus the
options and odd shapes that the tests run: worker counts without a compiled kernel, ragged tensors,
packed rows that are not 16-byte aligned, averaged momentum, Algorithm 1's counter, tracing.

`exact` computes the same passes in 64 bits with plain torch: Philox4x32-10, Box-Muller, momentum
SGD on the noisy quadratic, the replica mean and per-tensor variance, Algorithm 2's controller.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2007_06134_amd as A
import workloads as W

# kinds: how the pass drives the engine
#   run      reset, then run(steps): a whole training run, as bench.py times it
#   traced   reset, then run_traced(steps): the run with per-step variance and gradient norm
#   manual   `rounds` periods of local_steps(p - 1), step_average(), schedule(): a program that
#            drives Algorithm 2 itself
#   split    `rounds` times local_steps(steps), then a separate average()
#   noalloc  local_steps(1), then the context-free adpsgd_average_noalloc on the replicas
_DEFAULT = dict(kind="run", K=8, P=65536, T=1, lo=64, seed_sizes=1002, fixed="", multiple=4, steps=8, rounds=1,
                sigma=0.05, momentum=0.9, wd=0.0, h_lo=1e-2, lr_kind=W.LR_CONST, lr0=0.05, total=100,
                mode=W.PERIOD_CONST, p=4, k_s=0, avg_m=False, pad=True)


def _case(name=None, **kw):
    c = dict(_DEFAULT, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    adaptive, const, alg1 = W.PERIOD_ADAPTIVE, W.PERIOD_CONST, W.PERIOD_ALG1
    return [
        # the smallest full workload, whole: 200 steps of 65,536 parameters, where launches count
        _case("run_k4_p65k", K=4, P=65_536, sigma=0.1, total=200, steps=200),
        # the smallest call: one step and a separate sync, where a program waits for the variance
        _case("step_sync_k4_p65k", kind="split", K=4, P=65_536, sigma=0.1, steps=1, rounds=1, total=200),
        # 400 small tensors, 32 workers, adaptive: the first 400 steps of a shortened run
        _case("run_k32_p1m2_t400", K=32, P=1_200_000, T=400, lo=16, seed_sizes=1005, sigma=0.2, total=400,
              steps=400, mode=adaptive, p=4, k_s=100),
        # a ResNet18-sized vector with the step-decayed rate, adaptive from p = 1 (a sync a step at first)
        _case("run_k8_p11m_t62", K=8, P=11_200_000, T=62, sigma=0.05, wd=5e-4, lr_kind=W.LR_STEP, lr0=0.1,
              total=200, steps=200, mode=adaptive, p=1, k_s=50),
        # a ResNet50-sized vector, 16 workers, cosine rate, adaptive
        _case("run_k16_p26m_t161", K=16, P=25_600_000, T=161, seed_sizes=1003, sigma=0.1, wd=1e-4, h_lo=1e-3,
              lr_kind=W.LR_COSINE, lr0=0.1, total=100, steps=100, mode=adaptive, p=4, k_s=25),
        # the 138M-parameter vector (VGG16-sized), the bandwidth-bound workload
        _case("run_k8_p138m_t32", K=8, P=138_000_000, T=32, seed_sizes=1004, fixed="102000000,16800000,4100000",
              sigma=0.02, wd=5e-4, lr0=0.01, total=32, steps=32, mode=adaptive, p=4, k_s=16),
        # a program's own Algorithm 2 loop on the ResNet18-sized vector
        _case("loop_k8_p11m_t62", kind="manual", K=8, P=11_200_000, T=62, wd=5e-4, lr0=0.1, total=2000,
              mode=adaptive, p=4, k_s=500, rounds=4),
        # plain steps, then a separate sync (period 8 without the fused kernel)
        _case("steps_sync_k16_p26m", kind="split", K=16, P=25_600_000, T=161, seed_sizes=1003, sigma=0.1, wd=1e-4,
              h_lo=1e-3, lr0=0.1, total=1000, steps=8, rounds=1),
        # the variance and gradient norm of every step, for plots of the method
        _case("traced_k8_p11m_t62", kind="traced", K=8, P=11_200_000, T=62, wd=5e-4, lr_kind=W.LR_STEP, lr0=0.1,
              total=24, steps=24, mode=adaptive, p=4, k_s=12),
        # five workers, ragged tensors in packed rows (not 16-byte aligned), averaged momentum, Algorithm 1
        _case("run_k5_p1m_packed_ragged", K=5, P=1_000_003, T=19, lo=3, multiple=1, sigma=0.1, wd=1e-4,
              total=60, steps=60, mode=alg1, p=3, avg_m=True, pad=False),
        # more workers than a block has waves
        _case("run_k100_p500k", K=100, P=500_001, T=37, lo=5, multiple=1, sigma=0.1, total=40, steps=40, mode=const,
              p=4),
        # the sync for programs that cannot allocate device memory
        _case("noalloc_k32_p1m2_t400", kind="noalloc", K=32, P=1_200_000, T=400, lo=16, seed_sizes=1005, sigma=0.2,
              total=400, pad=False),
    ]


_MOST_UPDATES = 8 * 138_000_000 * 32     # K P steps of the largest listed case


def draw(rng):
    kind = rng.choice(["run", "run", "run", "run", "traced", "manual", "split", "noalloc"])
    K = rng.choice([2, 4, 8, 16, 32]) if rng.random() < 0.6 else rng.randint(2, 100)
    pad = rng.random() < 0.8
    # rows that need scalar accesses, the two-pass kernel for many workers and tracing cost more a step
    most = _MOST_UPDATES / (8 if not pad or K > 64 or kind == "traced" else 2)
    most_p = min(138e6, 1.2e9 / K, most / (8 * K))
    P = int(math.exp(rng.uniform(math.log(6_000), math.log(most_p))))
    multiple = rng.choice([1, 4])
    P -= P % multiple
    T = int(math.exp(rng.uniform(0, math.log(min(400, P // 64)))))
    mode = rng.choice([W.PERIOD_CONST, W.PERIOD_ADAPTIVE, W.PERIOD_ADAPTIVE, W.PERIOD_ALG1])
    p = rng.randint(1, 12)
    c = dict(kind=kind, K=K, P=P, T=T, lo=rng.randint(1, 64), seed_sizes=rng.randint(1, 10_000), multiple=multiple,
             sigma=rng.choice([0.02, 0.05, 0.1, 0.2]), momentum=rng.choice([0.0, 0.9, 0.9, 0.9]),
             wd=rng.choice([0.0, 1e-4, 5e-4]), h_lo=rng.choice([1e-3, 1e-2]),
             lr_kind=rng.choice([W.LR_CONST, W.LR_STEP, W.LR_COSINE]), lr0=rng.choice([0.01, 0.05, 0.1]),
             mode=mode, p=p, avg_m=rng.random() < 0.15, pad=pad)
    room = max(8, int(most / (K * P)))
    if kind in ("run", "traced"):
        c["steps"] = rng.randint(8, min(400, room))
        c["total"] = c["steps"]
        c["k_s"] = c["steps"] // 4 if mode == W.PERIOD_ADAPTIVE else 0
    elif kind == "manual":
        c.update(mode=W.PERIOD_ADAPTIVE, p=rng.randint(1, 8), rounds=rng.randint(1, 4), total=1000, k_s=500)
        c["p"] = max(1, min(c["p"], room // c["rounds"]))
    elif kind == "split":
        c.update(mode=W.PERIOD_CONST, rounds=rng.randint(1, 2), total=1000)
        c["steps"] = rng.randint(1, min(12, room // c["rounds"]))
    else:
        c.update(mode=W.PERIOD_CONST, total=1000, avg_m=False)   # (the context-free sync has no momentum)
    return _case(**c)


def _workload(c, seed):
    fixed = [int(v) for v in c["fixed"].split(",")] if c["fixed"] else None
    if c["T"] == 1:
        sizes = (c["P"],)
    else:
        hi = max(c["lo"] + 1, min(2.4e6 if c["lo"] >= 64 else 65_536, c["P"]))
        sizes = W.log_uniform_sizes(c["seed_sizes"], c["T"], c["lo"], hi, c["P"], multiple=c["multiple"],
                                    minimum=max(c["multiple"], 4 if c["multiple"] == 4 else 1), fixed=fixed)
    return W.Workload(name="case", K=c["K"], sizes=sizes, seed=seed, sigma=c["sigma"], momentum=c["momentum"],
                      weight_decay=c["wd"], h_lo=c["h_lo"], h_hi=1.0, lr_kind=c["lr_kind"], lr0=c["lr0"],
                      total_steps=c["total"], period_mode=c["mode"], p_init=c["p"], k_s=c["k_s"],
                      avg_momentum=c["avg_m"])


def prepare(case, seed):
    """The context with its device buffers, as a program makes it once before training."""
    w = _workload(case, seed)
    return {"case": case, "eng": A.Adpsgd.from_workload(w, pad_rows=case["pad"])}


def run(state):
    c, eng = state["case"], state["eng"]
    kind = c["kind"]
    out = {"x": eng.x, "m": eng.m}
    if kind == "run":
        eng.reset()
        recs, var, n = eng.run(c["steps"])
        out.update(t=recs["t"], p=recs["p"], S=recs["S"], C2=recs["C2"], var=var, n=n)
    elif kind == "traced":
        eng.reset()
        recs, var, n, steps = eng.run_traced(c["steps"])
        out.update(t=recs["t"], p=recs["p"], S=recs["S"], var=var, n=n, step_var=steps["var"],
                   grad_norm2=steps["grad_norm2"])
    elif kind == "manual":
        p = eng.get_state().p
        out["var"] = []
        for _ in range(c["rounds"]):
            eng.local_steps(p - 1)
            var = eng.step_average()
            p = eng.schedule(var)
            out["var"].append(var)
        out["next_p"] = p
    elif kind == "split":
        out["var"] = []
        for _ in range(c["rounds"]):
            eng.local_steps(c["steps"])
            out["var"].append(eng.average())
    else:
        eng.local_steps(1)
        out["var"] = A.adpsgd_average_noalloc(eng.K, eng.P, eng.row_stride, eng.offsets, eng.x.data_ptr(),
                                              eng.stream.cuda_stream)
    return out


def _steps_of(c):
    if c["kind"] in ("run", "traced"):
        return c["steps"]
    if c["kind"] == "manual":
        return c["p"] * c["rounds"]        # (the sampling phase: p does not move)
    return c["steps"] * c["rounds"] if c["kind"] == "split" else 1


def _syncs_of(c):
    if c["kind"] == "run":
        return c["steps"] / c["p"]
    if c["kind"] == "traced":
        return c["steps"]                  # every step is measured
    return c["rounds"] if c["kind"] in ("manual", "split") else 1


def work(case):
    K, P = case["K"], case["P"]
    # x and m read and written once, h and x* read once, whatever the number of steps: a step needs
    # nothing of another element.  (An adaptive run's periods wait for S, but x and m could stay on chip.)
    # Per update: 60 integer operations of Philox and 32 of Box-Muller per four elements, 8 of the step;
    # per element and sync 5 (the mean, the squared deviation and their sums).
    return {"bytes": 16.0 * K * P + 8.0 * P,
            "flops": K * P * (31.0 * _steps_of(case) + 5.0 * _syncs_of(case))}


def tolerance(case):
    # fp32 state against 64 bits, measured: x 0.8-2.7e-7, S and the variances 0.2-3.5e-7, m 0.7e-7 to
    # 3.6e-6 (the step-decayed run, whose momentum nearly cancels at the end); four times the largest
    return {"rel": 1.5e-5}


# ---------------------------------------------------------------- 64-bit reference, plain torch

_M0, _M1, _W0, _W1, _MASK = 0xD2511F53, 0xCD9E8D57, 0x9E3779B9, 0xBB67AE85, 0xFFFFFFFF


def _mulhilo(a, const):
    """(high, low) words of a * const for 32-bit words held in int64 (const < 2^32)."""
    lo = a * (const & 0xFFFF)                       # < 2^48
    hi = a * (const >> 16)                          # < 2^48
    mid = hi + (lo >> 16)
    return mid >> 16, ((mid & 0xFFFF) << 16) | (lo & 0xFFFF)


def _philox(c0, c1, c2, c3, seed):
    k0, k1 = seed & _MASK, (seed >> 32) & _MASK
    for _ in range(10):
        h0, l0 = _mulhilo(c0, _M0)
        h1, l1 = _mulhilo(c2, _M1)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + _W0) & _MASK, (k1 + _W1) & _MASK
    return c0, c1, c2, c3


def _words(g0, g1, k, t, tag, seed, dev):
    """The four words of groups g0 .. g1 - 1 for the workers k (a list): [len(k), g1 - g0] each."""
    g = torch.arange(g0, g1, device=dev, dtype=torch.int64)[None, :].expand(len(k), -1)
    kk = torch.tensor(k, device=dev, dtype=torch.int64)[:, None].expand(-1, g1 - g0)
    return _philox(g, kk, torch.full_like(g, t), torch.full_like(g, tag), seed)


def _normals(words):
    z = []
    for a, b in ((words[0], words[1]), (words[2], words[3])):
        r = torch.sqrt(-2.0 * torch.log(((a >> 8) + 1).double() * 2.0 ** -24))
        th = (b >> 8).double() * (2.0 * math.pi * 2.0 ** -24)
        z += [r * torch.cos(th), r * torch.sin(th)]
    return torch.stack(z, dim=-1).flatten(-2)       # [K, 4 G]


class _Exact:
    """Algorithm 2 in 64 bits on the flat replicas."""

    def __init__(self, c, seed):
        self.w = w = _workload(c, seed)
        self.dev = dev = torch.device("cuda")
        self.off = w.offsets()
        K, P = w.K, w.P
        self.x = torch.zeros((K, P), device=dev, dtype=torch.float64)
        self.m = torch.zeros_like(self.x)
        self.h = torch.empty(P, device=dev, dtype=torch.float64)
        self.xs = torch.empty_like(self.h)
        span = math.log(w.h_hi) - math.log(w.h_lo)
        for e0, e1 in self._cuts(1 << 24):
            u = torch.stack(_words(e0 // 4, (e1 + 3) // 4, [0], 0, 1, seed, dev), -1).flatten(-2)[0, :e1 - e0]
            self.h[e0:e1] = torch.exp((u >> 8).double() * (2.0 ** -24 * span) + math.log(w.h_lo))
            self.xs[e0:e1] = _normals(_words(e0 // 4, (e1 + 3) // 4, [0], 0, 2, seed, dev))[0, :e1 - e0]
        self.t = self.cnt = self.nC2 = 0
        self.p, self.C2 = w.p_init, 0.0

    def _cuts(self, n):
        n -= n % 4
        return [(e, min(e + n, self.w.P)) for e in range(0, self.w.P, n)]

    def lr(self, t):
        w, N = self.w, self.w.total_steps
        if w.lr_kind == W.LR_STEP:
            return w.lr0 * (0.01 if t >= 3 * N // 4 else 0.1 if t >= N // 2 else 1.0)
        if w.lr_kind == W.LR_COSINE:
            return w.lr0 * (1.0 + math.cos(math.pi * t / N)) / 2.0
        return w.lr0

    def step(self):
        w, t = self.w, self.t
        rows = max(1, min(w.K, (1 << 24) // w.P))
        for k0 in range(0, w.K, rows):
            ks = list(range(k0, min(k0 + rows, w.K)))
            for e0, e1 in self._cuts(1 << 24):
                z = _normals(_words(e0 // 4, (e1 + 3) // 4, ks, t, 0, w.seed, self.dev))[:, :e1 - e0]
                x, m = self.x[ks[0]:ks[-1] + 1, e0:e1], self.m[ks[0]:ks[-1] + 1, e0:e1]
                d = self.h[e0:e1] * (x - self.xs[e0:e1]) + w.sigma * z + w.weight_decay * x
                m.mul_(w.momentum).add_(d)
                x.sub_(self.lr(t) * m)
        self.t += 1
        self.cnt += 1

    def measure(self, mean_back, norm=False):
        """Per-tensor variance (and the squared gradient norm at the mean); the mean written back."""
        w = self.w
        d2 = torch.empty(w.P, device=self.dev, dtype=torch.float64)
        gn = torch.zeros((), device=self.dev, dtype=torch.float64)
        for e0, e1 in self._cuts((1 << 26) // w.K + 4):
            x = self.x[:, e0:e1]
            mean = x.mean(0)
            d2[e0:e1] = (x - mean).square().sum(0)
            if norm:
                gn += (self.h[e0:e1] * (mean - self.xs[e0:e1]) + w.weight_decay * mean).square().sum()
            if mean_back:
                x.copy_(mean.expand_as(x))
                if w.avg_momentum:
                    m = self.m[:, e0:e1]
                    m.copy_(m.mean(0).expand_as(m))
        var = torch.stack([d2[a:b].sum() for a, b in zip(self.off[:-1], self.off[1:])]).cpu().numpy() / w.K
        if mean_back:
            self.cnt = 0
        return var, float(gn)

    def control(self, t, S):
        w, g = self.w, self.lr(t)
        if w.period_mode != W.PERIOD_ADAPTIVE:
            return
        if t < w.k_s:
            self.nC2 += 1
            self.C2 += (S / g - self.C2) / self.nC2
        elif S < w.thr_lo * g * self.C2:
            self.p += 1
        elif S > w.thr_hi * g * self.C2:
            self.p = max(1, self.p - 1)

    def due(self):
        if self.w.period_mode == W.PERIOD_ALG1:
            return (self.t - 1) % self.p == 0
        return self.cnt >= self.p


def exact(case, seed):
    c = case
    e = _Exact(c, seed)
    out = {"x": e.x, "m": e.m}
    if c["kind"] in ("run", "traced"):
        traced = c["kind"] == "traced"
        log = dict(t=[], p=[], S=[], C2=[], var=[])
        sv, gn2 = [], []
        for _ in range(c["steps"]):
            e.step()
            due = e.due()
            if not (due or traced):
                continue
            var, gn = e.measure(due, traced)
            sv.append(var.sum())
            gn2.append(gn)
            if due:
                p = e.p
                e.control(e.t - 1, float(var.sum()))
                for k, v in dict(t=e.t - 1, p=p, S=var.sum(), C2=e.C2, var=var).items():
                    log[k].append(v)
        out.update(t=np.array(log["t"], dtype=np.int64), p=np.array(log["p"], dtype=np.int32), S=np.array(log["S"]),
                   var=np.array(log["var"]).reshape(-1, c["T"]), n=len(log["t"]))
        out.update(dict(step_var=np.array(sv), grad_norm2=np.array(gn2)) if traced else dict(C2=np.array(log["C2"])))
    elif c["kind"] == "manual":
        out["var"] = []
        for _ in range(c["rounds"]):
            for _ in range(e.p):
                e.step()
            var, _ = e.measure(True)
            e.control(e.t - 1, float(var.sum()))
            out["var"].append(var)
        out["next_p"] = e.p
    else:
        out["var"] = []
        for _ in range(c["rounds"] if c["kind"] == "split" else 1):
            for _ in range(c["steps"] if c["kind"] == "split" else 1):
                e.step()
            out["var"].append(e.measure(True)[0])
        if c["kind"] == "noalloc":
            out["var"] = out["var"][0]
    return out
