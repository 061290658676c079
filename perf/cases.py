"""The work that users of libpsl have it do, as cases that can be timed.

Each case is one pass through the library's public calls (paper_2107_09801_amd/libpsl.py)
on inputs made from a seed, with the sizes of the benchmark's workloads, its
studies and the tests, from the smallest unit call to the 1024-walk batch.
Kinds:

  eval   one neighbourhood evaluation of a resident walk, F and PSL of every
         neighbour into the caller's device arrays (the unit call, where
         latency counts);
  loop   a caller's own search iteration: an evaluation, then the forced flip
         of the move it picked, then a read of the walk;
  step   iterations of the search on resident walks (one or many, any mix of
         lengths), then a read of every walk's state;
  serve  a set of jobs of the serving mixture through the request loop;
  init   walks started (the O(L^2) correlation of Eq. (2)), read and released.

Walk slabs are carved from an arena tensor of the caller (a public feature of
the context), so a pass returns the walks' whole device state (bits and C)
without a copy; the scalars come from read_walk, as a search program reads
them between runs of steps.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import seeded_inputs as si
from paper_2107_09801_amd import libpsl

KEYS_I = ("t", "q", "alpha", "psl_pivot", "psl_best", "unimproved", "last_k", "last_start")
KEYS_F = ("value_local", "F_pivot", "last_value_step")
CHOICE_I = ("i_best", "j_best", "j_psl", "psl_min", "psl_k")
CHOICE_F = ("F_best", "F_min")
UNEVEN = "16383x512,32767x256,65535x128,131071x64,262143x32,524287x16,1048575x8"
BIG = 0x9E3779B97F4A7C15
M64 = (1 << 64) - 1


def listed():
    return [
        # the unit call at the smoke check's size: all latency
        {"name": "eval_L1001", "kind": "eval", "L": 1001, "n_lmt": 1001, "alpha1": 4},
        # a caller's own search at a ragged length, the second phase's exponent
        {"name": "loop_L40009_a13", "kind": "loop", "L": 40009, "n_lmt": 40009, "alpha1": 13},
        # a small odd length, the size of the parity tests: launches dominate
        {"name": "step_L1021", "kind": "step", "groups": "1021x1", "n_lmt": 0, "alpha1": 4, "alpha2": 13,
         "period": 50, "steps": 20, "graph": False},
        # the benchmark's single-walk workload
        {"name": "step_L16383", "kind": "step", "groups": "16383x1", "n_lmt": 0, "alpha1": 4, "alpha2": 13,
         "period": 50, "steps": 20, "graph": True},
        # the paper's speed settings (N_lmt = 6912), one walk
        {"name": "paper_L65535", "kind": "step", "groups": "65535x1", "n_lmt": 6912, "alpha1": 4, "alpha2": 10,
         "period": 0, "steps": 20, "graph": True},
        # the same settings as independent runs in one batch
        {"name": "paper_64xL131071", "kind": "step", "groups": "131071x64", "n_lmt": 6912, "alpha1": 4, "alpha2": 10,
         "period": 0, "steps": 10, "graph": False},
        # the benchmark's headline: 1024 walks, full neighbourhood
        {"name": "batch_1024xL131071", "kind": "step", "groups": "131071x1024", "n_lmt": 0, "alpha1": 4,
         "alpha2": 13, "period": 50, "steps": 4, "graph": False},
        # the benchmark's uneven batch: L = 2^m - 1, m = 14..20
        {"name": "uneven_1016", "kind": "step", "groups": UNEVEN, "n_lmt": 0, "alpha1": 4, "alpha2": 0,
         "period": 50, "steps": 2, "graph": False},
        # the longest length, one walk
        {"name": "large_L1048575", "kind": "step", "groups": "1048575x1", "n_lmt": 0, "alpha1": 4, "alpha2": 10,
         "period": 50, "steps": 2, "graph": False},
        # the request loop on the serving mixture (short budgets)
        {"name": "serve_32", "kind": "serve", "jobs": 32, "n_lmt": 256, "budget": 60, "mix": 2},
        # a round of the restart protocol begins: walks started at L = 65535
        {"name": "init_64xL65535", "kind": "init", "groups": "65535x64", "n_lmt": 6912, "alpha1": 4, "alpha2": 13},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval", "loop", "single", "paper", "batch", "uneven", "serve", "init"])
    if kind in ("eval", "loop"):
        L = _log(rng, 127, 60000) | 1
        n = L if rng.random() < 0.6 else _log(rng, 64, L)
        return {"kind": kind, "L": L, "n_lmt": n, "alpha1": rng.choice([4, 4, 10, 11, 13])}
    if kind == "single":
        L = _log(rng, 700, 300000)
        return {"kind": "step", "groups": "%dx1" % L, "n_lmt": 0 if rng.random() < 0.6 else min(L, _log(rng, 256, 6912)),
                "alpha1": 4, "alpha2": rng.choice([4, 10, 13]), "period": rng.choice([0, 50]),
                "steps": 20 if L < 50000 else 4, "graph": rng.random() < 0.5}
    if kind == "paper":
        L = 2 ** rng.randint(14, 18) - 1      # the paper's instances
        return {"kind": "step", "groups": "%dx%d" % (L, _log(rng, 4, 90)), "n_lmt": _log(rng, 1500, 6912), "alpha1": 4,
                "alpha2": rng.choice([10, 13]), "period": 0, "steps": 8, "graph": rng.random() < 0.5}
    if kind == "batch":
        L = _log(rng, 3000, 131071)
        n = max(2, min(_log(rng, 4, 400), int(0.25 * 1024 * 131071.0 ** 2 / L ** 2)))
        return {"kind": "step", "groups": "%dx%d" % (L, n), "n_lmt": 0, "alpha1": 4, "alpha2": 13, "period": 50, "steps": 2,
                "graph": False}
    if kind == "uneven":
        g = []
        for _ in range(rng.randint(3, 6)):
            L = _log(rng, 3000, 300000)
            g.append("%dx%d" % (L, max(1, min(_log(rng, 1, 64), int(0.02 * 1024 * 131071.0 ** 2 / L ** 2)))))
        return {"kind": "step", "groups": ",".join(g), "n_lmt": 0, "alpha1": 4, "alpha2": 0, "period": 50, "steps": 2,
                "graph": False}
    if kind == "serve":
        return {"kind": "serve", "jobs": rng.randint(8, 48), "n_lmt": rng.choice([128, 256, 256, 500]),
                "budget": rng.randint(20, 60), "mix": rng.randint(3, 1 << 20)}
    L = _log(rng, 2000, 131071)
    return {"kind": "init", "groups": "%dx%d" % (L, _log(rng, 1, 64)), "n_lmt": 0, "alpha1": 4, "alpha2": 13}


def _groups(case):
    return [tuple(int(v) for v in g.split("x")) for g in case["groups"].split(",")]


def _alpha2(case, L):
    return case["alpha2"] or si.alpha2_for(L)


def _walk_bytes(L):
    # at least what a walk's slab takes: three bit sets with guards, C twice, flips
    return 8 * L + L + (1 << 14)


def _context(groups):
    arena = torch.zeros(sum(n * _walk_bytes(L) for L, n in groups), dtype=torch.uint8, device="cuda:0")
    torch.cuda.synchronize()        # the context runs on a stream of its own
    return libpsl.Context(0, arena=arena), arena


def _start_walks(ctx, case, groups, seed):
    ids = []
    for L, n in groups:
        ids += ctx.init_walks(L, n, seed + 1000 * len(ids), alpha1=case["alpha1"], alpha2=_alpha2(case, L),
                              n_lmt=min(L, case["n_lmt"]), ls_lmt=2000, switch_period=case.get("period", 0))
    return ids


def _read(ctx, ids):
    s = [ctx.read_walk(w, bits=False, C=False) for w in ids]
    return {"i": np.array([[x[k] for k in KEYS_I] for x in s], dtype=np.int64),
            "f": np.array([[x[k] for k in KEYS_F] for x in s], dtype=np.float64)}


def _seed(seed):
    return si.BASE_SEED + 7919 * int(seed)


def _jobs(case, seed):
    # the mixture of lengths is the case's; the sequences are the seed's
    jobs = si.serve_jobs(case["jobs"], case["mix"], case["n_lmt"])
    for i, j in enumerate(jobs):
        j["budget"] = 1 + j["budget"] * case["budget"] // 500
        j["seed"] = _seed(seed) + i
    return jobs


def prepare(case, seed):
    k = case["kind"]
    st = {"case": dict(case), "seed": _seed(seed), "n": 0}
    if k in ("eval", "loop"):
        L = case["L"]
        st["ctx"], st["arena"] = _context([(L, 1)])
        (st["w"],) = st["ctx"].init_walks(L, 1, st["seed"], alpha1=case["alpha1"], alpha2=4)
        st["F"] = torch.empty(case["n_lmt"], dtype=torch.float64, device="cuda:0")
        st["P"] = torch.empty(case["n_lmt"], dtype=torch.int32, device="cuda:0")
    elif k == "step":
        st["ctx"], st["arena"] = _context(_groups(case))
        st["ids"] = _start_walks(st["ctx"], case, _groups(case), st["seed"])
    elif k == "serve":
        st["ctx"] = libpsl.Context(0)
        st["jobs"] = _jobs(case, seed)
        st["ctx"].serve_start(hbm_budget=8 << 30, max_slots=256)
    else:
        st["ctx"], st["arena"] = _context(_groups(case))
    return st


def _eval_start(st):
    # another start on each pass, as a search draws it
    return (st["seed"] + 7919 * st["n"]) % st["case"]["L"]


def run(st):
    case, ctx = st["case"], st["ctx"]
    k = case["kind"]
    if k in ("eval", "loop"):
        ch = ctx.eval_neighbourhood(st["w"], _eval_start(st), case["n_lmt"], st["F"], st["P"])
        st["n"] += 1
        out = {"F": st["F"], "P": st["P"], "ci": np.array([ch[x] for x in CHOICE_I], dtype=np.int64),
               "cf": np.array([ch[x] for x in CHOICE_F], dtype=np.float64)}
        if k == "loop":
            ctx.apply_flip(st["w"], ch["j_best"])
            r = ctx.read_walk(st["w"])
            out.update(C=r["C"], pivot=r["pivot"].view(np.int64), psl=r["psl_pivot"], F_pivot=float(r["F_pivot"]))
        return out
    if k == "step":
        ctx.step_batch(st["ids"], case["steps"], blocking=True, graph=case["graph"])
        out = _read(ctx, st["ids"])
        out["walks"] = st["arena"]
        return out
    if k == "serve":
        tickets = [ctx.serve_submit(j["L"], j["seed"], j["budget"], alpha2=j["alpha2"], n_lmt=j["n_lmt"],
                                    switch_period=50) for j in st["jobs"]]
        got = {}
        while len(got) < len(tickets):
            for t in tickets:
                if t not in got:
                    r = ctx.serve_poll(t)
                    if r is not None:
                        got[t] = r
        res = [got[t] for t in tickets]
        return {"i": np.array([[r["status"], r["psl_best"], r["psl_final"], r["alpha_final"], r["steps"]] for r in res],
                              dtype=np.int64),
                "F": np.array([r["F_final"] for r in res], dtype=np.float64),
                "best": np.concatenate([r["best"] for r in res]).view(np.int64)}
    ids = _start_walks(ctx, case, _groups(case), st["seed"])
    out = _read(ctx, ids)
    out["walks"] = st["arena"]
    ctx.free_walks(ids)
    return out


def work(case):
    # flops: per neighbour and shift one term chosen and one added (nominal:
    # N_lmt x (L-1) pairs); init: one product and one sum per pair of Eq. (2).
    # bytes: C and the bits read once, C and what a step changes written once.
    k = case["kind"]
    if k in ("eval", "loop"):
        L, n = case["L"], case["n_lmt"]
        b = 4 * L + L / 8 + 12 * n
        return {"bytes": b + (8 * L + L / 8 if k == "loop" else 0), "flops": 2.0 * n * (L - 1)}
    if k == "step":
        b = f = 0.0
        for L, n in _groups(case):
            N = min(L, case["n_lmt"]) or L
            b += case["steps"] * n * (8 * L + L / 8)
            f += case["steps"] * n * 2.0 * N * (L - 1)
        return {"bytes": b, "flops": f}
    if k == "serve":
        jobs = _jobs(case, 1)
        return {"bytes": float(sum(j["budget"] * 8.125 * j["L"] for j in jobs)),
                "flops": float(sum(2.0 * j["budget"] * j["n_lmt"] * (j["L"] - 1) + float(j["L"]) ** 2 for j in jobs))}
    return {"bytes": float(sum(n * (L / 8 + 8 * L) for L, n in _groups(case))),
            "flops": float(sum(n * float(L) ** 2 for L, n in _groups(case)))}


# ------------------------------------------------------------- in 64 bits

def _mix(seed, ctr):
    z = (seed + (ctr + 1) * BIG) & M64
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & M64
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & M64
    return z ^ (z >> 31)


class _Plain:
    """One walk of Algorithm 1 in plain 64-bit torch."""

    def __init__(self, L, seed, alpha1, alpha2, n_lmt, period, flip_lmt=10):
        self.dev = "cuda:0" if torch.cuda.is_available() else "cpu"
        self.L, self.seed, self.a1, self.a2, self.N = L, seed & M64, alpha1, alpha2, n_lmt or L
        self.period, self.flip_lmt = period, min(flip_lmt, L)
        words = np.array([_mix(self.seed, i) for i in range((L + 63) // 64)], dtype="<u8")
        bits = np.unpackbits(words.view(np.uint8), bitorder="little")[:L].astype(np.int32)
        self.s = torch.from_numpy(1 - 2 * bits).to(self.dev)
        self.alpha = alpha1
        self.C = self._corr(self.s)
        self.lb = self.s.clone()
        self.t = self.q = self.unimproved = self.last_k = self.last_start = 0
        self.F = self.vl = self._fit(self.C)
        self.vs = 0.0

    def _corr(self, s):
        n = 1 << (2 * self.L - 1).bit_length()
        f = torch.fft.rfft(s.double(), n)
        return torch.fft.irfft(f * f.conj(), n)[:self.L].round().to(torch.int32)

    def _table(self, n):
        x = torch.arange(n, dtype=torch.float64, device=self.dev)
        t = x.clone()
        for _ in range(self.alpha - 1):
            t = t * x
        return t

    def _fit(self, C):
        a = C[1:].abs().long()
        return float(self._table(int(a.max()) + 1)[a].sum())

    def scan(self, start, N):
        """F and PSL of the N neighbours from `start`."""
        L, dev = self.L, self.dev
        T = self._table(int(self.C[1:].abs().max()) + 5)
        z = torch.zeros(L, dtype=torch.int32, device=dev)
        ext = torch.cat([z, self.s, z])
        k = torch.arange(1, L, device=dev)
        Ck = self.C[1:]
        F, P = [], []
        step = max(1, 30_000_000 // L)
        for i0 in range(0, N, step):
            j = (start + 1 + torch.arange(i0, min(N, i0 + step), device=dev)) % L
            d = ext[(L + j)[:, None] + k] + ext[(L + j)[:, None] - k]
            c = (Ck[None] - 2 * self.s[j][:, None] * d).abs()
            F.append(T[c.long()].sum(1))
            P.append(c.amax(1))
        return torch.cat(F), torch.cat(P)

    def choose(self, start, N):
        F, P = self.scan(start, N)
        fmin = float(F.min())
        i = int(torch.nonzero(F <= fmin * (1 + 1e-12))[0])
        return F, P, i, fmin

    def flip(self, j):
        L = self.L
        z = torch.zeros(L, dtype=torch.int32, device=self.dev)
        ext = torch.cat([z, self.s, z])
        k = torch.arange(1, L, device=self.dev)
        self.C[1:] -= 2 * self.s[j] * (ext[L + j + k] + ext[L + j - k])
        self.s[j] = -self.s[j]

    def step(self):
        start = _mix(self.seed, (1 << 60) | self.t) % self.L
        F, _, i, _ = self.choose(start, self.N)
        j = (start + 1 + i) % self.L
        self.flip(j)
        v = float(F[i])
        self.last_k, self.last_start, self.vs, self.F = j, start, v, v
        sw = False
        if v < self.vl * (1 - 1e-12):
            self.vl, self.unimproved, self.lb = v, 0, self.s.clone()
        elif v > self.vl * (1 + 1e-12):
            self.unimproved += 1
            sw = self.period == 0 and self.unimproved > 2000
        sw = sw or (self.period > 0 and (self.t + 1) % self.period == 0)
        self.t += 1
        if sw:
            self.s = self.lb.clone()
            seen, r = set(), 0
            while len(seen) < self.flip_lmt:
                p = _mix(self.seed, (2 << 60) | (self.q << 24) | r) % self.L
                r += 1
                if p not in seen:
                    seen.add(p)
                    self.s[p] = -self.s[p]
            self.alpha = self.a2 if self.alpha == self.a1 else self.a1
            self.q += 1
            self.C = self._corr(self.s)
            self.F = self.vl = self._fit(self.C)
            self.unimproved = 0


def exact(case, seed):
    k = case["kind"]
    if k in ("eval", "loop"):
        L, N = case["L"], case["n_lmt"]
        w = _Plain(L, _seed(seed), case["alpha1"], 4, L, 0)
        start = _seed(seed) % L
        F, P, i, fmin = w.choose(start, N)
        out = {"F": F, "P": P.to(torch.int32), "ci": None, "cf": np.array([float(F[i]), fmin])}
        if k == "loop":
            w.flip((start + 1 + i) % L)
            out.update(C=w.C.cpu().numpy(), pivot=None, psl=int(w.C[1:].abs().max()), F_pivot=w._fit(w.C))
        return out
    if k == "step":
        (L, n), *more = _groups(case)
        N = min(L, case["n_lmt"]) or L
        if more or n * case["steps"] * float(N) * L > 2e10:
            return None
        fs = []
        for b in range(n):
            w = _Plain(L, _seed(seed) + b, case["alpha1"], _alpha2(case, L), N, case["period"])
            for _ in range(case["steps"]):
                w.step()
            fs.append([w.vl, w.F, w.vs])
        return {"i": None, "f": np.array(fs), "walks": None}
    if k == "init":
        fs = []
        base = 0
        for L, n in _groups(case):
            for b in range(n):
                w = _Plain(L, _seed(seed) + 1000 * base + b, case["alpha1"], 4, L, 0)
                fs.append([w.vl, w.F, 0.0])
            base += n
        return {"i": None, "f": np.array(fs), "walks": None}
    return None
