"""The work a user has this library do, as timed cases through its public entry points.

Kinds (each a way in which a program uses the library):

  count    a prepared graph is kept, and motif counts are asked of it again and
           again (Graph.count)
  oneshot  a CSR arrives and is counted once: validation, preparation, both
           samplers, estimates, release (count_motifs)
  batch    many prepared graphs of unequal sizes counted by one captured
           launch (Batch.run)
  served   requests for a relative error on a pool of resident graphs,
           submitted together and waited for (Server.submit / Server.wait)
  ingest   a raw pair list with repeats and loops becomes a CSR
           (csr_from_edges)
  exact    exact counts of a prepared graph, the ground truth of the
           estimates (Graph.exact)

Graphs are the seeded synthetic ones of the package: Erdos-Renyi (one small
graph), Chung-Lu with exponent 2.3 (heavy-tailed, degrees capped) and R-MAT
(heavier-tailed, with hub rows of hundreds of thousands of neighbours and
isolated vertices), drawn from the seed alone.
"""
from __future__ import annotations

import math
from decimal import Decimal, getcontext
from fractions import Fraction

import numpy as np
import torch

from paper_1411_4942_amd import pathsamp as ps
from paper_1411_4942_amd import synth, workloads

DELTA = 0.01  # 99% bars


def listed():
    return [
        # the smallest call: a small graph kept prepared, k = 1e5 (launches and latency)
        {"name": "count er 2e4", "kind": "count", "graph": "er", "n": 2000, "m": 20000, "k_path": 100000,
         "k_cent": 100000},
        # an ordinary social-network-sized graph, k = 2e6
        {"name": "count chung-lu 1e7", "kind": "count", "graph": "cl", "n": 1000000, "m": 10000000,
         "k_path": 2000000, "k_cent": 2000000},
        # the benchmark: R-MAT scale 22, 1.2e8 edges, k = 1e7
        {"name": "count rmat22", "kind": "count", "graph": "rmat", "scale": 22, "edge_factor": 31,
         "k_path": 10000000, "k_cent": 10000000},
        # one-shot jobs: a small graph; an ordinary one with odd sizes; the
        # benchmark graph, at the paper's budget of 200K samples per sampler
        {"name": "oneshot er 2e4", "kind": "oneshot", "graph": "er", "n": 2000, "m": 20000, "k": 100000},
        {"name": "oneshot chung-lu 1e6", "kind": "oneshot", "graph": "cl", "n": 100003, "m": 1000003, "k": 200000},
        {"name": "oneshot rmat22", "kind": "oneshot", "graph": "rmat", "scale": 22, "edge_factor": 31, "k": 200000},
        # the many-graph pool (n 1e3..2e5, m 5e3..2e6), 64 of its graphs, 2e5 samples each
        {"name": "batch 64 graphs", "kind": "batch", "graphs": 64, "m_cap": 2000000, "k": 200000},
        # 64 requests at 2% on a pool of 12 resident graphs up to 5e6 edges
        {"name": "served 64 requests", "kind": "served", "graphs": 12, "m_hi": 5000000, "requests": 64,
         "rel_err": 0.02},
        # raw pair lists: a small one and the benchmark graph's 1.3e8 draws
        {"name": "ingest rmat15", "kind": "ingest", "graph": "rmat", "n": 32768, "scale": 15, "edge_factor": 20.5,
         "m": 540000},
        {"name": "ingest rmat22", "kind": "ingest", "graph": "rmat", "n": 4194304, "scale": 22, "edge_factor": 31,
         "m": 120000000},
        # exact counts: R-MAT scale 16 (dense core: cliques) and Chung-Lu 1e7 (4-cycles, many small rows)
        {"name": "exact rmat16", "kind": "exact", "graph": "rmat", "scale": 16, "edge_factor": 16},
        {"name": "exact chung-lu 1e7", "kind": "exact", "graph": "cl", "n": 1000000, "m": 10000000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, m_lo, m_hi):
    m = _log(rng, m_lo, m_hi)
    if m > 1.5e7 or rng.random() < 0.5:
        ef = rng.uniform(8, 31)
        scale = min(22, max(10, round(math.log2(m / (0.9 * ef)))))
        return {"graph": "rmat", "scale": scale, "edge_factor": round(ef, 2)}
    return {"graph": "cl", "n": max(200, int(m / rng.uniform(5, 20))), "m": m}


def draw(rng):
    kind = rng.choice(["count", "count", "oneshot", "oneshot", "batch", "served", "ingest", "exact"])
    if kind == "count":
        return {"kind": kind, **_draw_graph(rng, 1e4, 1e8), "k_path": _log(rng, 1e4, 1e7),
                "k_cent": _log(rng, 1e4, 1e7)}
    if kind == "oneshot":
        return {"kind": kind, **_draw_graph(rng, 1e4, 1e8), "k": _log(rng, 1e4, 1e6)}
    if kind == "batch":
        return {"kind": kind, "graphs": rng.randint(2, 64), "m_cap": _log(rng, 1e5, 2e6), "k": _log(rng, 2e4, 2e5)}
    if kind == "served":
        return {"kind": kind, "graphs": rng.randint(2, 12), "m_hi": _log(rng, 1e5, 5e6),
                "requests": rng.randint(1, 64), "rel_err": round(math.exp(rng.uniform(math.log(0.02), math.log(0.1))), 4)}
    if kind == "ingest":
        # vertex ids need not fill [0, n)
        if rng.random() < 0.5:
            scale, ef = rng.randint(16, 21), round(rng.uniform(8, 31), 2)
            return {"kind": kind, "graph": "rmat", "n": (1 << scale) + rng.randint(0, 1000), "scale": scale,
                    "edge_factor": ef, "m": int(0.8 * ef * (1 << scale))}
        m = _log(rng, 4e3, 1.5e7)
        return {"kind": kind, "graph": "cl", "n": max(200, int(m / rng.uniform(2, 20))), "m": m}
    return {"kind": kind, **_draw_graph(rng, 1e4, 1e6)}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _csr(case, seed):
    """(off int64[n+1], col int32[2m]) on the GPU."""
    if case["graph"] == "er":
        off, col = synth.erdos_renyi(case["n"], case["m"], seed)
        return torch.from_numpy(off).cuda(), torch.from_numpy(col).cuda()
    if case["graph"] == "cl":
        n, m = case["n"], case["m"]
        return synth.chung_lu_torch(n, min(m, n * (n - 1) // 4), 2.3, min(n - 1.0, 5000.0, math.sqrt(2.0 * m)), seed)
    return synth.rmat_torch(case["scale"], case["edge_factor"], seed=seed)


def _pool(case, seed):
    """Graph recipes of a batch or of a served pool: [(case of _csr, seed)]."""
    if case["kind"] == "batch":
        specs = workloads.batched_specs(case["graphs"], seed=seed)
        for sp in specs:
            sp["m"] = min(sp["m"], case["m_cap"])
    else:
        specs = workloads.served_specs(case["graphs"], seed=seed, m_hi=float(case["m_hi"]))
    for i, sp in enumerate(specs):
        sp["gen_seed"] = seed * 1000 + i
    return specs


def _pairs(case, seed):
    """A raw pair list (int32) of exactly m distinct edges, with repeats in both
    directions and loops: R-MAT draws as they come, less the draws of evenly
    chosen surplus edges; or a Chung-Lu graph's edges in random order and
    direction with 5% repeated and 1% loops added."""
    n, m = case["n"], case["m"]
    if case["graph"] == "rmat":
        u, v = synth.rmat_edges_torch(case["scale"], case["edge_factor"], seed=seed)
        key = torch.minimum(u, v) * n + torch.maximum(u, v)
        real = torch.unique(key[u != v])
        surplus = real.numel() - m
        if surplus < 0:
            raise ValueError("fewer distinct edges than m")
        if surplus:
            drop = real[torch.arange(surplus, device=real.device) * real.numel() // surplus]
            at = torch.searchsorted(drop, key).clamp_(max=surplus - 1)
            keep = drop[at] != key
            u, v = u[keep], v[keep]
        return u.to(torch.int32), v.to(torch.int32)
    off, col = synth.chung_lu_torch(n, min(m, n * (n - 1) // 4), 2.3, min(n - 1.0, 5000.0, math.sqrt(2.0 * m)), seed)
    u = torch.repeat_interleave(torch.arange(n, device=off.device, dtype=torch.int32), off[1:] - off[:-1])
    up = u < col
    gen = torch.Generator(device=off.device)
    gen.manual_seed(seed)
    u, v = u[up], col[up]
    more = torch.randint(0, u.numel(), (u.numel() // 20 + 1,), generator=gen, device=off.device)
    loops = torch.randint(0, n, (u.numel() // 100 + 1,), generator=gen, device=off.device, dtype=torch.int32)
    u, v = torch.cat([u, u[more], loops]), torch.cat([v, v[more], loops])
    flip = torch.rand(u.numel(), generator=gen, device=off.device) < 0.5
    mix = torch.randperm(u.numel(), generator=gen, device=off.device)
    return torch.where(flip, v, u)[mix].contiguous(), torch.where(flip, u, v)[mix].contiguous()


def _philox(seed):
    return 1000003 * seed + 17


def prepare(case, seed):
    kind = case["kind"]
    if kind == "count":
        return {"case": case, "g": ps.Graph(*_csr(case, seed)), "seed": _philox(seed)}
    if kind == "exact":
        return {"case": case, "g": ps.Graph(*_csr(case, seed))}
    if kind == "oneshot":
        off, col = _csr(case, seed)
        return {"case": case, "off": off, "col": col, "seed": _philox(seed)}
    if kind == "batch":
        graphs = [ps.Graph(*workloads.build(sp)) for sp in _pool(case, seed)]
        params = [ps.make_params(case["k"], case["k"], seed=_philox(seed) + i) for i in range(len(graphs))]
        return {"case": case, "batch": ps.Batch(graphs, params)}
    if kind == "served":
        srv = ps.Server()
        ids = [srv.add_graph(*workloads.build(sp)) for sp in _pool(case, seed)]
        for gid in ids:
            srv.preload(gid)
        rng = np.random.Generator(np.random.PCG64(seed))
        reqs = [(int(rng.integers(0, len(ids))), _philox(seed) + q) for q in range(case["requests"])]
        return {"case": case, "srv": srv, "reqs": reqs}
    src, dst = _pairs(case, seed)
    return {"case": case, "n": case["n"], "src": src, "dst": dst}


def _stack(results):
    return {"tallies": np.array([r["tally_path"] + r["tally_cent"] for r in results], dtype=np.int64),
            "k": np.array([[r["k_path"], r["k_cent"]] for r in results], dtype=np.int64),
            **{f: np.array([r[f] for r in results]) for f in ("est", "lo", "hi", "est_basic")}}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "count":
        return state["g"].count(case["k_path"], case["k_cent"], seed=state["seed"])
    if kind == "oneshot":
        return ps.count_motifs(state["off"], state["col"], case["k"], seed=state["seed"])
    if kind == "batch":
        return _stack(state["batch"].run())
    if kind == "served":
        srv = state["srv"]
        tickets = [srv.submit(gid, rel_err=case["rel_err"], delta=DELTA, seed=sd) for gid, sd in state["reqs"]]
        return _stack([srv.wait(t)[0] for t in tickets])
    if kind == "exact":
        return state["g"].exact()
    off, col = ps.csr_from_edges(state["n"], state["src"], state["dst"])
    return {"off": off, "col": col}


# --------------------------------------------------------------------------
# the work a pass cannot do without
# --------------------------------------------------------------------------

SAMPLE_BYTES = 132  # guide, prefixes, endpoints, row bounds, two picks, three tests


def _sizes(case):
    """(vertices, directed slots) of a case's graph; R-MAT keeps about 93% of its draws."""
    if case["graph"] == "rmat":
        return 1 << case["scale"], int(2 * 0.93 * case["edge_factor"] * (1 << case["scale"]))
    return case["n"], 2 * case["m"]


def work(case):
    """Samples cost their own reads; a graph that is prepared or counted exactly
    is read once; a CSR that is made is written once.  Integer work throughout:
    no matrix product and no floating-point count worth naming.  A served
    pass's budgets follow from its pilots, so only the pilots are counted."""
    kind = case["kind"]
    if kind == "count":
        n, slots = _sizes(case)
        # a graph smaller than its samples' reads need be read once only
        return {"bytes": min(SAMPLE_BYTES * (case["k_path"] + case["k_cent"]), 60 * slots), "flops": 0}
    if kind == "oneshot":
        n, slots = _sizes(case)
        return {"bytes": 8 * (n + 1) + 4 * slots + min(SAMPLE_BYTES * 2 * case["k"], 60 * slots), "flops": 0}
    if kind == "batch":
        return {"bytes": SAMPLE_BYTES * 2 * case["k"] * case["graphs"], "flops": 0}
    if kind == "served":
        return {"bytes": SAMPLE_BYTES * 2 * 65536 * case["requests"], "flops": 0}
    if kind == "ingest":
        pairs = int(case["edge_factor"] * (1 << case["scale"])) if case["graph"] == "rmat" else int(1.06 * case["m"])
        return {"bytes": 8 * pairs + 8 * (case["n"] + 1) + 8 * case["m"], "flops": 0}
    n, slots = _sizes(case)
    return {"bytes": 4 * (n + 1) + 4 * slots, "flops": 0}


# --------------------------------------------------------------------------
# the same estimates in plain torch (integers) and decimal arithmetic
# --------------------------------------------------------------------------

M32 = 0xFFFFFFFF
TOP = -(1 << 63)


class _Prepared:
    """Section 4's relabelled graph, both weights and their prefix sums."""

    def __init__(self, off, col):
        n = off.numel() - 1
        deg = off[1:] - off[:-1]
        order = torch.sort(deg, stable=True).indices
        rank = torch.empty_like(order)
        rank[order] = torch.arange(n, device=off.device)
        key = rank[torch.repeat_interleave(torch.arange(n, device=off.device), deg)] * n + rank[col.long()]
        self.key = torch.sort(key).values
        self.n, self.deg = n, deg[order]
        self.start = torch.cumsum(self.deg, 0) - self.deg
        self.u = self.key // n
        self.v = self.key - self.u * n
        du, dv = self.deg[self.u], self.deg[self.v]
        self.luv = du - 1 - (torch.arange(self.key.numel(), device=off.device) - self.start[self.u])
        back = torch.searchsorted(self.key, self.v * n + self.u)
        lvu = dv - 1 - (back - self.start[self.v])
        self.lvu = lvu
        self.p = (torch.cumsum((du - 1) * (dv - 1), 0), torch.cumsum(self.luv * lvu, 0))
        self.R = tuple(int(p[-1]) if p.numel() else 0 for p in self.p)
        self.N1 = sum(int(c) * (d * (d - 1) * (d - 2) // 6)
                      for d, c in zip(*[x.tolist() for x in torch.unique(deg, return_counts=True)]))

    def adjacent(self, a, b):
        k = a * self.n + b
        i = torch.searchsorted(self.key, k).clamp_(max=self.key.numel() - 1)
        return self.key[i] == k


def _philox4x32(c, k0, k1):
    c = list(c)
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & M32) ^ c[1] ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c[3] ^ k1, p0 & M32]
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c


def _uniform(seed, tag, first, count, R):
    """Exact uniforms in [0, R) of samples first .. first + count - 1: a rejected
    first candidate takes the second, then the next block's."""
    ids = torch.arange(first, first + count, device="cuda")
    out = torch.empty_like(ids)
    reject = ((1 << 64) - R) % R
    reject = torch.tensor(reject - (1 << 64) if reject >= 1 << 63 else reject, device="cuda") + TOP
    r0, r1 = R & M32, R >> 32
    todo = torch.arange(count, device="cuda")
    for attempt in range(64):
        i = ids[todo]
        w = _philox4x32([i & M32, i >> 32, torch.full_like(i, tag), torch.full_like(i, attempt)], seed & M32, seed >> 32)
        left = torch.ones_like(i, dtype=torch.bool)
        for x0, x1 in ((w[0], w[1]), (w[2], w[3])):
            p00, p01, p10, p11 = x0 * r0, x0 * r1, x1 * r0, x1 * r1
            mid = ((p00 >> 32) & M32) + (p01 & M32) + (p10 & M32)
            hi = p11 + ((p01 >> 32) & M32) + ((p10 >> 32) & M32) + (mid >> 32)
            lo = (mid << 32) | (p00 & M32)
            take = left & (lo + TOP >= reject)  # unsigned comparison
            out[todo[take]] = hi[take]
            left = left & ~take
        todo = todo[left]
        if todo.numel() == 0:
            return out
    raise RuntimeError("64 blocks without an accepted candidate")


def _tallies(G, seed, centered, k):
    """Counts of motifs 2..6 (3-path sampler) or 4..6 (centered) over ids 0 .. k - 1."""
    got = [0] * 7
    if G.R[centered] == 0:
        return got
    P = G.p[centered]
    for first in range(0, k, 1 << 22):
        r = _uniform(seed, centered, first, min(1 << 22, k - first), G.R[centered])
        s = torch.searchsorted(P, r, right=True)
        o = r - torch.where(s > 0, P[(s - 1).clamp(min=0)], torch.zeros_like(r))
        u, v = G.u[s], G.v[s]
        ou, ov, du, dv = G.start[u], G.start[v], G.deg[u], G.deg[v]
        if centered:
            lvu = G.lvu[s]
            a, b = o // lvu, o % lvu
            x, y = G.v[s + 1 + a], G.v[ov + dv - lvu + b]
        else:
            a, b = o // (dv - 1), o % (dv - 1)
            x, y = G.v[ou + torch.where(a == s - ou, du - 1, a)], G.v[ov + b]
            y = torch.where(y == u, G.v[ov + dv - 1], y)
        ends = G.adjacent(x, y)
        chords = G.adjacent(x, v).long() + G.adjacent(u, y).long()
        kept = x != y
        if centered:
            cls = torch.where(kept & ends, 4 + chords, 0)
        else:
            cls = torch.where(ends, 4 + chords, torch.where(chords == 2, 5, 2 + chords))
            cls = torch.where(kept, cls, 0)
        for c, h in enumerate(torch.bincount(cls, minlength=7).tolist()):
            got[c] += h
    return got


def _bars(count, k):
    """(p_l, p_u) with k D(count / k, p) = ln(1 / delta), to 30 digits."""
    getcontext().prec = 40
    d = Decimal(DELTA)
    edge = (d.ln() / k).exp()
    if count == 0:
        return Decimal(0), 1 - edge
    if count == k:
        return edge, Decimal(1)
    a, goal = Decimal(count) / k, -d.ln() / k
    lna, ln1a = a.ln(), (1 - a).ln()
    out = []
    for sign in (-1, 1):
        # the root in double precision, then Newton's steps to full precision
        f, lo, hi = count / k, (0.0 if sign < 0 else count / k), (count / k if sign < 0 else 1.0)
        for _ in range(80):
            mid = 0.5 * (lo + hi)
            if not 0.0 < mid < 1.0:
                break
            far = f * math.log(f / mid) + (1 - f) * math.log((1 - f) / (1 - mid)) > float(goal)
            if far == (sign > 0):
                hi = mid
            else:
                lo = mid
        p = Decimal(0.5 * (lo + hi))
        for _ in range(6):
            D = a * (lna - p.ln()) + (1 - a) * (ln1a - (1 - p).ln()) - goal
            p -= D * p * (1 - p) / (p - a)
        out.append(p)
    return tuple(out)


A2 = {2: 1, 3: 2, 4: 4, 5: 6, 6: 12}
B = {4: 1, 5: 1, 6: 3}


def _finalized(G, tp, tc, k_path, k_cent):
    """est, lo, hi and est_basic of a count, laid out as the library's."""
    W, L = G.R[0] // 2, G.R[1] // 2
    basic, lo, hi, est = [Fraction(0)] * 7, [Decimal(0)] * 7, [Decimal(0)] * 7, [Fraction(0)] * 7
    basic[1] = Fraction(G.N1)
    blo, bhi = [Decimal(0)] * 7, [Decimal(0)] * 7
    if W and k_path:
        for i, a in A2.items():
            basic[i] = Fraction(tp[i] * W, k_path * a)
            blo[i], bhi[i] = (Decimal(W) / a * p for p in _bars(tp[i], k_path))
        basic[1] = G.N1 - basic[3] - 2 * basic[5] - 4 * basic[6]
    est[1:4], lo[2:4], hi[2:4] = basic[1:4], blo[2:4], bhi[2:4]
    lo[1] = G.N1 - (bhi[3] + 2 * bhi[5] + 4 * bhi[6])
    hi[1] = G.N1 - (blo[3] + 2 * blo[5] + 4 * blo[6])
    if L and k_cent:
        for i, b in B.items():
            est[i] = Fraction(tc[i] * L, k_cent * b)
            lo[i], hi[i] = (Decimal(L) / b * p for p in _bars(tc[i], k_cent))
    return {f: [float(x) for x in v] for f, v in (("est", est), ("lo", lo), ("hi", hi), ("est_basic", basic))}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("count", "oneshot"):
        kp, kc = (case["k"], case["k"]) if kind == "oneshot" else (case["k_path"], case["k_cent"])
        G = _Prepared(*_csr(case, seed))
        got = _finalized(G, _tallies(G, _philox(seed), 0, kp), _tallies(G, _philox(seed), 1, kc), kp, kc)
        return {**dict.fromkeys(("tally_path", "tally_cent", "W", "Lambda", "N1", "k_path", "k_cent")), **got}
    if kind == "batch":
        rows = []
        for i, sp in enumerate(_pool(case, seed)):
            G = _Prepared(*workloads.build(sp))
            sd = _philox(seed) + i
            rows.append(_finalized(G, _tallies(G, sd, 0, case["k"]), _tallies(G, sd, 1, case["k"]), case["k"], case["k"]))
        return {"tallies": None, "k": None, **{f: np.array([r[f] for r in rows]) for f in ("est", "lo", "hi", "est_basic")}}
    return None  # whole numbers (exact, ingest), or budgets that the library sizes by itself (served)
