"""The work that users of this framework have it do, as measurable cases.

A failure has taken nodes out of a DP x PP training grid and the best execution plan for what is left is wanted.
Programs do that in a few ways: load the event and search it once (from scratch), keep a loaded scenario and search
it again, fill a plan cache over many failure sets, score lists or windows of plans they have drawn up themselves,
or re-plan the degrees of parallelism.  Each listed case is one of these; `draw` gives more of the same over the
range of shapes the library takes.  Every output is made of whole numbers, so every case is compared exactly.
"""
import math
import random

import numpy as np
import torch

from paper_2508_21613_amd import binding, synth

INF = (1 << 63) - 1


# ------------------------------------------------------------------------------------------------ cases
def _shape(name, kind, L, PP, DP, M, n_failed=1, cap_x=4.0, comm=200, **kw):
    """one case; cap_x = memory cap of a node over the mean memory of a stage"""
    c = dict(kind=kind, L=L, PP=PP, DP=DP, M=M, n_failed=n_failed, cap_x=cap_x, comm=comm, hetero=False, act=False,
             assign=False, allreduce=0, reroute_cap=0, dist="uniform", mem_lo=400, mem_hi=600, bounded=False)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a scenario kept loaded (a small grid) is searched again; latency and launches count
        _shape("search_small", "search", 32, 4, 2, 8, cap_x=2.0, comm=150),
        # the event itself: tables in, best plan out, 32 cards, with the bounded search a real-time decision uses
        _shape("event_32card", "event", 48, 8, 4, 16, bounded=True),
        # exhaustive search of the same shape: 62.9 M partitions for eight stages, 153 reroute vectors each
        _shape("search_32card", "search", 48, 8, 4, 16),
        # nodes of different speeds, two failures, capped rerouting over seven peers (2,380,833 vectors a stage)
        _shape("search_hetero", "search", 40, 4, 8, 32, n_failed=2, cap_x=2.0, comm=150, hetero=True, reroute_cap=16),
        # every modelling option at once on an uneven grid
        _shape("search_options", "search", 34, 6, 3, 12, n_failed=2, cap_x=3.0, comm=150, hetero=True, act=True,
               assign=True, allreduce=700),
        # a deep pipeline (more stages than the shapes above)
        _shape("search_deep", "search", 26, 20, 2, 32, comm=150),
        # a wide grid: nine peers share the orphaned micro-batches (12,870 vectors)
        _shape("search_wide", "search", 32, 4, 10, 8, cap_x=2.0, comm=150),
        # plan cache: the best plan for many failure sets, searched in one call
        _shape("cache_batch", "batch", 40, 8, 4, 16, n_sets=64),
        # a large list of explicit partitions (cut positions), each of the three strategies
        _shape("list_cuts", "cuts", 96, 16, 2, 64, cap_x=12400 * 16 / 57600, dist="lognormal", mem_lo=300, mem_hi=900, n=1 << 24),
        # costs of a list of partition ranks, an odd number of them, re-partition onto seven uneven nodes
        _shape("list_ranks", "ranks", 48, 8, 4, 16, hetero=True, strategy=1, n=1000003),
        # costs of a window of consecutive rerouting plans (8 bytes out per plan)
        _shape("window_plans", "window", 48, 8, 4, 16, at=0.37, n=1 << 26),
        # new DP/PP degrees for the 31 nodes left of 32
        _shape("replan_31", "replan", 48, 8, 4, 16, dp_lo=2, dp_hi=6, pp_lo=4, pp_hi=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _vectors(peers, total, cap):
    """number of vectors of `peers` entries in [0, cap] (cap <= 0: any) with the given sum"""
    if cap <= 0:
        return math.comb(total + peers - 1, peers - 1)
    return sum((-1) ** j * math.comb(peers, j) * math.comb(total - j * (cap + 1) + peers - 1, peers - 1)
               for j in range(peers + 1) if total - j * (cap + 1) >= 0)


def draw(rng):
    kind = rng.choice(["search", "search", "search", "event", "event", "batch", "cuts", "ranks", "window", "replan"])
    while True:
        deep, wide = rng.random() < 0.12, rng.random() < 0.12
        PP = rng.randint(17, 24) if deep and kind in ("search", "event") else rng.randint(2, 16)
        L = rng.randint(PP + 1, min(96, PP + 6)) if PP > 16 else rng.randint(PP + 1, 96)
        DP = rng.randint(10, 12) if wide and kind in ("search", "event") else rng.randint(2, 8)
        M = _log_int(rng, 2, 8 if DP > 9 else 64)
        n_failed = 2 if DP >= 3 and PP >= 3 and rng.random() < 0.35 else 1
        cap = 0 if rng.random() < 0.7 else max(1, -(-M // (DP - 1)) + rng.randint(1, M))
        c = _shape(None, kind, L, PP, DP, M, n_failed=n_failed, cap_x=round(rng.uniform(3.0, 4.5), 2), comm=rng.randint(0, 300),
                   hetero=rng.random() < 0.4, act=rng.random() < 0.2, assign=rng.random() < 0.3,
                   allreduce=rng.choice([0, 0, 0, rng.randint(100, 1000)]), reroute_cap=cap,
                   bounded=kind in ("search", "event") and rng.random() < 0.4)
        parts = math.comb(L - 1, PP - 1)
        vectors = _vectors(DP - 1, M, cap)
        plain = PP <= 16 and DP <= 9 and vectors <= 1 << 22
        if (L > 64 and c["allreduce"]) or 3 * parts * vectors ** n_failed >= 1 << 61:
            continue
        if kind in ("search", "event") and parts * vectors <= (10 ** 10 if plain else 10 ** 8) and parts <= (3 * 10 ** 7 if plain else 10 ** 6):
            return c
        if kind == "batch" and parts <= 10 ** 7 and vectors <= 4096 and parts * vectors <= 10 ** 9:
            c["n_sets"] = rng.randint(3, 24)
            return c
        if kind in ("cuts", "ranks") and vectors <= 4096:
            c["n"] = _log_int(rng, 1000, 4 * 10 ** 6)
            c["strategy"] = rng.randint(0, 1) if PP > 2 else 0
            return c
        if kind == "window" and n_failed == 1 and 2 <= vectors <= 10 ** 5 and parts * vectors >= 10 ** 4:
            c["at"] = round(rng.random(), 3)
            c["n"] = min(parts * vectors, _log_int(rng, 1000, 5 * 10 ** 7))
            return c
        if kind == "replan":
            dp, pp = rng.randint(2, 4), rng.randint(5, 8)
            L = rng.randint(30, 46)
            return _shape(None, kind, L, pp, dp, rng.randint(8, 24), comm=rng.randint(0, 300), act=rng.random() < 0.3, dp_lo=max(1, dp - 1),
                          dp_hi=dp + 1, pp_lo=max(2, pp - 3), pp_hi=pp + 2, bounded=rng.random() < 0.4)


# ------------------------------------------------------------------------------------------------ inputs
def _failed(rnd, DP, PP, n):
    """n failed nodes in different stages and, as far as there are that many, different pipelines"""
    stages = rnd.sample(range(PP), min(n, PP))
    pipes = rnd.sample(range(DP), n) if n <= DP else [rnd.randrange(DP) for _ in range(n)]
    return [d * PP + s for d, s in zip(pipes, stages)]


def _scenario(case, seed, failed=None):
    rnd = random.Random("%d failed" % seed)
    L, PP, DP = case["L"], case["PP"], case["DP"]
    fwd, bwd, mem = synth.layer_tables(seed, L, dist=case["dist"], mem_lo=case["mem_lo"], mem_hi=case["mem_hi"])
    mean = L * (case["mem_lo"] + case["mem_hi"]) // 2 / PP
    cap = max(int(case["cap_x"] * mean), int(mem.max()) * 4)
    sc = synth.scenario(L, PP, DP, case["M"], fwd, bwd, mem, _failed(rnd, DP, PP, case["n_failed"]) if failed is None else failed,
                        case["comm"], cap, speed=synth.speed_factors(seed, DP, PP) if case["hetero"] else None,
                        reroute_cap=case["reroute_cap"], transfer_assign=int(case["assign"]), allreduce_us=case["allreduce"])
    if case["act"]:
        sc = synth.with_activations(sc, seed, cap_scale=1.1)
    return sc


def _replan(case, seed):
    rnd = random.Random("%d failed" % seed)
    return dict(synth.replan_case(seed, case["L"], case["DP"], case["PP"], [rnd.randrange(case["DP"] * case["PP"])],
                                  case["DP"] * case["M"], (case["dp_lo"], case["dp_hi"]), (case["pp_lo"], case["pp_hi"]),
                                  comm_us=case["comm"], cap_scale=case["cap_x"], horizon_us=2048 * 415400, act=case["act"]),
                bounded_search=int(case["bounded"]))


def _random_cuts(n, L, k, seed, device="cuda"):
    """n sets of k distinct cut positions in 1..L-1, ascending, every subset equally likely"""
    gen = torch.Generator(device=device)
    gen.manual_seed(seed * 7919 + k)
    out = torch.empty((n, k), dtype=torch.uint8, device=device)
    step = 1 << 19
    for i in range(0, n, step):
        m = min(step, n - i)
        keys = torch.rand((m, L - 1), generator=gen, device=device)
        out[i:i + m] = (keys.topk(k, dim=1, sorted=False).indices + 1).sort(dim=1).values.to(torch.uint8)
    return out


def _random_ranks(n, n_part, seed):
    rnd = np.random.default_rng(seed)
    return rnd.integers(0, n_part, size=n, dtype=np.int64)


def _stages(case, strategy):
    return case["PP"] - 1 if strategy == 1 else case["PP"]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "replan":
        return dict(kind=kind, rp=_replan(case, seed))
    if kind == "batch":
        rnd = random.Random("%d sets" % seed)
        nodes = case["DP"] * case["PP"]
        sets = [sorted(rnd.sample(range(nodes), 1 + (i % 4 != 0))) for i in range(case["n_sets"])]
        return dict(kind=kind, handles=[binding.Scenario(_scenario(case, seed, failed=f)) for f in sets])
    sc = _scenario(case, seed)
    if kind == "event":
        return dict(kind=kind, sc=sc, bounded=case["bounded"])
    st = dict(kind=kind, handle=binding.Scenario(sc))
    if kind == "search":
        st["handle"].set_bounded_search(case["bounded"])
    elif kind == "cuts":
        if "name" in case:
            by_cuts = {k: _random_cuts(case["n"], case["L"], k, seed) for k in (case["PP"] - 1, case["PP"] - 2)}
            st["lists"] = [(s, by_cuts[_stages(case, s) - 1]) for s in (0, 1, 2)]
        else:
            st["lists"] = [(case["strategy"], _random_cuts(case["n"], case["L"], _stages(case, case["strategy"]) - 1, seed))]
            st["costs"] = torch.empty(case["n"], dtype=torch.int64, device="cuda")
    elif kind == "ranks":
        fam = st["handle"].family(case["strategy"])
        st["strategy"] = case["strategy"]
        st["ranks"] = torch.from_numpy(_random_ranks(case["n"], fam["n_part"], seed)).cuda()
        st["costs"] = torch.empty(case["n"], dtype=torch.int64, device="cuda")
    elif kind == "window":
        fam = st["handle"].family(2)
        size = fam["n_part"] * fam["n_reroute"]
        st["count"] = min(case["n"], size)
        st["first"] = fam["offset"] + int(case["at"] * (size - st["count"]))
        st["costs"] = torch.empty(st["count"], dtype=torch.int64, device="cuda")
    return st


# ------------------------------------------------------------------------------------------------ one pass
def _row(rc, b, position=0):
    """a return code and a plan as one row of whole numbers of fixed length"""
    row = [rc, position, b["index"], b["cost"], b["strategy"], b["stages"], b["n_affected"], b["t_step_us"], b["t_trans_us"]]
    row += b["cuts"] + [0] * (32 - len(b["cuts"])) + b["affected_stage"] + [0] * (4 - b["n_affected"])
    for r in b["reroute"]:
        row += r
    return np.array(row + [0] * (16 * (4 - b["n_affected"])), dtype=np.uint64)


def _replan_row(p):
    """the same for a re-plan: per pipeline length, micro-batches, time and cuts"""
    if not p["found"]:
        return np.array([0, p["n_candidates"]] + [0] * 565, dtype=np.int64)
    dp, pad = p["dp"], [0] * (16 - p["dp"])
    row = [1, p["n_candidates"], dp, p["t_step_us"], p["fetch_mib"], p["t_trans_us"], p["comm_rounds"]]
    row += p["length"] + pad + p["micro_batches"] + pad + p["pipeline_us"] + pad
    for c in p["cuts"]:
        row += c + [0] * (32 - len(c))
    return np.array(row + [0] * (32 * (16 - dp)), dtype=np.int64)


def run(st):
    kind = st["kind"]
    if kind == "search":
        return _row(*st["handle"].search_best(7))
    if kind == "event":
        g = binding.Scenario(st["sc"])
        g.set_bounded_search(st["bounded"])
        rc, best = g.search_best(7)
        g.close()
        return _row(rc, best)
    if kind == "batch":
        return np.stack([_row(*x) for x in binding.search_best_batch(st["handles"], 7)])
    if kind == "cuts":
        costs = st.get("costs")
        out = [_row(*st["handle"].search_cuts(s, cuts, costs=costs)) for s, cuts in st["lists"]]
        return out if costs is None else out + [costs]
    if kind == "ranks":
        return st["handle"].score_ranks(st["strategy"], st["ranks"], out=st["costs"])
    if kind == "window":
        return st["handle"].score_plans(st["first"], st["count"], out=st["costs"])
    return _replan_row(binding.replan(st["rp"]))


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def _partition_ops(case, stages):
    """stage sums, memory check and weights to fetch, and the time of each distinct pipeline (a few sums and maxima a stage)"""
    return stages * (10 + 11 * (case["DP"] if case["hetero"] else min(case["DP"], 2)))


def work(case):
    kind, L, PP, DP = case["kind"], case["L"], case["PP"], case["DP"]
    table = 4 * (3 * L + DP * PP)
    if kind == "replan":
        nodes, ops = DP * PP - 1, 0.0
        for n in {nodes // dp + r for dp in range(case["dp_lo"], case["dp_hi"] + 1) for r in (0, 1)}:
            if case["pp_lo"] <= n <= case["pp_hi"] and n <= L:
                ops += math.comb(L - 1, n - 1) * 21.0 * n
        return dict(bytes=4 * (3 * L + 1), flops=L * L * PP if case["bounded"] else max(ops, L * L))
    if kind in ("search", "event", "batch"):
        per = sum(math.comb(L - 1, s - 1) * _partition_ops(case, s) for s in (PP, _stages(case, 1), PP) if s >= 1)
        if case["bounded"]:
            per = min(per, 3 * (L * L * PP + 128 * _partition_ops(case, PP)))
        n = case.get("n_sets", 1)
        return dict(bytes=n * (table + 300), flops=n * per)
    if kind == "cuts":
        rows = [PP - 1, _stages(case, 1) - 1, PP - 1] if "name" in case else [_stages(case, case["strategy"]) - 1]
        return dict(bytes=case["n"] * (sum(rows) + (0 if "name" in case else 8)), flops=case["n"] * sum(_partition_ops(case, k + 1) for k in rows))
    if kind == "ranks":
        return dict(bytes=16 * case["n"], flops=case["n"] * _partition_ops(case, _stages(case, case["strategy"])))
    return dict(bytes=8 * case["n"], flops=case["n"] * 2 * DP)


def tolerance(case):
    return "exact"           # costs, indices and plans are whole numbers


# ------------------------------------------------------------------------------------------------ plain 64-bit reference
def _scaled(x, q):
    return (x * int(q) + 32768) >> 16


def _makespan(F, B, M):
    """1F1B time of the pipelines whose stage times are the columns of F and B: in round t every stage runs forward t,
    then backward t - (n - 1 - s); a stage's operation starts when the stage and the operation it waits for are done"""
    n = len(F)
    E = [np.zeros_like(F[0]) for _ in range(n)]
    for t in range(M + n - 1):
        x = np.zeros_like(F[0])
        for s in range(n):
            old = E[s]
            if t < M:
                x = np.maximum(E[s], x) + F[s]
                E[s] = x + B[s] if s == n - 1 else x
            if s >= 1 and 0 <= t - n + s < M:
                E[s - 1] = np.maximum(E[s - 1], old) + B[s - 1]
    return E[0]


class _Model:
    def __init__(self, sc):
        self.sc = sc
        L, S, D, M = self.L, self.S, self.D, self.M = sc["L"], sc["PP"], sc["DP"], sc["M"]
        pre = lambda a: np.concatenate([[0], np.cumsum(np.asarray(a, dtype=np.int64))])
        self.pf, self.pb, self.pw = pre(sc["fwd_us"]), pre(sc["bwd_us"]), pre(sc["mem_mib"])
        self.pa = pre(sc["act_mib"] if sc["act_mib"] is not None else np.zeros(L))
        self.p0 = np.concatenate([[0], np.cumsum([L // S + (s >= S - L % S) for s in range(S)])]).astype(np.int64)
        q = sc["speed_q16"]
        self.q = [[int(q[d * S + s]) if q is not None else 65536 for s in range(S)] for d in range(D)]
        dead = self.dead = [[d * S + s in sc["failed_nodes"] for s in range(S)] for d in range(D)]
        lost = [sum(row) for row in dead]
        lost_at = [sum(dead[d][s] for d in range(D)) for s in range(S)]
        left = {S - n for n in lost if n}
        self.left = min(left) if left else 0
        has = [S >= 2 and not any(dead[d][s] and dead[d][s - 1] for d in range(D) for s in range(S)),
               len(left) == 1 and self.left >= 1, all(n < D for n in lost_at)]
        self.share = self._shares([S - n for n in lost])
        self.hit = [s for s in range(S) if lost_at[s]]
        self.peers = [[d for d in range(D) if not dead[d][s]] for s in self.hit]
        self.orphans = [lost_at[s] * M for s in self.hit]
        self.counts = [_vectors(len(p), o, sc["reroute_cap"]) for p, o in zip(self.peers, self.orphans)]
        has[2] = has[2] and all(self.counts)
        self.families, at = [], 0
        for k in range(3):
            if has[k]:
                stages = self.left if k == 1 else S
                n_part, rr = math.comb(L - 1, stages - 1), math.prod(self.counts) if k == 2 else 1
                self.families.append(dict(strategy=k, stages=stages, offset=at, n_part=n_part, n_reroute=rr))
                at += n_part * rr

    def _shares(self, nodes):
        total = self.D * self.M
        out = [total * n // sum(nodes) for n in nodes]
        d, rest = 0, total - sum(out)
        while rest:
            if nodes[d]:
                out[d] += 1
                rest -= 1
            d = (d + 1) % self.D
        while True:
            alive = [d for d in range(self.D) if nodes[d]]
            empty, big = [d for d in alive if out[d] == 0], max(alive, key=lambda d: (out[d], -d))
            if not empty or out[big] < 2:
                return out
            out[big] -= 1
            out[empty[0]] += 1

    def family(self, k):
        return next((f for f in self.families if f["strategy"] == k), None)

    def cuts(self, ranks, stages):
        """rows of cut positions (with 0 and L at the ends) of partition ranks"""
        rem = np.array(ranks, dtype=np.int64)
        out = np.zeros((len(rem), stages + 1), dtype=np.int64)
        out[:, stages] = self.L
        for i in range(stages - 1, 0, -1):
            column = np.array([min(math.comb(x, i), 1 << 62) for x in range(self.L - 1)], dtype=np.int64)
            x = np.searchsorted(column, rem, side="right") - 1
            out[:, i] = x + 1
            rem -= column[x]
        return out

    def rank(self, cuts):
        return sum(math.comb(int(c) - 1, i + 1) for i, c in enumerate(cuts[1:-1]))

    def _overlap(self, c, j, s):
        lo, hi = np.maximum(c[:, j], self.p0[s]), np.minimum(c[:, j + 1], self.p0[s + 1])
        return np.where(hi > lo, self.pw[np.maximum(hi, lo)] - self.pw[lo], 0)

    def base(self, k, c):
        """(fits, step time without reroute penalty, transition time) of the partitions with the given cuts"""
        sc, n = self.sc, c.shape[1] - 1
        part = lambda p: [p[c[:, j + 1]] - p[c[:, j]] for j in range(n)]
        f, b, w, a = part(self.pf), part(self.pb), part(self.pw), part(self.pa)
        both = lambda v: [v[j] + v[(j + 1) % n] for j in range(n)]
        if k == 0:
            f, b, wm, am = both(f), both(b), both(w), both(a)
        else:
            wm, am = w, a
        fits = np.ones(len(c), dtype=bool)
        step = np.zeros(len(c), dtype=np.int64)
        missing = np.zeros(len(c), dtype=np.int64)
        seen = set()
        for d in range(self.D):
            nodes = [s for s in range(self.S) if k == 2 or not self.dead[d][s]]
            M = self.share[d] if k == 1 else self.M
            if k == 1 and len(nodes) == self.S:          # an untouched pipeline keeps the fault-free layout
                cc = np.tile(self.p0, (1, 1))
                ff = [self.pf[cc[:, j + 1]] - self.pf[cc[:, j]] for j in range(self.S)]
                bb = [self.pb[cc[:, j + 1]] - self.pb[cc[:, j]] for j in range(self.S)]
                for j in range(self.S):
                    peak = self.pw[self.p0[j + 1]] - self.pw[self.p0[j]] + (self.S - j) * (self.pa[self.p0[j + 1]] - self.pa[self.p0[j]])
                    fits &= bool(peak <= sc["mem_cap_mib"])
                t = _makespan([_scaled(x, self.q[d][j]) for j, x in enumerate(ff)], [_scaled(x, self.q[d][j]) for j, x in enumerate(bb)], M)
                step = np.maximum(step, int(t[0]) + (self.S - 1) * sc["comm_us"])
                continue
            q = [65536 if self.dead[d][s] else self.q[d][s] for s in nodes]
            if (tuple(nodes), tuple(q), M) in seen:
                continue
            seen.add((tuple(nodes), tuple(q), M))
            src = list(range(n)) if k == 1 else nodes
            for i, j in enumerate(src):
                if k != 2 or any(not self.dead[e][j] for e in range(self.D)):
                    fits &= wm[j] + (len(src) - i) * am[j] <= sc["mem_cap_mib"]
            t = _makespan([_scaled(f[j], q[i]) for i, j in enumerate(src)], [_scaled(b[j], q[i]) for i, j in enumerate(src)], M)
            step = np.maximum(step, t + (len(src) - 1) * sc["comm_us"])
            if k == 1:
                if sc["transfer_assign"]:
                    G = [np.zeros(len(c), dtype=np.int64) for _ in range(n + 1)]
                    for s in nodes:
                        new = [G[0]]
                        for j in range(n):
                            new.append(np.maximum(np.maximum(G[j + 1], new[j]), G[j] + self._overlap(c, j, s)))
                        G = new
                    have = G[n]
                else:
                    have = sum(self._overlap(c, j, s) for j, s in enumerate(nodes))
                missing = np.maximum(missing, self.pw[-1] - have)
        if k != 1:
            missing = self.pw[-1] - sum(self._overlap(c, j, j) for j in range(n))
        if sc["allreduce_us"]:
            size = [c[:, j + 1] - c[:, j] for j in range(n)]
            if k == 0:
                alive = [any(not self.dead[d][s] for d in range(self.D)) for s in range(n)]
                rounds, taken = np.zeros(len(c), dtype=np.int64), []
                for s in range(n):
                    used = np.zeros(len(c), dtype=np.uint64)
                    if s >= 1 and alive[s - 1]:
                        used = used | taken[s - 1]
                    if s >= 1 and s == n - 1 and alive[s]:
                        used = used | taken[0]
                    mine, need = np.zeros(len(c), dtype=np.uint64), size[s].copy()
                    for bit in range(self.L):
                        free = (need > 0) & ((used >> np.uint64(bit)) & np.uint64(1) == 0)
                        mine |= free.astype(np.uint64) << np.uint64(bit)
                        need -= free
                        rounds = np.where(free, np.maximum(rounds, bit + 1), rounds)
                    taken.append(mine)
            else:
                rounds = np.maximum.reduce(size)
                if k == 1 and any(not any(row) for row in self.dead):
                    rounds = np.maximum(rounds, int(np.diff(self.p0).max()))
            step = step + sc["allreduce_us"] * rounds
        return fits, step, sc["reconf_us"][k] + sc["xfer_us_per_mib"] * missing

    def weights(self, a, c):
        """forward + backward time of stage hit[a] on each of its peers"""
        s = self.hit[a]
        f, b = self.pf[c[:, s + 1]] - self.pf[c[:, s]], self.pb[c[:, s + 1]] - self.pb[c[:, s]]
        return [_scaled(f, self.q[d][s]) + _scaled(b, self.q[d][s]) for d in self.peers[a]]

    def _room(self, a, v, w):
        cap = self.sc["reroute_cap"] if self.sc["reroute_cap"] > 0 else self.orphans[a]
        return np.minimum(cap, v // w)

    def penalty(self, a, c):
        """least penalty over the reroute vectors: the least v within which the peers can take all orphans"""
        w = self.weights(a, c)
        lo, hi = np.zeros(len(c), dtype=np.int64), self.orphans[a] * np.maximum.reduce(w)
        while (lo < hi).any():
            mid = (lo + hi) // 2
            ok = sum(self._room(a, mid, x) for x in w) >= self.orphans[a]
            lo, hi = np.where(ok, lo, mid + 1), np.where(ok, mid, hi)
        return lo

    def vector(self, a, c):
        """lexicographically first vector within the least penalty, for one partition (one row of cuts)"""
        v, w = self.penalty(a, c), self.weights(a, c)
        room = [int(self._room(a, v, x)[0]) for x in w]
        rem, out = self.orphans[a], []
        for i in range(len(room)):
            out.append(max(0, rem - sum(room[i + 1:])))
            rem -= out[-1]
        return out

    def rr_rank(self, a, vec):
        cap, rem, rank = self.sc["reroute_cap"], self.orphans[a], 0
        for i, x in enumerate(vec):
            after = len(vec) - 1 - i
            rank += sum(_vectors(after, rem - t, cap) if after else int(rem == t) for t in range(x))
            rem -= x
        return rank

    def costs(self, k, c, with_penalty=True):
        out = np.empty(len(c), dtype=np.int64)
        for i in range(0, len(c), 1 << 14):
            cc = c[i:i + (1 << 14)]
            fits, step, trans = self.base(k, cc)
            if k == 2 and with_penalty:
                for a in range(len(self.hit)):
                    step = step + self.penalty(a, cc)
            out[i:i + (1 << 14)] = np.where(fits, self.sc["horizon_steps"] * step + trans, INF)
        return out

    def plan(self, k, cuts):
        """the description the library gives of the best plan with this partition"""
        fam, c = self.family(k), cuts.reshape(1, -1)
        cost = int(self.costs(k, c)[0])
        trans = int(self.base(k, c)[2][0])
        vecs = [self.vector(a, c) for a in range(len(self.hit))] if k == 2 else []
        joint = 0
        for a, v in enumerate(vecs):
            joint = joint * self.counts[a] + self.rr_rank(a, v)
        rows = []
        for a, v in enumerate(vecs):
            row = [0] * 16
            for d, x in zip(self.peers[a], v):
                row[d] = x
            rows.append(row)
        return dict(index=fam["offset"] + self.rank(cuts) * fam["n_reroute"] + joint, cost=cost, strategy=k, stages=fam["stages"],
                    cuts=[int(x) for x in cuts[1:-1]], n_affected=len(vecs), affected_stage=list(self.hit) if k == 2 else [],
                    reroute=rows, t_step_us=(cost - trans) // self.sc["horizon_steps"], t_trans_us=trans)

    def search(self):
        best = None
        for fam in self.families:
            c = self.cuts(np.arange(fam["n_part"]), fam["stages"])
            costs = self.costs(fam["strategy"], c)
            at = int(np.argmin(costs))
            if best is None or costs[at] < best[0]:
                best = (int(costs[at]), fam["strategy"], c[at])
        return self.plan(best[1], best[2])

    def all_vectors(self, a):
        cap = self.sc["reroute_cap"] if self.sc["reroute_cap"] > 0 else self.orphans[a]
        rows = np.zeros((1, 0), dtype=np.int64)
        left = np.array([self.orphans[a]], dtype=np.int64)
        peers = len(self.peers[a])
        for i in range(peers):
            after = (peers - 1 - i) * cap
            lo, hi = np.maximum(0, left - after), np.minimum(cap, left)
            take = np.concatenate([np.arange(x, y + 1) for x, y in zip(lo, hi)]) if len(lo) else np.zeros(0, dtype=np.int64)
            rep = np.repeat(np.arange(len(left)), np.maximum(hi - lo + 1, 0))
            rows, left = np.concatenate([rows[rep], take[:, None]], axis=1), left[rep] - take
        return rows


def exact(case, seed):
    kind, cells = case["kind"], 0
    if kind in ("replan", "batch"):
        return None                                     # (hundreds of millions of splits; see the searches for the same sums)
    parts = math.comb(case["L"] - 1, case["PP"] - 1)
    pipes = case["DP"] if case["hetero"] else 2
    cells = case["PP"] * (case["M"] + case["PP"]) * pipes
    if kind in ("search", "event") and parts * cells > 1.2e9:
        return None
    if kind in ("cuts", "ranks") and case["n"] * cells > 1.2e9:
        return None
    m = _Model(_scenario(case, seed))
    if kind in ("search", "event"):
        return _row(0, m.search())
    if kind == "ranks":
        fam = m.family(case["strategy"])
        return torch.from_numpy(m.costs(case["strategy"], m.cuts(_random_ranks(case["n"], fam["n_part"], seed), fam["stages"])))
    if kind == "cuts":
        if "name" in case:
            return None
        fam = m.family(case["strategy"])
        device = "cuda" if torch.cuda.is_available() else "cpu"
        c = _random_cuts(case["n"], case["L"], fam["stages"] - 1, seed, device=device).cpu().numpy().astype(np.int64)
        ends = np.zeros((len(c), 1), dtype=np.int64)
        c = np.concatenate([ends, c, ends + case["L"]], axis=1)
        costs = m.costs(fam["strategy"], c)
        at = int(np.argmin(costs))
        if costs[at] == INF:
            return None
        return [_row(0, m.plan(fam["strategy"], c[at]), at), torch.from_numpy(costs)]
    fam = m.family(2)
    size = fam["n_part"] * fam["n_reroute"]
    count = min(case["n"], size)
    first = int(case["at"] * (size - count))
    R = fam["n_reroute"]
    lo, hi = first // R, (first + count - 1) // R
    if (hi - lo + 1) * cells > 1.2e9:
        return None
    c = m.cuts(np.arange(lo, hi + 1), fam["stages"])
    base = m.costs(2, c, with_penalty=False)
    vecs, w = m.all_vectors(0), np.stack(m.weights(0, c), axis=1)
    out = np.empty((hi - lo + 1, R), dtype=np.int64)
    for i in range(0, len(c), 4096):
        pen = np.zeros((len(w[i:i + 4096]), R), dtype=np.int64)
        for p in range(vecs.shape[1]):
            np.maximum(pen, w[i:i + 4096, p:p + 1] * vecs[None, :, p], out=pen)
        b = base[i:i + 4096, None]
        out[i:i + 4096] = np.where(b == INF, INF, b + m.sc["horizon_steps"] * pen)
    return torch.from_numpy(out.reshape(-1)[first - lo * R:first - lo * R + count])
