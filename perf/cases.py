"""The work a user of this package has it do, as measurable cases.

Each case is one call path of the public Python API on inputs drawn on the
GPU from a seed: a decode step over a team table, the dense step, the
preparation of a prompt (contiguous parents, or k-means parents), and the
routing diagnostic.  Shapes are those of the package's own workloads
(``datagen.WORKLOADS``) and of its tests, or generic odd sizes beside them.

Key distribution (as in ``datagen``): clusters of centre norm r with unit
noise, four channels ten times larger, queries near one cluster per KV head;
Zipf cluster populations where a case says so.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2609_35629_amd as sp

# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------


def _decode(name, B, N, K, T, P=1024, R=16, Hq=28, Hkv=4, d=128, dtype="bf16", zipf=0.0):
    return dict(name=name, kind="decode", B=B, Hq=Hq, Hkv=Hkv, N=N, d=d, dtype=dtype, P=P, R=R, K=K, T=T, zipf=zipf)


def _dense(name, B, N, T, Hq=28, Hkv=4, d=128, dtype="bf16"):
    return dict(name=name, kind="dense", B=B, Hq=Hq, Hkv=Hkv, N=N, d=d, dtype=dtype, T=T, zipf=0.0)


def _prep(name, kind, B, N, P=1024, R=16, Hkv=4, d=128, dtype="bf16"):
    return dict(name=name, kind=kind, B=B, Hq=Hkv, Hkv=Hkv, N=N, d=d, dtype=dtype, P=P, R=R, zipf=0.0)


def listed():
    return [
        # one interactive sequence early in its life: a step of one layer, all latency
        _decode("decode-8k", B=1, N=8192, K=32, T=64),
        # the package's headline: one sequence, a 32K prompt
        _decode("decode-32k", B=1, N=32768, K=32, T=128),
        # a serving batch of such sequences with longer answers
        _decode("decode-32k-b8", B=8, N=32768, K=32, T=512),
        # long documents, a few topics dominating (uneven teams): the largest step
        _decode("decode-131k-b4", B=4, N=131072, K=64, T=256, zipf=1.2),
        # the paper's own granularity: teams of about four rows (P = 16, R = 4)
        _decode("decode-32k-fine", B=1, N=32768, K=32, T=128, P=16, R=4),
        # fp32 caches of a smaller head, a prompt that no tile divides
        _decode("decode-fp32-d64", B=2, N=8191, K=32, T=33, Hq=16, d=64, dtype="fp32"),
        # the exact step a user falls back to (and compares with), single sequence
        _dense("dense-32k", B=1, N=32768, T=128),
        # the same for a batch, ragged lengths
        _dense("dense-30011-b8", B=8, N=30011, T=37),
        # after prefill: the team table of one layer
        _prep("build-32k", "build", B=1, N=32768),
        # the same for fp32 caches and a prompt with a short last parent
        _prep("build-fp32-9001", "build", B=1, N=9001, dtype="fp32"),
        # after prefill with k-means parents: labels, then the table
        _prep("kmeans-32k", "kmeans", B=1, N=32768),
        # how well a table routes, for both kinds of routing key
        dict(_prep("routing-kl-32k", "kl", B=1, N=32768), Hq=28),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 6 + ["dense"] * 3 + ["build"] * 3 + ["kmeans", "kl"])
    dtype = "bf16" if kind == "kmeans" or rng.random() < 0.75 else "fp32"
    d = 128 if rng.random() < 0.7 else 64
    Hq, Hkv = rng.choice([(28, 4), (28, 4), (16, 4), (32, 8), (12, 2), (8, 8)])
    if kind == "decode":
        P, R = rng.choice([(1024, 16), (1024, 16), (256, 8), (512, 24), (16, 4)])
        most = 8192 * P // R - P if dtype == "bf16" else 32768  # teams a step can sample from
        N = _log_int(rng, 1024, min(most, 131072 if dtype == "bf16" else 32768))
        B = rng.randint(1, max(1, min(8, 262144 // N)))
        M = _team_count(N, P, R)
        K = min(_log_int(rng, 8, 128), max(1, M // 2))
        return dict(kind=kind, B=B, Hq=Hq, Hkv=Hkv, N=N, d=d, dtype=dtype, P=P, R=R, K=K, T=rng.randint(0, 512),
                    zipf=rng.choice([0.0, 0.0, 1.2]))
    if kind == "dense":
        N = _log_int(rng, 1024, 131072 if dtype == "bf16" else 32768)
        B = rng.randint(1, max(1, min(8, 240000 // N if dtype == "bf16" else 65536 // N)))
        return dict(kind=kind, B=B, Hq=Hq, Hkv=Hkv, N=N, d=d, dtype=dtype, T=rng.randint(0, 512), zipf=0.0)
    if kind == "build":
        P, R = rng.choice([(1024, 16), (1024, 16), (256, 8), (512, 24), (16, 4)])
        N = _log_int(rng, 1024, 65536 if dtype == "bf16" else 16384)
        return dict(kind=kind, B=1, Hq=Hkv, Hkv=Hkv, N=N, d=d, dtype=dtype, P=P, R=R, zipf=rng.choice([0.0, 1.2]))
    if kind == "kmeans":
        N = _log_int(rng, 2048, 32768)
        P = max(256, -(-N // 32))
        return dict(kind=kind, B=1, Hq=4, Hkv=rng.choice([2, 4]), N=N, d=d, dtype=dtype, P=P, R=16, zipf=0.0)
    P, R = rng.choice([(1024, 16), (256, 8), (16, 4)])
    N = _log_int(rng, 2048, 32768)
    return dict(kind=kind, B=1, Hq=Hq, Hkv=Hkv, N=N, d=d, dtype=dtype, P=P, R=R, zipf=0.0)


def _team_count(N, P, R):
    full = -(-N // P) - 1
    return full * min(R, P) + min(R, N - full * P)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------


def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _draws(case, seed):
    """K, V [B,Hkv,N,d], suffix K, V [B,Hkv,T,d] (None without rows) and q
    [B,Hq,d], the same bytes for the same case and seed."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    B, Hq, Hkv, N, d, T = case["B"], case["Hq"], case["Hkv"], case["N"], case["d"], case.get("T", 0)
    BH, C, dt = B * Hkv, 256, _torch_dtype(case)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    centers = normal(BH, C, d)
    centers *= 8.0 / centers.norm(dim=2, keepdim=True)
    big = torch.rand((BH, d), generator=g, device="cuda").argsort(1)[:, :4]
    weights = (torch.arange(C, device="cuda") + 1.0) ** -case["zipf"]

    def keys(rows):
        lab = torch.multinomial(weights, BH * rows, replacement=True, generator=g).view(BH, rows, 1)
        x = normal(BH, rows, d)
        x += centers.gather(1, lab.expand(BH, rows, d))
        x.scatter_(2, big[:, None].expand(BH, rows, 4), 10.0 * x.gather(2, big[:, None].expand(BH, rows, 4)))
        return x.to(dt).view(B, Hkv, rows, d)

    K, V = keys(N), normal(B, Hkv, N, d).to(dt)
    sK, sV = (keys(T), normal(B, Hkv, T, d).to(dt)) if T else (None, None)
    focus = torch.randint(0, C, (BH, 1, 1), generator=g, device="cuda")
    q = centers.gather(1, focus.expand(BH, 1, d)) + 0.5 * normal(BH, Hq // Hkv, d)
    return K, V, sK, sV, q.view(B, Hq, d).contiguous()


class _Owned:
    """A device array of a team table, which it keeps alive."""

    def __init__(self, teams, ptr, shape, typestr):
        self.teams = teams
        self.__cuda_array_interface__ = {"shape": shape, "typestr": typestr, "data": (ptr, False), "version": 3}


def _tables(teams):
    """The arrays of a table, in place (nothing is copied or waited for)."""
    t, BH = teams.desc, (teams.B, teams.Hkv)
    row = "<i2" if teams.torch_dtype == torch.bfloat16 else "<f4"

    def at(ptr, shape, typestr="<i4"):
        return torch.as_tensor(_Owned(teams, ptr, BH + shape, typestr), device="cuda")

    def rows(ptr, n):
        return at(ptr, (n, teams.d), row).view(teams.torch_dtype)

    return {"packed_K": rows(t.packed_K, teams.N), "packed_V": rows(t.packed_V, teams.N), "reps": rows(t.reps, teams.M),
            "team_begin": at(t.team_begin, (teams.M,)), "team_size": at(t.team_size, (teams.M,)),
            "log_n": at(t.log_n, (teams.M,), "<f8"), "rep_token": at(t.rep_token, (teams.M,)),
            "perm": at(t.perm, (teams.N,)), "team_count": at(t.team_count, ())}


def prepare(case, seed):
    K, V, sK, sV, q = _draws(case, seed)
    s = dict(case=case, seed=seed, q=q, sK=sK, sV=sV)
    kind = case["kind"]
    if kind in ("build", "kmeans"):
        s.update(K=K, V=V)
        return s
    s["out"] = torch.empty_like(q)
    if kind == "dense":
        s.update(K=K, V=V, ws=sp.dense_workspace(case["B"], case["Hq"], case["Hkv"], case["N"], case["T"], case["d"]))
        return s
    teams = sp.build_teams(K, V, case["P"], case["R"])
    s["teams"] = teams
    if kind == "decode":
        s["ws"] = sp.decode_workspace(teams, case["Hq"], case["T"], case["K"])
    else:
        s["ws"] = sp.routing_kl_workspace(teams, case["Hq"])
        s["kl"] = [torch.empty(q.shape[:2], dtype=torch.float64, device="cuda") for _ in range(2)]
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "decode":
        return sp.decode(s["teams"], s["q"], s["sK"], s["sV"], case["K"], seed=s["seed"], step=_step(s["seed"]),
                         out=s["out"], workspace=s["ws"])
    if kind == "dense":
        return sp.dense_decode(s["q"], s["K"], s["V"], s["sK"], s["sV"], out=s["out"], workspace=s["ws"])
    if kind == "build":
        return _tables(sp.build_teams(s["K"], s["V"], case["P"], case["R"]))
    if kind == "kmeans":
        labels, parents, steps = sp.kmeans_parents(s["K"], case["P"], seed=s["seed"])
        teams = sp.build_teams_from_labels(s["K"], s["V"], labels, parents, case["R"])
        return {"labels": labels, "parents": parents, "steps": steps, "table": _tables(teams)}
    kl = []
    for kind, out in zip(("representative", "centroid"), s["kl"]):
        sp.set_route_keys(s["teams"], kind)
        kl.append(sp.routing_kl(s["teams"], s["q"], out=out, workspace=s["ws"]))
    return {"representative": kl[0], "centroid": kl[1], "reps": _tables(s["teams"])["reps"]}


def _step(seed):
    return seed % 4096  # which step of its answer the sequence is at


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------


def work(case):
    B, Hq, Hkv, N, d = case["B"], case["Hq"], case["Hkv"], case["N"], case["d"]
    G, row = Hq // Hkv, d * (2 if case["dtype"] == "bf16" else 4)
    pairs, io = B * Hkv, 2 * B * Hq * d * 4
    kind = case["kind"]
    if kind == "dense":
        rows = N + case["T"]
        return {"bytes": pairs * rows * 2 * row + io, "flops": pairs * rows * G * 4 * d}
    M = _team_count(N, case["P"], case["R"])
    if kind == "decode":
        # rows of the union of the G heads' K teams, as if heads sampled
        # independently (measured unions lie on both sides of it)
        rows = N * (1.0 - (1.0 - case["K"] / M) ** G) + case["T"]
        mine = N * case["K"] / M + case["T"]  # rows of one head
        return {"bytes": pairs * (M * row + rows * 2 * row) + io, "flops": pairs * G * (2 * d * M + 4 * d * mine)}
    if kind == "kl":
        # per kind of routing key: keys, routing keys; the centroid pass reads the keys once more
        return {"bytes": pairs * row * (3 * N + 4 * M) + 2 * B * Hq * (4 * d + 8), "flops": pairs * G * 2 * 2 * d * (N + M)}
    table = pairs * (N * (4 * row + 4) + M * (row + 20))  # K, V read and written in team order, the permutation
    if kind == "build":
        return {"bytes": table, "flops": pairs * N * 3 * d * (case["R"] + 2)}  # distances, and the parents' means
    # seeding rounds on its sample, at least a dozen minibatch steps, the labels; then the teams of each parent
    parents = min(N, max(2, N // case["P"]))
    trials, sample = 2 + int(math.log(parents)), min(N, 12288)
    steps = min(12, 100 * N // 4096)
    points = sample * trials * parents + (steps * 4096 + N) * parents
    return {"bytes": table + pairs * (row * (sample + N + steps * 4096) + 8 * N),
            "flops": pairs * (points * 3 * d + N * 3 * d * (case["R"] + 2))}


def tolerance(case):
    if case["kind"] in ("decode", "dense"):
        return {"rel": 8e-6, "max": 2e-4}  # fp32 scores and sums
    if case["kind"] == "kl":
        return {"rel": 1e-12, "max": 1e-10}  # fp64 scores and sums; the routing keys are the same
    return "exact"  # indices, and copies of rows


# ---------------------------------------------------------------------------
# The same results in 64 bits, from torch and numpy alone
# ---------------------------------------------------------------------------


def _mulhi(a, b):
    lo = np.uint64(0xFFFFFFFF)
    s = np.uint64(32)
    a0, a1, b0, b1 = a & lo, a >> s, b & lo, b >> s
    mid = ((a0 * b0) >> s) + ((a0 * b1) & lo) + ((a1 * b0) & lo)
    return a1 * b1 + ((a0 * b1) >> s) + ((a1 * b0) >> s) + (mid >> s)


def _gumbel(case, seed, M):
    """Gumbel noise [B, Hq, M] of a step (Philox4x64-10, key (seed, 0), counter (g / 4, h, b, step), word g mod 4)."""
    B, Hq, blocks = case["B"], case["Hq"], -(-M // 4)
    c = [np.broadcast_to(x, (B, Hq, blocks)).astype(np.uint64) for x in (
        np.arange(blocks), np.arange(Hq)[:, None], np.arange(B)[:, None, None], np.array(_step(seed)))]
    k = [np.uint64(seed), np.uint64(0)]
    m0, m1 = np.uint64(0xD2E7470EE14C6C93), np.uint64(0xCA5A826395121157)
    with np.errstate(over="ignore"):
        for _ in range(10):
            c = [_mulhi(m1, c[2]) ^ c[1] ^ k[0], m1 * c[2], _mulhi(m0, c[0]) ^ c[3] ^ k[1], m0 * c[0]]
            k = [k[0] + np.uint64(0x9E3779B97F4A7C15), k[1] + np.uint64(0xBB67AE8584CAA73B)]
    w = np.stack(c, -1).reshape(B, Hq, 4 * blocks)[:, :, :M]
    u = ((w >> np.uint64(12)).astype(np.float64) + 0.5) * 2.0 ** -52
    return torch.from_numpy(-np.log(-np.log(u))).cuda()


def _teams64(K, P, R):
    """(team of each token [B*Hkv, N], representative token of each team [B*Hkv, M]) of contiguous parents."""
    BH, N, d = K.shape
    team = torch.empty((BH, N), dtype=torch.int64, device=K.device)
    reps, done = [], 0
    for n, count in ((P, N // P), (N % P, 1)):
        if not n or not count:
            continue
        X = K[:, done:done + n * count].view(BH, count, n, d)
        r = min(R, n)

        def dist(c):
            return (X - c).square().sum(-1)

        def member(i):
            return X.gather(2, i[..., None, None].expand(BH, count, 1, d))

        rep = dist(X.mean(2, keepdim=True)).argmin(-1)
        near, own, chosen = torch.full((BH, count, n), math.inf, dtype=X.dtype, device=K.device), None, []
        own = torch.zeros((BH, count, n), dtype=torch.int64, device=K.device)
        for u in range(r):
            dd = dist(member(rep))
            own = torch.where(dd < near, u, own)
            near = torch.minimum(near, dd)
            near.scatter_(2, rep[..., None], -1.0)
            own.scatter_(2, rep[..., None], u)
            chosen.append(rep)
            rep = near.argmax(-1)
        base = done + n * torch.arange(count, device=K.device)
        first = sum(x.shape[1] for x in reps)
        reps.append((torch.stack(chosen, -1) + base[None, :, None]).view(BH, count * r))
        team[:, done:done + n * count] = (own + (first + r * torch.arange(count, device=K.device))[None, :, None]).view(BH, -1)
        done += n * count
    return team, torch.cat(reps, 1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("build", "kmeans"):
        return None  # indices and copies: there is nothing to be nearer to
    K, V, sK, sV, q = _draws(case, seed)
    B, Hq, Hkv, N, d = case["B"], case["Hq"], case["Hkv"], case["N"], case["d"]
    G, BH, scale = Hq // Hkv, B * Hkv, 1.0 / math.sqrt(d)
    K, V, q = K.view(BH, N, d).double(), V.view(BH, N, d).double(), q.view(BH, G, d).double()

    def scores(keys):
        return scale * torch.matmul(q, keys.transpose(1, 2).contiguous())

    def suffix(w, values):
        if sK is None:
            return w, values
        return (torch.cat([w, scores(sK.view(BH, -1, d).double())], 2), torch.cat([values, sV.view(BH, -1, d).double()], 1))

    if kind == "dense":
        w, values = suffix(scores(K), V)
        return torch.matmul(torch.softmax(w, 2), values).view(B, Hq, d)
    team, rep = _teams64(K, case["P"], case["R"])
    M = rep.shape[1]
    size = torch.zeros((BH, M), dtype=torch.float64, device="cuda").scatter_add_(1, team, torch.ones_like(team, dtype=torch.float64))
    rep_keys = K.gather(1, rep[..., None].expand(BH, M, d))
    if kind == "decode":
        phi = scores(rep_keys) + size.log()[:, None]
        Y = phi + _gumbel(case, seed, M).view(BH, G, M)
        top, at = Y.topk(case["K"] + 1, 2)
        logc = torch.log(-torch.expm1(-torch.exp(phi - top[..., -1:])))
        shift = torch.full_like(Y, -math.inf).scatter_(2, at[..., :-1], -logc.gather(2, at[..., :-1]))
        w, values = suffix(scores(K) + shift.gather(2, team[:, None].expand(BH, G, N)), V)
        return torch.matmul(torch.softmax(w, 2), values).view(B, Hq, d)
    logp = torch.log_softmax(scores(K), 2)

    def divergence(keys):
        logq = torch.log_softmax(scores(keys) + size.log()[:, None], 2) - size.log()[:, None]
        return (logp.exp() * (logp - logq.gather(2, team[:, None].expand(BH, G, N)))).sum(2).view(B, Hq)

    mean = torch.zeros((BH, M, d), dtype=torch.float64, device="cuda").scatter_add_(1, team[..., None].expand(BH, N, d), K)
    mean = (mean / size[..., None]).to(_torch_dtype(case)).double()
    return {"representative": divergence(rep_keys), "centroid": divergence(mean), "reps": None}
