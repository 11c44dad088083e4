"""The sampling launch that keeps scores in memory (tables of more than 1200
teams, budgets up to 144, at most half as many heads as compute units, and a
workspace that holds the scores) against the oracle and against the
sampling kernel that a smaller workspace takes: the same teams, tau and log c
for budgets at the edges of its ranking (64 listed teams) and on both sides of
its limit, for the largest table, where scores lie close for their size, and
where absent teams tie.  (Larger budgets take the other kernel in either
workspace.)"""
import numpy as np
import pytest
import torch

import datagen
import oracle
import paper_2609_35629_amd as sp
from tests.gpu_util import compare_step, dev_batch, log, oracle_teams

pytestmark = pytest.mark.gpu


def _small_workspace(teams, db, wl, K):
    """The least workspace that the step takes (refused sizes launch nothing)."""
    full = sp.decode_workspace(teams, wl.Hq, wl.T, K)
    lo, hi = 0, full.numel() // 256
    while lo + 1 < hi:
        mid = (lo + hi) // 2
        try:
            sp.decode(teams, db.q, db.sK, db.sV, K, workspace=full[:256 * mid])
            hi = mid
        except sp.SantappError as e:
            assert e.status == sp._lib.EWORKSPACE
            lo = mid
    assert 256 * hi < full.numel()
    return full, full[:256 * hi]


@pytest.mark.parametrize("dtype,d,Hq,Hkv,N,P,R,budgets", [
    ("bf16", 128, 7, 1, 1032, 1, 1, (1, 63, 64, 255, 256, 1031)),
    ("bf16", 64, 16, 2, 4100, 16, 4, (32, 65, 130, 300, 1023)),
    ("fp32", 128, 5, 1, 2051, 4, 2, (31, 128, 700)),
    ("fp32", 64, 8, 1, 2561, 2, 1, (40, 1200)),
    ("bf16", 128, 8, 1, 8192, 1, 1, (33, 200, 4000)),
    ("bf16", 64, 8, 1, 8192, 4, 2, (128, 144, 145)),
])
def test_budgets_match_oracle_and_small_workspace(dtype, d, Hq, Hkv, N, P, R, budgets):
    wl = datagen.WORKLOADS["qwen8k" if dtype == "bf16" else "tiny"].with_(
        name="sampling", d=d, Hq=Hq, Hkv=Hkv, N=N, P=P, R=R, T=5)
    b = datagen.generate(wl)
    db = dev_batch(b)
    ot = oracle_teams(b)
    teams = sp.build_teams(db.K, db.V, P, R)
    assert teams.M > 1024
    pairs = [(0, h) for h in range(Hq)]
    for K in budgets:
        log(f"[gpu] sampling {dtype} d={d} Hq={Hq} Hkv={Hkv} M={teams.M} K={K}")
        full, small = _small_workspace(teams, db, wl, K)
        got = []
        for ws in (full, small):
            dbg = sp.DebugOut(1, Hq, Hkv, teams.M, K)
            out = sp.decode(teams, db.q, db.sK, db.sV, K, seed=11, step=K, workspace=ws, debug=dbg)
            torch.cuda.synchronize()
            got.append((out.cpu().numpy(), dbg))
        so = oracle.decode(b.q, b.f64(b.K), b.f64(b.V), b.f64(b.sK), b.f64(b.sV), ot, K, 11, K, wl.scale, heads=pairs)
        for out, dbg in got:
            cmp = compare_step(wl, K, out, dbg, so, pairs, True)
            cmp.assert_selection_bar()
            assert cmp.rel_l2_equal.max() <= 1e-4
            assert cmp.max_logc_abs <= 1e-5 and cmp.max_tau_rel_equal <= 1e-12
        assert torch.equal(got[0][1].sel, got[1][1].sel)
        assert torch.equal(got[0][1].union_teams, got[1][1].union_teams)
        assert torch.equal(got[0][1].union_rows, got[1][1].union_rows)


@pytest.mark.parametrize("offset", [0.0, 200.0, 5000.0, 2e7])
@pytest.mark.parametrize("dtype,d,N,budgets", [("bf16", 128, 8192, (100, 144, 145)), ("fp32", 64, 1500, (20, 144))])
def test_scores_close_for_their_size(dtype, d, N, budgets, offset):
    """Equal keys, so that scores are `offset` plus the noise: from some offset on
    more than 256 teams share the upper half of their fp32 score with rank K, then
    the whole fp32 score, and only the fp64 scores tell them apart."""
    wl = datagen.WORKLOADS["qwen8k" if dtype == "bf16" else "tiny"].with_(
        name="close", d=d, Hq=4, Hkv=2, N=N, P=1, R=1, T=0)
    b = datagen.generate(wl)
    b.K[:] = b.K[:, :, :1]
    dot = (b.q.astype(np.float64).reshape(1, 2, 2, d) * b.f64(b.K[:, :, :1])).sum(-1)
    b.q[:] = (b.q.reshape(1, 2, 2, d) / dot[..., None]).reshape(1, 4, d)  # q . k = 1
    scale = max(offset, 1e-3)
    db = dev_batch(b)
    teams = sp.build_teams(db.K, db.V, 1, 1)
    ot = oracle_teams(b)
    pairs = [(0, h) for h in range(4)]
    for K in budgets:
        log(f"[gpu] close scores {dtype} d={d} M={teams.M} K={K} offset={offset}")
        full, small = _small_workspace(teams, db, wl, K)
        so = oracle.decode(b.q, b.f64(b.K), b.f64(b.V), b.f64(b.sK), b.f64(b.sV), ot, K, 7, K, scale, heads=pairs)
        for ws in (full, small):
            dbg = sp.DebugOut(1, 4, 2, teams.M, K)
            out = sp.decode(teams, db.q, None, None, K, seed=7, step=K, scale=scale, workspace=ws, debug=dbg)
            torch.cuda.synchronize()
            sel, o = dbg.sel.cpu().numpy()[0], out.cpu().numpy()[0]
            for h in range(4):
                np.testing.assert_array_equal(sel[h], so.heads[0][h].sel)
                assert oracle.rel_l2(o[h], so.heads[0][h].out) <= 1e-4


def test_absent_teams_tie():
    # one pair with fewer real teams than the budget: every real team is taken,
    # and equal absent ones fill the sample in team order
    wl = datagen.WORKLOADS["qwen8k"].with_(name="absent", N=3000, Hq=4, Hkv=2, T=3)
    b = datagen.generate(wl)
    db = dev_batch(b)
    rng = np.random.default_rng(2)
    lab = np.stack([rng.integers(0, 400, size=3000), rng.integers(0, 20, size=3000)])[None].astype(np.int32)
    teams = sp.build_teams_from_labels(db.K, db.V, torch.from_numpy(lab).cuda(), 400, 3)
    count = teams.team_count().cpu().numpy()[0]
    K = 100
    assert teams.M > 1024 and count[1] <= K < count[0]
    log(f"[gpu] absent teams M={teams.M} counts={count.tolist()} K={K}")
    dbg = sp.DebugOut(1, 4, 2, teams.M, K)
    out = sp.decode(teams, db.q, db.sK, db.sV, K, seed=3, step=1, scale=wl.scale, debug=dbg).cpu().numpy()
    sel = dbg.sel.cpu().numpy()[0]
    for h in (2, 3):
        np.testing.assert_array_equal(sel[h], np.arange(K))
        ref = oracle.dense(b.q[:, h:h + 1], b.f32(b.K)[:, 1:], b.f32(b.V)[:, 1:], b.f32(b.sK)[:, 1:], b.f32(b.sV)[:, 1:],
                           wl.scale)[0, 0]
        assert oracle.rel_l2(out[0, h], ref) <= 1e-4
    assert (sel[:2] < count[0]).all()


def test_graph_replays_and_shared_workspace():
    # a captured step brings the same token at every replay; between replays
    # other steps (another budget, and one over every team) use its workspace
    wl = datagen.WORKLOADS["qwen8k"].with_(name="replay", N=4104, P=4, R=1, Hq=8, Hkv=2, T=4)
    b = datagen.generate(wl)
    db = dev_batch(b)
    teams = sp.build_teams(db.K, db.V, wl.P, wl.R)
    assert teams.M > 1024
    n = max(sp.decode_workspace(teams, wl.Hq, wl.T, k).numel() for k in (32, 300, teams.M))
    ws = torch.zeros(n, dtype=torch.uint8, device="cuda")
    want = sp.decode(teams, db.q, db.sK, db.sV, 32, seed=1, step=2)
    other = {k: sp.decode(teams, db.q, db.sK, db.sV, k, seed=1, step=2) for k in (300, teams.M)}
    out = torch.empty_like(want)
    sp.decode(teams, db.q, db.sK, db.sV, 32, seed=1, step=2, out=out, workspace=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sp.decode(teams, db.q, db.sK, db.sV, 32, seed=1, step=2, out=out, workspace=ws)
    log("[gpu] graph replays of a step with scores in memory")
    for _ in range(4):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        for k, ref in other.items():
            got = sp.decode(teams, db.q, db.sK, db.sV, k, seed=1, step=2, workspace=ws)
            torch.cuda.synchronize()
            assert torch.equal(got, ref)


def test_rule_by_teams_and_heads():
    # the scores' regions come in past 1024 teams, and only while the heads
    # take at most half the compute units
    half = torch.cuda.get_device_properties(0).multi_processor_count // 2
    for B, keys in ((1, True), (half // 4, True), (half // 4 + 1, False)):
        size = []
        for N in (1024, 1025):
            log(f"[gpu] sampling rule B={B} Hq=4 M={N}")
            K = torch.randn((B, 1, N, 64), device="cuda").bfloat16()
            teams = sp.build_teams(K, K, 1, 1)
            assert teams.M == N
            size.append(sp.decode_workspace(teams, 4, 0, 8).numel())
        assert (size[1] - size[0] > 20 * B * 4 * 1024) == keys
