"""Device blocks of closed tables, kept and given out again: a table built in
the block of another of a different shape, while a step over that one is still
queued on another stream; tables built and closed by several threads; the
bounds on what is kept, and giving it back."""
import threading

import pytest
import torch

import datagen
import paper_2609_35629_amd as sp
from tests.gpu_util import assert_tables_equal, dev_batch, gpu_tables, log, oracle_teams

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _arrays(teams):
    return gpu_tables(teams) + tuple(x.view(torch.uint8).cpu().numpy().tobytes()
                                     for x in (teams.packed_K(), teams.packed_V(), teams.reps(), teams.team_count()))


def test_recycled_block_with_a_step_queued_on_another_stream():
    old = datagen.WORKLOADS["qwen8k"].with_(name="old", N=4096, P=4, R=1, T=5)
    new = datagen.WORKLOADS["tiny"].with_(name="new", Hq=6, Hkv=3, N=5300, d=64, P=190, R=7, T=0)
    bo, bn = datagen.generate(old), datagen.generate(new)
    do, dn = dev_batch(bo), dev_batch(bn)
    ot = oracle_teams(bn)
    teams = sp.build_teams(do.K, do.V, old.P, old.R)
    ws = sp.decode_workspace(teams, old.Hq, old.T, old.K)
    want = sp.decode(teams, do.q, do.sK, do.sV, old.K, workspace=ws)
    teams.close()
    sp.trim()
    side = torch.cuda.Stream()
    x = torch.randn(4096, 4096, device="cuda")
    for labels in (False, True):
        log(f"[gpu] recycled block labels={labels}")
        teams = sp.build_teams(do.K, do.V, old.P, old.R)
        out = torch.empty_like(want)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(20):
                x @ x
            sp.decode(teams, do.q, do.sK, do.sV, old.K, out=out, workspace=ws)
        before = teams.desc.packed_K
        teams.close()
        if labels:  # contiguous parents as labels: the general build, its scratch from the pool too
            lab = (torch.arange(new.N, device="cuda", dtype=torch.int32) // new.P).expand(1, 3, new.N).contiguous()
            got = sp.build_teams_from_labels(dn.K, dn.V, lab, -(-new.N // new.P), new.R)
        else:
            got = sp.build_teams(dn.K, dn.V, new.P, new.R)
            assert got.desc.packed_K == before  # the old table's block
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        for kv in range(3):
            assert_tables_equal(gpu_tables(got), ot, 0, kv)
        got.close()


def test_threads_build_and_close():
    cases = [(1024, 16, 4), (3000, 1100, 5), (777, 50, 50), (4096, 1024, 16)]
    data, want = [], []
    for n, p, r in cases:
        K = torch.randn((1, 2, n, 64), device="cuda").bfloat16()
        data.append(K)
        t = sp.build_teams(K, -K, p, r)
        want.append(_arrays(t)[4:])
        t.close()
    log("[gpu] threads build and close tables")
    bad = []

    def work(k):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for i in range(24):
                c = (i + k) % len(cases)
                n, p, r = cases[c]
                t = sp.build_teams(data[c], -data[c], p, r)
                if _arrays(t)[4:] != want[c]:
                    bad.append((k, i, c))
                t.close()

    torch.cuda.synchronize()
    th = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not bad


def test_bounds_and_trim():
    sp.trim()
    K = torch.randn((1, 2, 131072, 64), device="cuda").bfloat16()  # tables of 65 MiB
    sp.build_teams(K, K, 1024, 16).close()
    sp.trim()
    base = _free()
    log("[gpu] blocks kept and given back")
    tables = [sp.build_teams(K, K, 1024, 16) for _ in range(20)]
    used = base - _free()
    assert used >= 20 * 64 * MIB
    for t in tables:
        t.close()
    kept = base - _free()
    assert 0 < kept <= 1024 * MIB + 64 * MIB
    sp.trim()
    assert base - _free() <= 4 * MIB
    small = K[:, :, :2048].contiguous()  # tables of 1 MiB: at most 16 blocks
    tables = [sp.build_teams(small, small, 1024, 16) for _ in range(40)]
    for t in tables:
        t.close()
    assert base - _free() <= 16 * 3 * MIB
    sp.trim()
    assert base - _free() <= 4 * MIB
