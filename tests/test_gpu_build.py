"""Team tables at the edges of the build kernel: parents around the sizes
where members per thread and rows in registers change, and keys whose fp32
distance estimates cannot decide a choice (exact ties, near ties, norms
outside the estimate's range).  Every table equals the oracle's exactly: each
choice is made on the definition's fp64 distances wherever the estimates
leave more than one candidate."""
import numpy as np
import pytest
import torch

import datagen
import oracle
import paper_2609_35629_amd as sp
from tests.gpu_util import assert_tables_equal, dev_batch, gpu_tables, log, oracle_teams, to_dev

pytestmark = pytest.mark.gpu


def _keys(kind, N, d, dtype, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((1, 2, N, d))
    if kind == "lattice":        # few distinct distances: ties at every choice
        x = rng.integers(-1, 2, size=x.shape).astype(np.float64)
    elif kind == "few":          # at most five distinct rows
        x = x[:, :, rng.integers(0, 5, size=N)]
    elif kind == "equal":
        x = np.broadcast_to(x[:, :, :1], x.shape)
    elif kind == "zero":
        x = np.zeros_like(x)
    elif kind == "close":        # distances far below the norms' rounding in fp32
        x = 8.0 + 2.0 ** -6 * x
    elif kind == "huge":         # squared norms past fp32's range
        x = 1e22 * x
    elif kind == "small":        # squares below fp32's normal range
        x = 1e-24 * x
    elif kind == "mixed":        # norms far apart within one parent
        x = x * 10.0 ** rng.uniform(-6, 6, size=(1, 2, N, 1))
    x = x.astype(np.float32)
    return datagen.round_bf16_bits(x) if dtype == datagen.BF16 else x


def _widen(K, dtype):
    return (datagen.bf16_bits_to_f32(K) if dtype == datagen.BF16 else K).astype(np.float64)


KINDS = ["normal", "lattice", "few", "equal", "zero", "close", "huge", "small", "mixed"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("dtype,d,N,P,R", [
    ("bf16", 128, 300, 140, 6), ("bf16", 64, 50, 17, 20), ("fp32", 128, 300, 150, 5), ("fp32", 64, 1300, 1100, 4),
])
def test_hard_keys_match_oracle(kind, dtype, d, N, P, R):
    log(f"[gpu] build keys={kind} {dtype} d={d} N={N} P={P} R={R}")
    K = _keys(kind, N, d, dtype, 3)
    Kd = to_dev(K, dtype)
    x = _widen(K, dtype)
    teams = sp.build_teams(Kd, Kd, P, R)
    torch.cuda.synchronize()
    gt = gpu_tables(teams)
    lab = np.random.default_rng(5).integers(0, 3, size=(1, 2, N)).astype(np.int32)
    lists = sp.build_teams_from_labels(Kd, Kd, torch.from_numpy(lab).cuda(), 3, R)
    torch.cuda.synchronize()
    gl = gpu_tables(lists)
    for kv in range(2):
        assert_tables_equal(gt, [[oracle.build_teams(x[0, k], P, R) for k in range(2)]], 0, kv)
        t = oracle.build_teams_from_labels(x[0, kv], lab[0, kv], R)
        np.testing.assert_array_equal(gl[0][0, kv], t.members)
        np.testing.assert_array_equal(gl[1][0, kv, :t.M], t.team_ptr[:-1])
        np.testing.assert_array_equal(gl[3][0, kv, :t.M], t.rep_token)


@pytest.mark.parametrize("kind", ["few", "equal", "pad", "outlier", "offset", "late", "huge"])
@pytest.mark.parametrize("dtype,d,N,P,R", [
    ("bf16", 128, 2100, 1024, 9), ("bf16", 64, 1500, 1000, 70), ("fp32", 64, 2100, 1024, 9), ("fp32", 128, 1024, 1024, 5),
    ("bf16", 128, 330, 150, 12), ("fp32", 64, 200, 100, 3),
])
def test_open_parents_match_oracle(kind, dtype, d, N, P, R):
    """Parents with more candidates at one choice than the estimates' kernel
    compares (64), from the first choice or after some rounds: the second build
    kernel goes on from the representatives found."""
    log(f"[gpu] build open parents keys={kind} {dtype} d={d} N={N} P={P} R={R}")
    rng = np.random.default_rng(9)
    x = rng.standard_normal((1, 2, N, d))
    if kind in ("few", "equal"):
        x = x[:, :, rng.integers(0, 5 if kind == "few" else 1, size=N)]
    elif kind == "pad":
        x[:, :, N // 2:] = 0.0
    elif kind == "outlier":
        x[:, :, ::P] *= 300.0
    elif kind == "offset":
        x += 300.0
    elif kind == "late":  # distinct far rows first, then copies of a nearer one
        x = 0.01 * x
        x[:, :, ::3] = rng.standard_normal((1, 2, 1, d))
        far = rng.integers(0, N, size=(N + P - 1) // P * 3)
        x[:, :, far] = 5.0 * rng.standard_normal((1, 2, far.size, d))
    else:
        x *= 1e22
    K = x.astype(np.float32)
    K = datagen.round_bf16_bits(K) if dtype == "bf16" else K
    Kd = to_dev(K, dtype)
    x = _widen(K, dtype)
    teams = sp.build_teams(Kd, -Kd, P, R)
    torch.cuda.synchronize()
    gt = gpu_tables(teams)
    as_int = torch.int16 if dtype == "bf16" else torch.int32
    for kv in range(2):
        assert_tables_equal(gt, [[oracle.build_teams(x[0, k], P, R) for k in range(2)]], 0, kv)
        perm, rt = torch.from_numpy(gt[0][0, kv]).long().cuda(), torch.from_numpy(gt[3][0, kv]).long().cuda()
        for got, src, idx in ((teams.packed_K(), Kd, perm), (teams.packed_V(), -Kd, perm), (teams.reps(), Kd, rt)):
            assert torch.equal(got.view(as_int)[0, kv], src.view(as_int)[0, kv][idx])
    if R < P:  # a step over the table: the chunk capacities are those of the finished one
        q = torch.randn((1, 4, d), device="cuda")
        out = sp.decode(teams, q, None, None, min(4, teams.M - 1), seed=1, step=1, scale=0.01)
        assert torch.isfinite(out).all()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("fp32", 128), ("fp32", 64)])
@pytest.mark.parametrize("N,P,R", [
    (97, 1, 1), (97, 15, 4), (160, 16, 4), (161, 17, 3), (200, 64, 64), (195, 65, 8),
    (1024, 1024, 16), (1023, 1024, 3), (1090, 1025, 5), (2500, 2100, 70), (1, 8, 2),
])
def test_parent_sizes_match_oracle(dtype, d, N, P, R):
    base = "qwen8k" if dtype == "bf16" else "tiny"
    wl = datagen.WORKLOADS[base].with_(name="sizes", d=d, N=N, P=P, R=R, Hq=2, Hkv=2, T=0)
    log(f"[gpu] build {dtype} d={d} N={N} P={P} R={R}")
    b = datagen.generate(wl)
    db = dev_batch(b)
    ot = oracle_teams(b)
    teams = sp.build_teams(db.K, db.V, P, R)
    torch.cuda.synchronize()
    gt = gpu_tables(teams)
    as_int = torch.int16 if dtype == "bf16" else torch.int32
    for kv in range(2):
        assert_tables_equal(gt, ot, 0, kv)
        perm, rt = torch.from_numpy(gt[0][0, kv]).long().cuda(), torch.from_numpy(gt[3][0, kv]).long().cuda()
        for got, src, idx in ((teams.packed_K(), db.K, perm), (teams.packed_V(), db.V, perm), (teams.reps(), db.K, rt)):
            assert torch.equal(got.view(as_int)[0, kv], src.view(as_int)[0, kv][idx])


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp32", 128), ("fp32", 64)])
def test_long_lists_match_oracle(dtype, d):
    # one parent past one member per thread, one at it, a single member
    N = 2300
    base = "qwen8k" if dtype == "bf16" else "tiny"
    wl = datagen.WORKLOADS[base].with_(name="lists", d=d, N=N, Hq=2, Hkv=2, T=0)
    b = datagen.generate(wl)
    db = dev_batch(b)
    lab = np.repeat(np.array([0, 2, 3], np.int32), [1275, 1024, 1])
    lab = np.stack([np.random.default_rng(k).permutation(lab) for k in range(2)])[None]
    log(f"[gpu] build long lists {dtype} d={d}")
    teams = sp.build_teams_from_labels(db.K, db.V, torch.from_numpy(lab).cuda(), 5, 9)
    torch.cuda.synchronize()
    perm, tb, ts, rt = gpu_tables(teams)
    for kv in range(2):
        t = oracle.build_teams_from_labels(b.f64(b.K[0, kv]), lab[0, kv], 9)
        np.testing.assert_array_equal(perm[0, kv], t.members)
        np.testing.assert_array_equal(tb[0, kv, :t.M], t.team_ptr[:-1])
        np.testing.assert_array_equal(ts[0, kv, :t.M], t.sizes)
        np.testing.assert_array_equal(rt[0, kv, :t.M], t.rep_token)
