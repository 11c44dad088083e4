"""GPU parity of the routing-key variants and the KL routing diagnostic
(section "Attention-distribution diagnostic"; eq. diagnostic-kl) against the
CPU oracle, through the C ABI.

Bars: centroid keys bit-exact (both sides take the fp64 mean in team order
and round it to nearest-even bf16, or to fp32); KL within 1e-9 absolute plus
1e-9 relative (fp64 on both sides, different summation orders); decoding
with centroid keys held to the decode bars of test_gpu_parity."""
import numpy as np
import pytest
import torch

import datagen
import oracle
import paper_2609_35629_amd as sp
from tests.gpu_util import compare_step, dev_batch, gpu_tables, log, oracle_teams

pytestmark = pytest.mark.gpu


def _bits_bf16(vals: np.ndarray) -> np.ndarray:
    """bf16 bit patterns of values that are exact bf16 numbers."""
    return (np.asarray(vals, np.float64).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)


def _oracle_keys(b, ot, kind):
    return [[oracle.routing_keys(b.f64(b.K[bi, kv]), ot[bi][kv], kind, b.wl.dtype)
             for kv in range(b.wl.Hkv)] for bi in range(b.wl.B)]


def _check_keys(teams, b, keys):
    got = teams.reps().cpu()
    for bi in range(b.wl.B):
        for kv in range(b.wl.Hkv):
            if b.wl.dtype == datagen.BF16:
                g = got[bi, kv].view(torch.int16).numpy().view(np.uint16)
                np.testing.assert_array_equal(g, _bits_bf16(keys[bi][kv]), err_msg=f"b={bi} kv={kv}")
            else:
                np.testing.assert_array_equal(got[bi, kv].numpy(), keys[bi][kv].astype(np.float32))


@pytest.mark.parametrize("name", ["qwen8k", "tiny"])
def test_centroid_and_representative_keys(name):
    wl = datagen.WORKLOADS[name]
    log(f"[gpu] route keys {name}")
    b = datagen.generate(wl)
    db = dev_batch(b)
    ot = oracle_teams(b)
    teams = sp.build_teams(db.K, db.V, wl.P, wl.R)
    sp.set_route_keys(teams, "centroid")
    torch.cuda.synchronize()
    _check_keys(teams, b, _oracle_keys(b, ot, "centroid"))
    sp.set_route_keys(teams, "representative")
    torch.cuda.synchronize()
    _check_keys(teams, b, _oracle_keys(b, ot, "representative"))


def test_centroid_rounding_ties():
    # two-token teams (P = 2, R = 1) of bf16 values in [1, 2): the mean of
    # two such values is a rounding tie whenever their sum is odd in the
    # last place, so about half of all key entries exercise ties-to-even
    wl = datagen.WORKLOADS["qwen8k"].with_(name="ties", N=4096, P=2, R=1, Hq=2, Hkv=1)
    b = datagen.generate(wl)
    rng = np.random.default_rng(11)
    mant = rng.integers(0, 128, size=b.K.shape, dtype=np.uint16)
    b.K[...] = np.uint16(0x3F80) | mant  # 1 + m / 128
    log("[gpu] centroid rounding ties")
    db = dev_batch(b)
    ot = oracle_teams(b)
    keys = _oracle_keys(b, ot, "centroid")
    m = oracle.team_means(b.f64(b.K[0, 0]), ot[0][0])
    tie = (oracle.round_to_bf16(m) != m)
    assert tie.mean() > 0.3  # the case really is full of ties
    teams = sp.build_teams(db.K, db.V, wl.P, wl.R)
    sp.set_route_keys(teams, "centroid")
    torch.cuda.synchronize()
    _check_keys(teams, b, keys)


@pytest.mark.parametrize("name", ["qwen8k", "tiny", "limit"])
def test_routing_kl_matches_oracle(name):
    wl = datagen.WORKLOADS[name]
    log(f"[gpu] routing KL {name}")
    b = datagen.generate(wl)
    db = dev_batch(b)
    ot = oracle_teams(b)
    teams = sp.build_teams(db.K, db.V, wl.P, wl.R)
    kinds = ("representative",) if name == "limit" else ("representative", "centroid")
    for kind in kinds:
        sp.set_route_keys(teams, kind)
        kl = sp.routing_kl(teams, db.q, scale=wl.scale)
        torch.cuda.synchronize()
        kl = kl.cpu().numpy()
        keys = _oracle_keys(b, ot, kind)
        for bi in range(wl.B):
            for h in range(wl.Hq):
                kv = h // wl.G
                ref = oracle.routing_kl(b.q[bi, h], b.f64(b.K[bi, kv]), ot[bi][kv], keys[bi][kv], wl.scale)
                assert abs(kl[bi, h] - ref) <= 1e-9 + 1e-9 * abs(ref), (kind, bi, h, kl[bi, h], ref)
        log(f"[gpu]   {kind}: mean KL {kl.mean():.4f} nats")
        if name == "limit":
            # every key its own team: routing equals dense attention
            assert np.abs(kl).max() < 1e-9


def test_decode_with_centroid_keys():
    wl = datagen.WORKLOADS["qwen8k"]
    log("[gpu] decode with centroid routing keys")
    b = datagen.generate(wl)
    db = dev_batch(b)
    ot = oracle_teams(b)
    teams = sp.build_teams(db.K, db.V, wl.P, wl.R)
    sp.set_route_keys(teams, "centroid")
    keys = _oracle_keys(b, ot, "centroid")
    ws = sp.decode_workspace(teams, wl.Hq, wl.T, wl.K)
    dbg = sp.DebugOut(wl.B, wl.Hq, wl.Hkv, teams.M, wl.K)
    out = sp.decode(teams, db.q, db.sK, db.sV, wl.K, seed=wl.seed, step=3, scale=wl.scale, workspace=ws,
                    debug=dbg)
    torch.cuda.synchronize()
    pairs = [(bi, h) for bi in range(wl.B) for h in range(wl.Hq)]
    so = oracle.decode(b.q, b.f32(b.K), b.f32(b.V), b.f32(b.sK), b.f32(b.sV), ot, wl.K, wl.seed, 3,
                       wl.scale, route_keys=keys)
    cmp = compare_step(wl, wl.K, out.cpu().numpy(), dbg, so, pairs, True)
    log(f"[gpu]   sel_equal={cmp.sel_equal}/{cmp.heads} max_rel_l2={cmp.rel_l2.max():.2e} "
        f"max_phi_rel={cmp.max_phi_rel:.1e}")
    assert not cmp.unexcused
    assert cmp.max_phi_rel < 1e-10
    assert cmp.rel_l2.max() <= 1e-2


@pytest.mark.parametrize("dtype,d,Hq,Hkv,N,P,R", [
    ("bf16", 128, 3, 1, 257, 17, 3), ("bf16", 64, 16, 2, 1023, 64, 64), ("fp32", 128, 8, 1, 1000, 300, 5),
    ("fp32", 64, 5, 1, 63, 100, 1), ("bf16", 128, 2, 2, 1, 4, 2), ("bf16", 64, 1, 1, 5000, 1, 1),
])
def test_routing_kl_ragged_shapes(dtype, d, Hq, Hkv, N, P, R):
    # rows past the last 256, teams across its bounds and many teams in it
    wl = datagen.WORKLOADS["qwen8k" if dtype == "bf16" else "tiny"].with_(
        name="kl", d=d, N=N, P=P, R=R, Hq=Hq, Hkv=Hkv, T=0)
    log(f"[gpu] routing KL {dtype} d={d} Hq={Hq} Hkv={Hkv} N={N} P={P} R={R}")
    b = datagen.generate(wl)
    db = dev_batch(b)
    ot = oracle_teams(b)
    teams = sp.build_teams(db.K, db.V, P, R)
    for kind in ("representative", "centroid"):
        sp.set_route_keys(teams, kind)
        kl = sp.routing_kl(teams, db.q).cpu().numpy()
        keys = _oracle_keys(b, ot, kind)
        _check_keys(teams, b, keys)
        for h in range(Hq):
            kv = h // wl.G
            ref = oracle.routing_kl(b.q[0, h], b.f64(b.K[0, kv]), ot[0][kv], keys[0][kv], wl.scale)
            assert abs(kl[0, h] - ref) <= 1e-9 + 1e-9 * abs(ref), (kind, h, kl[0, h], ref)


def test_routing_kl_absent_teams():
    # pairs of unequal team counts: the absent teams' log n excludes them
    wl = datagen.WORKLOADS["qwen8k"].with_(name="kl-lists", N=700, Hq=4, Hkv=2, T=0)
    b = datagen.generate(wl)
    db = dev_batch(b)
    lab = np.random.default_rng(1).integers(0, 9, size=(1, 2, 700)).astype(np.int32)
    lab[0, 1] = np.minimum(lab[0, 1], 3)
    log("[gpu] routing KL with absent teams")
    teams = sp.build_teams_from_labels(db.K, db.V, torch.from_numpy(lab).cuda(), 9, 4)
    kl = sp.routing_kl(teams, db.q).cpu().numpy()
    for h in range(4):
        kv = h // 2
        x = b.f64(b.K[0, kv])
        t = oracle.build_teams_from_labels(x, lab[0, kv], 4)
        ref = oracle.routing_kl(b.q[0, h], x, t, oracle.routing_keys(x, t, "representative", wl.dtype), wl.scale)
        assert abs(kl[0, h] - ref) <= 1e-9 + 1e-9 * abs(ref), (h, kl[0, h], ref)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("fp32", 128), ("fp32", 64)])
def test_centroid_keys_by_team_size(dtype, d):
    # teams of the sizes where the mean's blocks of rows change
    sizes = [1, 2, 3, 4, 5, 8, 9, 16, 17, 31, 32, 33, 48, 49, 64, 65, 300]
    lab = np.random.default_rng(4).permutation(np.repeat(np.arange(len(sizes), dtype=np.int32), sizes))
    wl = datagen.WORKLOADS["qwen8k" if dtype == "bf16" else "tiny"].with_(
        name="sizes", d=d, N=lab.size, Hq=1, Hkv=1, T=0)
    log(f"[gpu] centroid keys by team size {dtype} d={d}")
    b = datagen.generate(wl)
    db = dev_batch(b)
    teams = sp.build_teams_from_labels(db.K, db.V, torch.from_numpy(lab[None, None]).cuda(), len(sizes), 1)
    sp.set_route_keys(teams, "centroid")
    t = oracle.build_teams_from_labels(b.f64(b.K[0, 0]), lab, 1)
    _check_keys(teams, b, [[oracle.routing_keys(b.f64(b.K[0, 0]), t, "centroid", wl.dtype)]])
