"""Nearest-center choice of the k-means parents where its fp32 estimates cannot
decide: equal keys and centers (ties go to the lower center), zero keys, keys
whose squares leave fp32's range on either side, more centers than one tile of
32, and token counts around a workgroup's 64 points.  Labels and steps are
compared with the oracle bit for bit: where an estimate leaves the choice open
the definition's fp64 distances take it, so nothing has a tolerance.  Also a
seeding sample and a batch past what one load per thread and lane covers, and
member lists by label bits at the smallest and largest label counts.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_35629_amd as sp
from tests.gpu_util import gpu_tables, log

pytestmark = pytest.mark.gpu


def _keys(kind, N, d, dtype):
    g = np.random.default_rng(N + d)
    x = g.standard_normal((N, d))
    if kind == "grid":  # few distinct rows: tied centers and points
        x = np.sign(x) * (np.arange(d) < 3)
    elif kind == "copies":  # near copies of two rows, apart by less than the estimates resolve
        x = x[np.arange(N) % 2] + 2.0**-7 * (g.integers(0, 3, (N, d)) - 1) * (np.arange(d) < 2)
    elif kind == "zeros":
        x[:] = 0.0
    elif kind == "half_zero":
        x[np.arange(N) % 3 != 0] = 0.0
    elif kind == "huge":
        x *= 1e22
    elif kind == "tiny":
        x *= 1e-25
    elif kind == "mixed":
        x *= 10.0 ** g.integers(-22, 22, (N, 1))
    return torch.from_numpy(x).to(dtype)


@pytest.mark.parametrize("kind,N,P,d,dtype", [
    ("normal", 65, 16, 128, torch.bfloat16),
    ("normal", 2113, 64, 64, torch.float32),
    ("normal", 1500, 20, 128, torch.float32),  # 75 centers: three tiles, the last ragged
    ("normal", 63, 63, 64, torch.bfloat16),  # two centers
    ("huge", 63, 63, 64, torch.float32),  # two centers, no estimate
    ("grid", 500, 30, 128, torch.bfloat16),
    ("grid", 500, 13, 64, torch.float32),
    ("copies", 640, 80, 64, torch.float32),
    ("copies", 640, 64, 128, torch.bfloat16),
    ("zeros", 200, 40, 128, torch.bfloat16),
    ("half_zero", 300, 30, 64, torch.bfloat16),
    ("huge", 400, 50, 128, torch.float32),
    ("tiny", 400, 50, 64, torch.float32),
    ("mixed", 400, 25, 128, torch.float32),
])
def test_labels_match_oracle(kind, N, P, d, dtype):
    x = _keys(kind, N, d, dtype)
    log(f"[gpu] kmeans assign {kind} N={N} P={P} d={d} {dtype}")
    th = oracle.KMeansSettings(batch=200, max_iter=12)
    labels, _, steps = sp.kmeans_parents(x[None, None].cuda(), P, batch_size=th.batch, max_iter=th.max_iter)
    r = oracle.kmeans_parents(x.to(torch.float64).numpy(), P, th)
    assert steps[0] == r.steps
    np.testing.assert_array_equal(labels.cpu().numpy()[0, 0], r.labels)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_large_sample_and_batch(dtype):
    # 18000 sample positions: 18 per thread, past the 16 kept in registers;
    # 6000 batch points: 94 inertia partials
    log(f"[gpu] kmeans large sample {dtype}")
    x = _keys("normal", 20000, 64, dtype)
    th = oracle.KMeansSettings(batch=6000, max_iter=1)
    labels, _, steps = sp.kmeans_parents(x[None, None].cuda(), 4000, batch_size=th.batch, max_iter=th.max_iter)
    r = oracle.kmeans_parents(x.to(torch.float64).numpy(), 4000, th)
    assert steps[0] == r.steps
    np.testing.assert_array_equal(labels.cpu().numpy()[0, 0], r.labels)


@pytest.mark.parametrize("num", [1, 2, 63, 64, 65, 1024])
@pytest.mark.parametrize("N", [1, 64, 1025, 9001])
def test_member_lists_by_label_bits(num, N):
    log(f"[gpu] member lists labels={num} N={N}")
    x = _keys("normal", N, 64, torch.float32)
    lab = np.random.default_rng(num).integers(0, num, N).astype(np.int32)
    K = x[None, None].cuda()
    perm, tb, ts, rt = gpu_tables(sp.build_teams_from_labels(K, K, torch.from_numpy(lab)[None, None].cuda(), num, 2))
    t = oracle.build_teams_from_labels(x.to(torch.float64).numpy(), lab, 2)
    np.testing.assert_array_equal(perm[0, 0], t.members)
    np.testing.assert_array_equal(tb[0, 0, :t.M], t.team_ptr[:-1])
    np.testing.assert_array_equal(ts[0, 0, :t.M], t.sizes)
    np.testing.assert_array_equal(rt[0, 0, :t.M], t.rep_token)


@pytest.mark.parametrize("kind,N,P,d,dtype", [
    ("huge", 1500, 20, 128, torch.bfloat16),  # 75 centers: five tiles of 16, the last ragged
    ("huge", 700, 41, 64, torch.float32),  # 17 centers
    ("offset", 640, 40, 64, torch.float32),
    ("offset", 640, 20, 128, torch.bfloat16),
    ("some", 900, 30, 128, torch.float32),
])
def test_points_compared_with_every_center(kind, N, P, d, dtype):
    """Workgroups where most points, or a few, are left open by the estimates:
    compared with all centers together, or half a wave each."""
    x = _keys("huge" if kind == "huge" else "normal", N, d, dtype).float()
    if kind == "offset":
        x += 200.0
    elif kind == "some":
        x[::40] *= 1e20
    x = x.to(dtype)
    log(f"[gpu] kmeans assign all centers {kind} N={N} P={P} d={d} {dtype}")
    th = oracle.KMeansSettings(batch=200, max_iter=12)
    labels, _, steps = sp.kmeans_parents(x[None, None].cuda(), P, batch_size=th.batch, max_iter=th.max_iter)
    r = oracle.kmeans_parents(x.to(torch.float64).numpy(), P, th)
    assert steps[0] == r.steps
    np.testing.assert_array_equal(labels.cpu().numpy()[0, 0], r.labels)
