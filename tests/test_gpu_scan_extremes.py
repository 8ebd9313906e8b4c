"""Queries and vectors whose estimates meet a threshold exactly, are infinite or are not numbers: every scan has to keep the vectors
that the popcount kernel keeps."""
import numpy as np
import pytest
import torch

from oracle import build
from paper_2602_23999_amd import rabitq

pytestmark = pytest.mark.gpu


def same(a, b):
    return torch.equal(a[0], b[0]) and bool(((a[1] == b[1]) | (a[1].isnan() & b[1].isnan())).all())


def on_every_route(gi, q, k, nprobe):
    """The popcount kernel's result after comparing all others with it."""
    gi.set_option("split_min_pairs", 0)
    gi.set_option("scan_impl", 0)
    want = gi.search(q, k, nprobe)
    D = gi.index_info("dim")
    routes = [(1, -1, (0, 0))]
    if D < 960:
        routes.append((4, 1 << 20, (1, 0)))
    if D <= 256 or D >= 960:
        routes.append((4, 0, (1, 1)))
    for impl, group_min, route in routes:
        gi.set_option("scan_impl", impl)
        gi.set_option("group_min", group_min)
        got = gi.search(q, k, nprobe)
        assert (gi.index_info("last_scan_split"), gi.index_info("last_scan_group")) == route
        bad = [i for i in range(len(q)) if not same([t[i] for t in got], [t[i] for t in want])]
        assert not bad, (impl, route, bad)
    return want


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("D,bits", [(64, 4), (96, 3), (128, 8), (256, 2), (512, 4), (960, 5), (1024, 8)])
def test_queries_at_and_beyond_the_range(D, bits, metric):
    rng = np.random.default_rng(D + bits)
    nlist, n, nq = 5, 1500, 120
    C = rng.standard_normal((nlist, D))
    X = (C[rng.integers(0, nlist, n)] + 0.5 * rng.standard_normal((n, D))).astype(np.float32)
    Q = (C[rng.integers(0, nlist, nq)] + 0.5 * rng.standard_normal((nq, D))).astype(np.float32)
    far = [(1, 1e10), (2, -1e8)]                  # one coordinate: distances that agree in all their bits
    for i, v in far:
        Q[i, 3] = v
    for i, f in ((3, 1e4), (4, 1e7), (5, 1e15), (6, 1e-10), (7, 1e-30), (8, 0.0)):
        Q[i] *= np.float32(f)
    Q[9] = np.nan
    Q[10, 2] = np.nan
    if metric == "l2":                            # (under the inner product these have estimates)
        Q[11] = np.inf
        Q[12, 1] = -np.inf
        Q[13] = 1e30
        Q[14] = -1e25
    gi = rabitq.Index.build(torch.from_numpy(X).cuda(), nlist, bits, build.random_rotation(D, 7), metric=metric, kmeans_iters=2)
    for nprobe in (1, 4):
        ids, d = on_every_route(gi, torch.from_numpy(Q).cuda(), 10, nprobe)
        none = [9, 10] + ([11, 12, 13, 14] if metric == "l2" else [])
        assert bool((ids[none] == -1).all())
        assert bool((ids[15:, 0] >= 0).all())
    gi.close()


@pytest.mark.parametrize("D,bits", [(64, 4), (512, 4), (960, 5)])
def test_lists_of_equal_vectors_and_a_far_query(D, bits):
    # residuals of the size of a rounding error: the bound, the threshold and every distance are the same number
    rng = np.random.default_rng(D)
    base = rng.standard_normal((3, D)).astype(np.float32)
    X = base[rng.integers(0, 3, 900)]
    X[::5] *= np.float32(1 + 2.0 ** -23)
    Q = (base[rng.integers(0, 3, 60)] * rng.choice([1.0, 30.0, 1e3, 1e5], (60, 1))).astype(np.float32)
    gi = rabitq.Index.build(torch.from_numpy(X).cuda(), 3, bits, build.random_rotation(D, 7), kmeans_iters=2)
    ids, _ = on_every_route(gi, torch.from_numpy(Q).cuda(), 10, 1)
    gi.close()


@pytest.mark.parametrize("D,bits", [(64, 4), (128, 8), (512, 4), (960, 5)])
def test_small_numbers(D, bits):
    # squared residuals and their products are below the normal range of 32 bits
    rng = np.random.default_rng(D)
    C = rng.standard_normal((4, D))
    X = (1e-20 * (C[rng.integers(0, 4, 900)] + 0.5 * rng.standard_normal((900, D)))).astype(np.float32)
    Q = (1e-20 * (C[rng.integers(0, 4, 60)] + 0.5 * rng.standard_normal((60, D)))).astype(np.float32)
    gi = rabitq.Index.build(torch.from_numpy(X).cuda(), 4, bits, build.random_rotation(D, 7), kmeans_iters=2)
    on_every_route(gi, torch.from_numpy(Q).cuda(), 10, 2)
    gi.close()


@pytest.mark.parametrize("D,bits", [(64, 4), (96, 8), (512, 4), (960, 5)])
def test_vectors_beyond_the_range(D, bits):
    rng = np.random.default_rng(D)
    nlist = 4
    C = rng.standard_normal((nlist, D))
    X = (C[rng.integers(0, nlist, 1200)] + 0.5 * rng.standard_normal((1200, D))).astype(np.float32)
    Q = (C[rng.integers(0, nlist, 80)] + 0.5 * rng.standard_normal((80, D))).astype(np.float32)
    X[100] = np.inf                               # (the first training rows are the lists' first centroids)
    X[200, 1] = np.nan
    X[300:310] = 1e30
    X[400] *= 1e15
    # (no training pass: the lists' centroids stay numbers)
    gi = rabitq.Index.build(torch.from_numpy(X).cuda(), nlist, bits, build.random_rotation(D, 7), kmeans_iters=0)
    for k in (10, 128):
        on_every_route(gi, torch.from_numpy(Q).cuda(), k, nlist)
    gi.close()
