"""Threshold seeding at the sizes where its selection can go wrong: list lengths around a tile, around the tiles held
in registers and beyond the list in LDS; k around the number of seeds (32), a wavefront (64) and the largest (128);
queries sharing a workgroup (few) and having a wavefront each (more than 2048); equal estimates."""
import numpy as np
import pytest
import torch

from oracle import build, search
from paper_2602_23999_amd import rabitq

from gpu_helpers import key_scale, oracle_stages, to_dev, upload

pytestmark = pytest.mark.gpu


def seeds_near_tie(s, st, i, k):
    """Is the last seed of query i (B = 1: the k-th estimate) within rounding of the 1-bit estimate of another vector
    that is not its copy?  Only then may fp32 take other seeds than the oracle."""
    ix = s.ix
    scale = key_scale(st["G"], st["E"], s.metric)[i]
    for c, G, E in zip(st["probes"][i], st["G"][i], st["E"][i]):
        if ix["offsets"][c + 1] - ix["offsets"][c] < k:
            continue
        e = np.sort(s.pair(c, G, E, st["Qr"][i], st["delta"][i], st["planes"][i], int(st["S"][i]))[3])
        last = e[min(k if s.B == 1 else max(k, s.seed_m), len(e)) - 1]
        d = np.abs(e - last)
        return bool(np.any((d > 0) & (d <= 1e-5 * (abs(last) + scale))))
    return False


def check_thresholds(s, st, k, tau):
    want = np.minimum(st["tau"], np.float64(np.finfo(np.float32).max))
    off = np.abs(tau - want) > 1e-4 * (np.abs(want) + key_scale(st["G"], st["E"], s.metric))
    assert all(seeds_near_tie(s, st, i, k) for i in np.nonzero(off)[0]), (k, tau, want)


@pytest.mark.parametrize("size", [128, 191, 1023, 1025, 5000])
@pytest.mark.parametrize("D,B", [(128, 4), (64, 1), (256, 5), (512, 3)])
def test_seeding_selects_what_the_oracle_selects(D, B, size):
    nq = 5
    rng = np.random.default_rng(D + size)
    X = rng.standard_normal((size + 40, D)).astype(np.float32)
    X[-40:] += 50.0                      # a second list, far away and shorter than most k
    X[7:size:11] = X[5]                  # equal vectors: their 1-bit estimates tie, the lower position wins
    C = np.stack([X[:-40].mean(0), X[-40:].mean(0)])
    ix = build.build_index(X, 2, B, centroids=C)
    s, gi = search.Searcher(ix), upload(ix)
    Q = (0.5 * rng.standard_normal((nq, D)) + X[5]).astype(np.float32)
    reps = 2100 // nq
    for k in (1, 31, 33, 64, 65, 100, 128):
        st = oracle_stages(s, Q, k, 2)
        d = to_dev(st)
        few = gi.seed_threshold(d["prep"], d["probes"], k)
        many = gi.seed_threshold({n: t.repeat((reps,) + (1,) * (t.dim() - 1)) for n, t in d["prep"].items()},
                                 {n: t.repeat(reps, 1) for n, t in d["probes"].items()}, k)
        assert torch.equal(many, few.repeat(reps)), k     # both forms of the kernel, bit for bit
        check_thresholds(s, st, k, few.cpu().numpy())
    gi.close()


@pytest.mark.parametrize("payload", [0x7fc00000, 0x7fffffff])
@pytest.mark.parametrize("B,good", [(4, 5), (4, 60), (1, 60)])
def test_fewer_numbers_than_k_give_no_threshold(B, good, payload):
    # factors that are NaN (of any payload) rank last among the seeds; where the k-th is one, nothing is filtered out
    # (1-bit codes: the threshold is that NaN itself), whatever the smaller ones are
    D, size, k = 64, 300, 64
    rng = np.random.default_rng(good)
    X = rng.standard_normal((size, D)).astype(np.float32)
    ix = build.build_index(X, 1, B, centroids=X.mean(0, keepdims=True).astype(np.float64))
    dev = build.pack_device_layout(ix)
    nan = np.uint32(payload).view(np.float32)
    if B == 1:
        f = dev["short_factors"].reshape(-1, 3, 64)
        for s in range(good, size):
            f[s // 64, 0, s % 64] = nan
    else:
        dev["long_factors"].reshape(-1, 2)[good:size, 0] = nan
    gi = rabitq.index_from_arrays(ix, dev)
    q = torch.from_numpy(X[:7] + np.float32(0.1)).cuda()
    for n in (7, 2100):
        g = q.repeat(n // 7, 1)
        q_rot = gi.rotate(g)
        prep = gi.query_prep(q_rot)
        tau = gi.seed_threshold(prep, gi.coarse_probe(q_rot, prep["sq_norm"], 1), k).cpu().numpy()
        assert np.all(np.isnan(tau)) if B == 1 else np.all(tau == np.finfo(np.float32).max), tau[:7]
    gi.close()


@pytest.mark.parametrize("size", [700, 5000])
@pytest.mark.parametrize("k", [1, 10, 40, 64, 65, 128])
def test_of_equal_estimates_the_lower_positions_are_seeds(k, size):
    # most of the list has one 1-bit code and the same factors of it, but long codes of their own: the seeds, and with
    # them the threshold, depend on which of the equals are taken
    D, B, near = 64, 4, 9
    rng = np.random.default_rng(size + k)
    X = rng.standard_normal((size, D)).astype(np.float32)
    ix = build.build_index(X, 1, B, centroids=X.mean(0, keepdims=True).astype(np.float64))
    sign = 1 << (B - 1)
    few = rng.permutation(size)[:size // 7]                   # the others: `near` below the equals, the rest above
    same = np.setdiff1d(np.arange(size), few)
    ix["u"][same] = (ix["u"][same[0]] & sign) | (ix["u"][same] & (sign - 1))
    ix["short_factors"][same] = ix["short_factors"][same[0]]
    ix["short_factors"][few[:near], 0] -= 1000.0
    ix["short_factors"][few[near:], 0] += 1000.0
    s, gi = search.Searcher(ix), upload(ix)
    Q = X[same[:15]] + np.float32(0.1)
    st = oracle_stages(s, Q, k, 1)
    d = to_dev(st)
    scale = key_scale(st["G"], st["E"], s.metric)
    m = max(k, s.seed_m)
    assert near < m < near + len(same)
    other = [np.sort(s.refined(0, size, st["G"][i, 0], st["Qr"][i], np.concatenate([few[:near], same[-(m - near):]])))[k - 1]
             for i in range(len(Q))]
    tol = 1e-5 * (np.abs(st["tau"]) + scale)
    assert np.any(np.abs(other - st["tau"]) > 2 * tol)          # another choice among the equals would show
    for reps in (1, 140):
        tau = gi.seed_threshold({n: t.repeat((reps,) + (1,) * (t.dim() - 1)) for n, t in d["prep"].items()},
                                {n: t.repeat(reps, 1) for n, t in d["probes"].items()}, k).cpu().numpy()
        assert np.all(np.abs(tau.reshape(reps, -1) - st["tau"]) <= tol), (reps, tau[:6], st["tau"])
    gi.close()


@pytest.mark.parametrize("order", ["nearer and nearer", "any"])
@pytest.mark.parametrize("D,B,size", [(128, 4, 1023), (128, 4, 5000), (64, 1, 1025), (64, 1, 12000), (64, 4, 12000),
                                      (256, 5, 3000), (512, 3, 2000)])
def test_lists_without_copies(D, B, size, order):
    # every vector its own, the nearest ones in the last tiles: the limit falls all the way and the list in LDS is cut
    # again and again, in the form with a wavefront per query and in the one with four
    nq = 6
    rng = np.random.default_rng(D + size)
    x0 = rng.standard_normal(D)
    U = rng.standard_normal((size, D))
    r = np.linspace(12.0, 0.3, size)
    if order == "any":
        r = rng.permutation(r)
    X = (x0 + r[:, None] * U / np.linalg.norm(U, axis=1, keepdims=True)).astype(np.float32)
    ix = build.build_index(X, 1, B, centroids=(x0 + 0.05 * rng.standard_normal(D))[None])
    s, gi = search.Searcher(ix), upload(ix)
    Q = (x0 + 0.05 * rng.standard_normal((nq, D))).astype(np.float32)
    reps = 2100 // nq
    for k in (1, 31, 33, 64, 65, 128):
        st = oracle_stages(s, Q, k, 1)
        d = to_dev(st)
        few = gi.seed_threshold(d["prep"], d["probes"], k)
        many = gi.seed_threshold({n: t.repeat((reps,) + (1,) * (t.dim() - 1)) for n, t in d["prep"].items()},
                                 {n: t.repeat(reps, 1) for n, t in d["probes"].items()}, k)
        assert torch.equal(many, few.repeat(reps)), k
        check_thresholds(s, st, k, few.cpu().numpy())
        if order != "any" and size > 1100:   # what the first 16 tiles alone would give is far off
            head = ix["offsets"].copy()
            head[1] = 1024
            cut = search.Searcher(dict(ix, offsets=head))
            first = [cut.seed_threshold(st["probes"][i], st["G"][i], st["E"][i], st["Qr"][i], st["delta"][i], st["planes"][i],
                                        int(st["S"][i]), k) for i in range(nq)]
            assert np.all(np.array(first) > 1.5 * st["tau"])
    gi.close()
