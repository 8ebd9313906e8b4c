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
        want = np.minimum(st["tau"], np.float64(np.finfo(np.float32).max))
        scale = key_scale(st["G"], st["E"], s.metric)
        bad = np.abs(few.cpu().numpy() - want) > 1e-4 * (np.abs(want) + scale)
        # (another seed may be taken where two 1-bit estimates at the last rank are equal up to their rounding)
        assert bad.sum() <= 1, (k, few.cpu().numpy(), want)
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
