"""Threshold seeding at the sizes where its selection can go wrong: list lengths around a tile, around the tiles held
in registers and beyond the list in LDS; k around the number of seeds (32), a wavefront (64) and the largest (128);
queries sharing a workgroup (few) and having a wavefront each (more than 2048); equal estimates."""
import numpy as np
import pytest
import torch

from oracle import build, search

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
