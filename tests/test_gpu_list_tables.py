"""Pair lists and work-item tables at the list counts where their running sums can go wrong: one list, a remainder of
a thread's 8 lists, and either side of the chunk of 2048 (256 threads) and of 8192 (1024 threads) lists."""
import numpy as np
import pytest
import torch

from oracle import build

from gpu_helpers import upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nlist", [1, 7, 9, 2047, 2048, 2049, 8191, 8192, 8193, 16390])
def test_tables_at_the_edges_of_a_chunk(nlist):
    D, n, nq, k = 64, 3000, 200, 3
    nprobe = min(5, nlist)
    rng = np.random.default_rng(nlist)
    C = rng.standard_normal((nlist, D))
    X = (C[rng.integers(0, nlist, n)] + 0.2 * rng.standard_normal((n, D))).astype(np.float32)
    Q = (C[rng.integers(0, nlist, nq)] + 0.3 * rng.standard_normal((nq, D))).astype(np.float32)
    gi = upload(build.build_index(X, nlist, 4, centroids=C))
    probes = np.stack([rng.choice(nlist, nprobe, replace=False) for _ in range(nq)]).astype(np.int32)
    pair_off, pair_ids = gi.build_probe_lists(torch.from_numpy(probes).cuda())
    flat = probes.reshape(-1)
    assert np.array_equal(pair_off.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(flat, minlength=nlist))]))
    assert np.array_equal(pair_ids.cpu().numpy(), np.argsort(flat, kind="stable"))
    # the item tables: the split search (three tables), the general kernel and, where the batch has few pairs per list,
    # the prefetching one in list order and longest list first must find the same neighbours
    q = torch.from_numpy(Q).cuda()
    got = []
    for impl, longest in ((0, 1), (0, 0), (4, 0)):
        gi.set_option("scan_impl", impl)
        gi.set_option("longest_first", longest)
        gi.set_option("split_min_pairs", 0)
        got.append([t.cpu().numpy() for t in gi.search(q, k, nprobe)])
    for ids, d in got[1:]:
        assert np.array_equal(ids, got[0][0]) and np.array_equal(d, got[0][1])
    gi.close()
