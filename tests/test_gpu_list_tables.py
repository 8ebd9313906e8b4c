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


@pytest.mark.parametrize("nlist", [2047, 2049, 8192, 8193])
def test_lists_of_several_segments_on_both_sides_of_a_chunk(nlist):
    # a few hundred vectors in some lists around the edges of a thread's 8 lists and of a chunk, scanned in segments of two
    # tiles: a list's items and survivor blocks are products of its pairs, segments and tiles.  The reference is the
    # search in batches of 50 queries, whose tables come from the small-batch builder.
    D, nprobe, k = 64, 5, 3
    rng = np.random.default_rng(nlist)
    C = rng.standard_normal((nlist, D))
    long = np.unique([c for c in (0, 7, 8, 1000, 2039, 2040, 2046, 2047, 2048, 2049, 5000, 8183, 8184, 8190, 8191, 8192) if c < nlist])
    which = np.concatenate([np.repeat(long, rng.integers(150, 500, len(long))), rng.integers(0, nlist, 2000)])
    X = (C[which] + 0.1 * rng.standard_normal((len(which), D))).astype(np.float32)
    gi = upload(build.build_index(X, nlist, 4, centroids=C))
    gi.set_option("scan_segment_tiles", 2)
    gi.set_option("split_min_pairs", 0)
    nq = 4 * nlist // nprobe + 100                        # just above four pairs per list: not the prefetching scan
    Q = torch.from_numpy((C[rng.choice(long, nq)] + 0.3 * rng.standard_normal((nq, D))).astype(np.float32)).cuda()
    want_i, want_d = (torch.cat(t) for t in zip(*[gi.search(Q[i:i + 50].contiguous(), k, nprobe) for i in range(0, nq, 50)]))
    for impl, n, split, stream in ((0, nq, 0, 0), (0, nq - 200, 0, 1), (4, nq, 1, 0), (4, nq - 200, 1, 0)):
        for longest in (1, 0):
            gi.set_option("scan_impl", impl)
            gi.set_option("longest_first", longest)
            ids, d = gi.search(Q[:n].contiguous(), k, nprobe)
            assert (gi.index_info("last_scan_split"), gi.index_info("last_scan_stream")) == (split, stream)
            assert torch.equal(ids, want_i[:n]) and torch.equal(d, want_d[:n]), (impl, n, longest)
    gi.close()


@pytest.mark.parametrize("D,nlist", [(64, 1), (64, 7), (64, 9), (64, 2047), (64, 2049), (64, 8191), (64, 8193), (64, 16390), (960, 9), (960, 2049)])
def test_tables_of_the_group_scan_at_the_edges_of_a_chunk(D, nlist):
    # the item table in the order in which the lists are dealt to the XCDs, and descriptors of 16 pairs: some lists of several tiles, which
    # the wide form scans in segments of two
    nprobe, k = min(5, nlist), 3
    rng = np.random.default_rng(nlist + D)
    C = rng.standard_normal((nlist, D))
    long = np.unique([c for c in (0, 6, 7, 8, nlist // 2, 2046, 2047, 2048, 8191, 8192, nlist - 1) if c < nlist])
    which = np.concatenate([np.repeat(long, rng.integers(150, 400, len(long))), rng.integers(0, nlist, 1000)])
    X = (C[which] + 0.1 * rng.standard_normal((len(which), D))).astype(np.float32)
    nq = 333
    Q = torch.from_numpy((C[rng.choice(long, nq)] + 0.3 * rng.standard_normal((nq, D))).astype(np.float32)).cuda()
    gi = upload(build.build_index(X, nlist, 4, centroids=C))
    gi.set_option("scan_segment_tiles", 2)
    gi.set_option("scan_impl", 0)
    want_i, want_d = gi.search(Q, k, nprobe)
    gi.set_option("scan_impl", 4)
    gi.set_option("split_min_pairs", 0)
    gi.set_option("group_min", 0)
    ids, d = gi.search(Q, k, nprobe)
    assert gi.index_info("last_scan_group") == 1
    assert torch.equal(ids, want_i) and torch.equal(d, want_d)
    gi.close()
