"""Which scan a search takes ("last_scan_split", "last_scan_group"), on both sides of the lines that the header draws; whichever
it is, the neighbours and distances are those of the popcount kernel."""
import numpy as np
import pytest
import torch

from oracle import build
from paper_2602_23999_amd import rabitq

pytestmark = pytest.mark.gpu

SINGLE, SPLIT, GROUP = (0, 0), (1, 0), (1, 1)
_index = {}


def index(D, bits, nlist):
    if (D, bits, nlist) not in _index:
        rng = np.random.default_rng(D + nlist)
        C = rng.standard_normal((nlist, D))
        X = (C[np.arange(nlist * 30) % nlist] + 0.3 * rng.standard_normal((nlist * 30, D))).astype(np.float32)
        gi = rabitq.Index.build(torch.from_numpy(X).cuda(), nlist, bits, build.random_rotation(D, 7), kmeans_iters=1)
        _index[D, bits, nlist] = gi, torch.from_numpy(X[::7].copy()).cuda()
    return _index[D, bits, nlist]


def check(D, bits, nlist, nq, nprobe, options, want, k=5):
    gi, q = index(D, bits, nlist)
    q = q[torch.arange(nq, device="cuda") % len(q)].contiguous()
    try:
        gi.set_option("scan_impl", 0)
        ref_i, ref_d = gi.search(q, k, nprobe)
        for name, value in [("scan_impl", 3), *options]:
            gi.set_option(name, value)
        ids, d = gi.search(q, k, nprobe)
        assert (gi.index_info("last_scan_split"), gi.index_info("last_scan_group")) == want
        assert torch.equal(ids, ref_i) and torch.equal(d, ref_d)
    finally:
        gi.set_option("scan_impl", 3)
        gi.set_option("split_min_pairs", 32)
        gi.set_option("group_min", -1)


@pytest.mark.parametrize("D,nq,nprobe,options,want", [
    (960, 24, 4, [("scan_impl", 4), ("split_min_pairs", 1)], GROUP),    # six groups
    (960, 1, 8, [("scan_impl", 4), ("split_min_pairs", 1)], GROUP),     # one pair a list
    (960, 24, 4, [("scan_impl", 4)], GROUP),                            # 12 pairs a list, at least 8 asked for
    (960, 15, 4, [("scan_impl", 4)], SINGLE),                           # 7.5
    (1024, 1023, 8, [], SINGLE),                                        # chosen by itself from 512 groups of 16 pairs on
    (1024, 1024, 8, [], GROUP),
])
def test_wide_codes_go_by_groups(D, nq, nprobe, options, want):
    check(D, 4, 8, nq, nprobe, options, want)


@pytest.mark.parametrize("bits,nq,k,options,want", [
    (5, 1535, 16, [], SINGLE), (5, 1536, 16, [], GROUP), (5, 1536, 17, [], SINGLE), (8, 4096, 17, [], SINGLE),
    (5, 1536, 17, [("scan_impl", 4)], GROUP), (5, 1536, 17, [("group_min", 768)], GROUP),
    (4, 1024, 128, [], GROUP), (2, 1023, 5, [], SINGLE),
])
def test_long_wide_codes_go_by_groups_for_few_neighbours(bits, nq, k, options, want):
    check(960, bits, 8, nq, 8, options, want, k)


@pytest.mark.parametrize("D,nq,nprobe,options,want", [
    (64, 8191, 8, [], SPLIT),                                           # 65 528 pairs: 4095.5 groups
    (64, 8192, 8, [], GROUP),
    (256, 8192, 8, [("scan_impl", 4)], GROUP),
    (64, 8192, 8, [("split_min_pairs", 8193)], SINGLE),                 # 8192 pairs a list
    (64, 100, 3, [("scan_impl", 4), ("split_min_pairs", 0)], SPLIT),    # few pairs a list ask for no fewer groups
    (64, 100, 3, [("scan_impl", 4), ("group_min", 0)], GROUP),          # 37 pairs a list
    (64, 100, 3, [("scan_impl", 4), ("group_min", 19)], SPLIT),
    (512, 100, 3, [("scan_impl", 4), ("group_min", 0)], SPLIT),         # not built for that width
    (960, 100, 3, [("group_min", 0)], GROUP),
    (960, 100, 3, [("scan_impl", 4), ("group_min", 19)], SINGLE),
])
def test_groups_from_group_min_on(D, nq, nprobe, options, want):
    check(D, 4, 8, nq, nprobe, options, want)


@pytest.mark.parametrize("D,k,options,want", [
    (64, 32, [], GROUP), (64, 33, [], SPLIT), (256, 64, [("scan_impl", 4)], SPLIT), (64, 65, [], GROUP), (64, 128, [], GROUP),
    (64, 50, [("group_min", 4096)], GROUP),                             # asked for
    (960, 50, [], GROUP),
])
def test_up_to_256_dimensions_some_k_are_split(D, k, options, want):
    check(D, 4, 8, 8192, 8, options, want, k)


@pytest.mark.parametrize("n,k,want", [(32 * 64, 9, GROUP), (32 * 64 + 1, 9, SPLIT), (64 * 64, 65, GROUP), (64 * 64 + 1, 65, SPLIT)])
def test_a_list_too_long_for_one_wavefront_is_split(n, k, want):
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 64)).astype(np.float32)
    gi = rabitq.Index.build(torch.from_numpy(X).cuda(), 1, 4, build.random_rotation(64, 7), kmeans_iters=1)
    q = torch.from_numpy(X[:50] + 0.1).cuda()
    gi.set_option("group_min", 0)
    ids, d = gi.search(q, k, 1)
    assert (gi.index_info("last_scan_split"), gi.index_info("last_scan_group")) == want
    gi.set_option("scan_impl", 0)
    ref_i, ref_d = gi.search(q, k, 1)
    assert torch.equal(ids, ref_i) and torch.equal(d, ref_d)
    gi.close()


@pytest.mark.parametrize("k", [5, 100])
def test_the_last_part_of_a_search_by_groups_is_split(k):
    D, nlist = 64, 8
    rng = np.random.default_rng(3)
    X = rng.standard_normal((40 * nlist, D)).astype(np.float32)
    q = torch.from_numpy(rng.standard_normal((12_288, D)).astype(np.float32)).cuda()
    gi = rabitq.Index.build(torch.from_numpy(X).cuda(), nlist, 4, build.random_rotation(D, 7), kmeans_iters=1)
    gi.set_option("max_batch", 8192)
    ids, d = gi.search(q, k, 8)           # 8192 queries by groups, then 4096, on a handle that has split nothing yet
    assert (gi.index_info("last_scan_split"), gi.index_info("last_scan_group")) == SPLIT
    gi.set_option("scan_impl", 0)
    ref_i, ref_d = gi.search(q, k, 8)
    assert torch.equal(ids, ref_i) and torch.equal(d, ref_d)
    gi.close()
