"""The group scan (one wavefront estimates and refines for 16 pairs of a list) against the kernels for single work items on the same
handle: the same integers, the same rounding, so the same neighbours and distances, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import build
from paper_2602_23999_amd import rabitq

pytestmark = pytest.mark.gpu


#        D    bits nlist n      nq   nprobe k    metric
CASES = [
    (32, 2, 5, 700, 33, 3, 10, "l2"),          # one code word; lists of a few tiles, ragged; 2-bit fields
    (64, 3, 7, 3_000, 90, 7, 1, "l2"),         # every list probed: 90 pairs a list, the last group of 10
    (96, 4, 3, 200, 100, 1, 100, "l2"),        # lists below k, some of less than a tile; 4-bit fields
    (96, 8, 16, 9_000, 257, 4, 128, "ip"),     # flipped bytes; regions cut at k = 128
    (128, 4, 1, 2_048, 64, 1, 64, "l2"),       # a list of 32 tiles, the longest that a few groups take
    (128, 4, 4, 4_200, 64, 4, 64, "l2"),       # lists of 16 tiles and more
    (128, 5, 1, 1_000, 17, 1, 10, "l2"),       # one list, a group of one pair beside a full one
    (256, 7, 6, 2_500, 130, 2, 33, "l2"),      # the widest of the narrow form
    (960, 5, 4, 1_500, 40, 3, 10, "l2"),       # the wide form, lists in segments
    (960, 4, 40, 2_600, 130, 3, 17, "ip"),     # lists of one or two tiles
    (1024, 8, 5, 1_100, 65, 2, 100, "l2"),
]


@pytest.mark.parametrize("D,bits,nlist,n,nq,nprobe,k,metric", CASES)
def test_group_scan_finds_what_the_single_kernels_find(D, bits, nlist, n, nq, nprobe, k, metric):
    rng = np.random.default_rng(D + bits + n)
    centre = rng.standard_normal((nlist, D))
    X = (centre[rng.integers(0, nlist, n)] + 0.5 * rng.standard_normal((n, D))).astype(np.float32)
    Q = (centre[rng.integers(0, nlist, nq)] + 0.5 * rng.standard_normal((nq, D))).astype(np.float32)
    X[1] = X[0]                    # equal distances
    Q[2] = 0.0                     # no scale for its digits
    Q[3] *= 1e-20
    gi = rabitq.Index.build(torch.from_numpy(X).cuda(), nlist, bits, build.random_rotation(D, 7), metric=metric, kmeans_iters=2)
    q = torch.from_numpy(Q).cuda()
    gi.set_option("split_min_pairs", 0)   # by groups however few the pairs
    gi.set_option("group_min", 0)
    for prune in (1, 0):
        gi.set_option("prune", prune)
        gi.set_option("scan_impl", 0)
        want_i, want_d = gi.search(q, k, nprobe)
        assert gi.index_info("last_scan_split") == 0
        gi.set_option("scan_impl", 4)
        got_i, got_d = gi.search(q, k, nprobe)
        assert gi.index_info("last_scan_split") == 1 and gi.index_info("last_scan_group") == 1
        assert torch.equal(got_d, want_d) and torch.equal(got_i, want_i)
    gi.close()
