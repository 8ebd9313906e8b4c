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
        for name, value in options:
            gi.set_option(name, value)
        ids, d = gi.search(q, k, nprobe)
        assert (gi.index_info("last_scan_split"), gi.index_info("last_scan_group")) == want
        assert torch.equal(ids, ref_i) and torch.equal(d, ref_d)
    finally:
        gi.set_option("scan_impl", 3)
        gi.set_option("split_min_pairs", 32)


@pytest.mark.parametrize("D,nq,nprobe,options,want", [
    (960, 24, 4, [("scan_impl", 4), ("split_min_pairs", 1)], GROUP),    # six groups
    (960, 1, 8, [("scan_impl", 4), ("split_min_pairs", 1)], GROUP),     # one pair a list
    (960, 24, 4, [("scan_impl", 4)], GROUP),                            # 12 pairs a list, at least 8 asked for
    (960, 15, 4, [("scan_impl", 4)], SINGLE),                           # 7.5
    (1024, 1023, 8, [("scan_impl", 3)], SINGLE),                        # chosen by itself from 512 groups of 16 pairs on
    (1024, 1024, 8, [("scan_impl", 3)], GROUP),
])
def test_wide_codes_go_by_groups(D, nq, nprobe, options, want):
    check(D, 4, 8, nq, nprobe, options, want)
