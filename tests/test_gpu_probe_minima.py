"""Probe selection from the smallest score of every 32 lists, which a search of a batch takes where there are many lists, against
the selection that reads whole score rows (`coarse_probe`): one vector per list and as many neighbours as probes, so the
neighbours of a query are the lists that it probed."""
import numpy as np
import pytest
import torch

from oracle import build
from paper_2602_23999_amd import rabitq

from gpu_helpers import upload

pytestmark = pytest.mark.gpu


#        nlist nprobe nq metric
CASES = [
    (129, 1, 70, "l2"),      # 5 minima, the last one of a single list
    (1000, 7, 100, "l2"),    # a ragged last tile; fewer than 8 tiles read
    (1024, 8, 65, "ip"),
    (1056, 8, 200, "l2"),    # 33 minima
    (4100, 32, 130, "ip"),   # 32 tiles read, ragged
    (8192, 64, 131, "l2"),   # the most probes; 256 minima, 4 words a lane
    (8193, 33, 700, "l2"),   # 257 minima: 16 words a lane
    (32768, 20, 70, "l2"),   # the most minima
]


@pytest.mark.parametrize("nlist,nprobe,nq,metric", CASES)
def test_minima_select_what_whole_rows_select(nlist, nprobe, nq, metric):
    D = 64
    rng = np.random.default_rng(nlist + nprobe)
    C = rng.standard_normal((nlist, D)).astype(np.float32)
    if metric == "ip":
        C /= np.linalg.norm(C, axis=1, keepdims=True)
    C[nlist - 1] = C[3]             # equal scores: the lower list comes first
    C[nlist // 2] = C[7]
    ix = build.build_index(C, nlist, 1, metric=metric, centroids=C)
    gi = upload(ix)
    Q = (C[rng.integers(0, nlist, nq)] + 0.5 * rng.standard_normal((nq, D))).astype(np.float32)
    Q[1] = np.nan                   # every score of the row is a NaN ...
    Q[2] = 1e30                     # ... or beyond the range
    Q[3] = C[3]
    Q[4] = C[7]
    q = torch.from_numpy(Q).cuda()
    q_rot = gi.rotate(q)
    lists = gi.coarse_probe(q_rot, gi.query_prep(q_rot)["sq_norm"], nprobe)["probe_ids"].cpu().numpy()
    ids, _ = gi.search(q, nprobe, nprobe)
    ids = ids.cpu().numpy()
    off = ix["offsets"]
    for i in range(nq):
        if i in (1, 2):             # no estimate, no neighbour: see the next test
            continue
        want = {int(v) for c in lists[i] for v in ix["ids"][off[c]:off[c + 1]]}
        got = {int(v) for v in ids[i] if v >= 0}
        assert got <= want and len(got) == min(nprobe, len(want)), (i, sorted(got ^ want))
    gi.close()


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("nlist,nprobe", [(1000, 7), (1056, 1), (4100, 32)])
def test_scores_that_are_no_numbers_rank_as_in_whole_rows(nlist, nprobe, metric):
    # lists whose centroid is not a number, infinite or out of range, queries likewise; batches of 50 select from whole rows
    D, n = 64, 3 * nlist
    rng = np.random.default_rng(nlist)
    X = rng.standard_normal((n, D)).astype(np.float32)
    first = np.arange(nlist) * n // nlist          # (without a training pass these rows are the centroids)
    X[first[5::9], 3] = np.nan
    X[first[7::40]] = 1e30
    X[first[-2:]] = np.inf
    gi = rabitq.Index.build(torch.from_numpy(X).cuda(), nlist, 1, build.random_rotation(D, 7), metric=metric, kmeans_iters=0, center=False)
    Q = (X[rng.integers(0, n, 200)] + 0.1 * rng.standard_normal((200, D))).astype(np.float32)
    Q[:8] = 0.0
    Q[0, :2] = 3e38
    Q[1] = np.nan
    Q[2] = 1e37 * rng.standard_normal(D)
    Q[3, 4] = -np.inf
    q = torch.from_numpy(Q).cuda()
    got = gi.search(q, 20, nprobe)
    want = [torch.cat(t) for t in zip(*[gi.search(q[i:i + 50].contiguous(), 20, nprobe) for i in range(0, 200, 50)])]
    assert torch.equal(got[0], want[0])
    assert bool(((got[1] == want[1]) | (got[1].isnan() & want[1].isnan())).all())
    gi.close()
