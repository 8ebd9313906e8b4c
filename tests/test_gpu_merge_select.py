"""The per-query merge around the edges of its two kernels: k up to 64 and above, fewer and more than 64 lists (one and
several rounds of lists), empty lists, full ones, fewer candidates than k, and equal distances, which go to the lower id."""
import numpy as np
import pytest
import torch

from oracle import build
from paper_2602_23999_amd import rabitq

from gpu_helpers import upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 10, 64, 65, 100, 128])
@pytest.mark.parametrize("nprobe,fill", [(1, "full"), (63, "some"), (64, "some"), (65, "full"), (130, "few"), (130, "full")])
def test_merge_selects_the_k_smallest(k, nprobe, fill):
    nq, nlist = 9, 130
    rng = np.random.default_rng(1000 * k + nprobe)
    C = rng.standard_normal((nlist, 32))
    gi = upload(build.build_index((C + 0.1).astype(np.float32), nlist, 1, centroids=C))
    cap = rabitq.load_library().rabitq_cand_capacity(k)
    cnt = {"full": np.full((nq, nprobe), cap), "some": rng.integers(0, 40, (nq, nprobe)),
           "few": (rng.random((nq, nprobe)) < 0.2).astype(int)}[fill].astype(np.int32)
    cnt[0] = 0                                   # a query without candidates
    d = rng.integers(0, 200, (nq, nprobe, cap)).astype(np.float32) - 20.0      # many equal distances
    ids = np.stack([rng.permutation(nprobe * cap) for _ in range(nq)]).reshape(nq, nprobe, cap)
    bits = d.view(np.uint32)
    order = np.where(bits >> 31, ~bits, bits | np.uint32(1 << 31)).astype(np.uint64)
    keys = (order << np.uint64(32)) | ids.astype(np.uint64)
    got_i, got_d = gi.merge(torch.from_numpy(keys.view(np.int64)).cuda(), torch.from_numpy(cnt).cuda(), nq, k, nprobe)
    got_i, got_d = got_i.cpu().numpy(), got_d.cpu().numpy()
    for q in range(nq):
        have = np.arange(cap)[None, :] < cnt[q][:, None]
        best = np.lexsort((ids[q][have], d[q][have]))[:k]
        n = len(best)
        assert np.array_equal(got_i[q, :n], ids[q][have][best]) and np.array_equal(got_d[q, :n], d[q][have][best])
        assert np.all(got_i[q, n:] == -1) and np.all(np.isinf(got_d[q, n:]))
    gi.close()


@pytest.mark.parametrize("k", [1, 10, 64, 65, 100, 128])
@pytest.mark.parametrize("nprobe", [16, 64, 130])
@pytest.mark.parametrize("kind", ["one", "smaller after copies", "copies at the last place"])
def test_merge_of_repeated_keys(k, nprobe, kind):
    # the stage takes whatever keys its caller hands it: copies of a key count like any other keys, also more of them
    # than the kernel's buffer of 512 holds
    nq, nlist = 5, 130
    rng = np.random.default_rng(1000 * k + nprobe)
    C = rng.standard_normal((nlist, 32))
    gi = upload(build.build_index((C + 0.1).astype(np.float32), nlist, 1, centroids=C))
    cap = rabitq.load_library().rabitq_cand_capacity(k)
    total = nprobe * cap
    val = np.full((nq, total), 7.0, np.float32)
    ids = np.full((nq, total), 3)
    if kind == "smaller after copies":
        for q in range(nq):       # fewer better keys than k, all of them behind at least 600 copies
            late = 600 + rng.permutation(total - 600)[:max(1, k - 1 - q)]
            val[q, late], ids[q, late] = 1.0 + rng.random(len(late)), late
    elif kind == "copies at the last place":
        val[:] = 100.0 + rng.random((nq, total))
        ids[:] = rng.permutation(total)[None]
        for q in range(nq):       # k - 1 better keys, then many copies of the k-th, somewhere among worse ones
            at = rng.permutation(total)
            val[q, at[:k - 1]], (val[q, at[k - 1:k + 700]], ids[q, at[k - 1:k + 700]]) = rng.random(k - 1), (50.0, 11)
    bits = val.view(np.uint32)
    order = np.where(bits >> 31, ~bits, bits | np.uint32(1 << 31)).astype(np.uint64)
    keys = (order << np.uint64(32)) | ids.astype(np.uint64)
    cnt = torch.full((nq, nprobe), cap, dtype=torch.int32, device="cuda")
    got_i, got_d = gi.merge(torch.from_numpy(keys.view(np.int64)).cuda(), cnt, nq, k, nprobe)
    got_i, got_d = got_i.cpu().numpy(), got_d.cpu().numpy()
    for q in range(nq):
        best = np.lexsort((ids[q], val[q]))[:k]
        assert np.array_equal(got_i[q], ids[q][best]) and np.array_equal(got_d[q], val[q][best]), q
    gi.close()


@pytest.mark.parametrize("k", [3, 4, 7, 8, 64, 65, 128])
@pytest.mark.parametrize("nprobe", [16, 63, 64, 130])
def test_few_and_many_queries_merge_alike(k, nprobe):
    # a query is merged by four wavefronts where there are few queries and by one where there are many, with kept keys that
    # fit the final selection as they are and with more of them
    nq, nlist = 8, 130
    rng = np.random.default_rng(1000 * k + nprobe)
    C = rng.standard_normal((nlist, 32))
    gi = upload(build.build_index((C + 0.1).astype(np.float32), nlist, 1, centroids=C))
    cap = rabitq.load_library().rabitq_cand_capacity(k)
    cnt = np.minimum(rng.integers(0, cap + 1, (nq, nprobe)), np.array([cap, cap, 20, 5, 5, 1, 2 * k // nprobe + 1, cap])[:, None])
    d = np.sort(rng.integers(0, 500, (nq, nprobe * cap)), 1).reshape(nq, nprobe, cap)[:, ::-1, ::-1].astype(np.float32)
    d[1::2] = rng.integers(0, 500, (nq // 2, nprobe, cap))       # (even rows: better and better keys, the limit keeps falling)
    ids = rng.integers(0, nprobe * cap // 2, (nq, nprobe, cap))
    order = d.view(np.uint32).astype(np.uint64) | np.uint64(1 << 31)
    keys = torch.from_numpy(((order << np.uint64(32)) | ids.astype(np.uint64)).view(np.int64)).cuda()
    cnt_d = torch.from_numpy(cnt.astype(np.int32)).cuda()
    for reps in (1, 64, 65, 128, 129):                            # 8, 512, 520, 1024, 1032 queries
        got_i, got_d = gi.merge(keys.repeat(reps, 1, 1), cnt_d.repeat(reps, 1), nq * reps, k, nprobe)
        got_i, got_d = got_i.cpu().numpy().reshape(reps, nq, k), got_d.cpu().numpy().reshape(reps, nq, k)
        for q in range(nq):
            have = np.arange(cap)[None, :] < cnt[q][:, None]
            best = np.lexsort((ids[q][have], d[q][have]))[:k]
            assert np.all(got_i[:, q, :len(best)] == ids[q][have][best]) and np.all(got_d[:, q, :len(best)] == d[q][have][best])
            assert np.all(got_i[:, q, len(best):] == -1)
    gi.close()
