"""The scans of groups of 16 pairs (as one kernel, and as two) against the CPU oracle through the stage entry point, whose callers hand
in the queries as bytes and floats: the integers of the estimates, and the neighbours under an injected threshold."""
import numpy as np
import pytest
import torch

from oracle import build, search
from paper_2602_23999_amd import rabitq, synth

from gpu_helpers import compare_topk, key_scale, oracle_stages, to_dev, upload

pytestmark = pytest.mark.gpu

CASES = {
    # name: (workload, n, nq, n_centres, nlist, B, k, nprobe)
    "l2_128_b4": ("l2_128", 30_000, 96, 64, 48, 4, 10, 6),
    "l2_128_b8": ("l2_128", 4_000, 40, 32, 12, 8, 10, 5),
    "l2_96_b3_k100": ("l2_96", 20_000, 64, 64, 40, 3, 100, 8),
    "ragged_b2": ("tiny", 1_500, 40, 50, 50, 2, 10, 50),
    "centred_b4": ("l2_128", 8_000, 64, 64, 32, 4, 10, 6),
    "ip_768_b8": ("ip_768_tight", 1_500, 24, 12, 10, 8, 10, 4),
    "l2_960_b5": ("l2_960", 4_000, 24, 16, 12, 5, 10, 4),
    "l2_960_b2_k100": ("l2_960", 3_000, 40, 8, 6, 2, 100, 3),
}
ONE = [n for n in CASES if not n.startswith("ip_768")]     # (not built from 257 to 959 dimensions)
TWO = [n for n in CASES if not n.startswith("l2_960")]     # (nor this from 960 on)
ROUTES = [(n, 1) for n in ONE] + [(n, 2) for n in TWO]
_cache = {}


def case(name):
    if name not in _cache:
        wl, n, nq, nc, nlist, B, k, nprobe = CASES[name]
        w = synth.WORKLOADS[wl].scaled(n=n, nq=nq, n_centres=nc)
        X, Q = synth.make_base(w), synth.make_queries(w)
        ix = build.build_index(X, nlist, B, metric=w.metric, kmeans_iters=4, center=name.startswith("centred"))
        s = search.Searcher(ix)
        st = oracle_stages(s, Q, k, nprobe)
        _cache[name] = dict(Q=Q, ix=ix, s=s, st=st, k=k, nprobe=nprobe, dev=to_dev(st))
    return _cache[name]


def handle(c, kernels):
    gi = upload(c["ix"])
    gi.set_option("scan_impl", 4)
    gi.set_option("split_min_pairs", 0)
    gi.set_option("group_min", 0 if kernels == 1 else 1 << 20)
    return gi


def route(gi):
    return gi.index_info("last_scan_split"), gi.index_info("last_scan_group")


@pytest.mark.parametrize("name,kernels", ROUTES)
def test_integer_inner_products(name, kernels):
    c = case(name)
    st, d, ix, s, nprobe = c["st"], c["dev"], c["ix"], c["s"], c["nprobe"]
    gi = handle(c, kernels)
    tiles = (np.diff(ix["offsets"]) + 63) // 64
    cluster = st["probes"].reshape(-1)[st["pair_ids"]]
    dbg_off = np.concatenate([[0], np.cumsum(tiles[cluster] * 64)])
    _, _, dbg = gi.scan(d["prep"], d["probes"], d["pair_off"], d["pair_ids"], d["tau"], c["k"], dbg_off=torch.from_numpy(dbg_off).cuda())
    assert route(gi) == (1, int(kernels == 1))
    dbg = dbg.cpu().numpy()
    for pos in np.random.default_rng(0).choice(len(cluster), size=min(200, len(cluster)), replace=False):
        q, cl = int(st["pair_ids"][pos]) // nprobe, int(cluster[pos])
        a, b = int(ix["offsets"][cl]), int(ix["offsets"][cl + 1])
        assert np.array_equal(dbg[dbg_off[pos]:dbg_off[pos] + (b - a)], search.ip_bitplane(s.words[a:b], st["planes"][q])), (pos, q, cl)
    gi.close()


@pytest.mark.parametrize("prune", [True, False])
@pytest.mark.parametrize("name,kernels", ROUTES)
def test_neighbours_under_an_injected_threshold(name, kernels, prune):
    c = case(name)
    st, d, s, k, nprobe = c["st"], c["dev"], c["s"], c["k"], c["nprobe"]
    nq = len(c["Q"])
    gi = handle(c, kernels)
    # the oracle's threshold, moved up by a hair so that the k-th seed does not sit on a boundary of rounding
    scale = key_scale(st["G"], st["E"], s.metric)
    tau = np.minimum(st["tau"], rabitq.FLT_MAX)
    tau = (tau + 1e-5 * (np.abs(tau) + scale)).astype(np.float32)
    tau[(st["tau"] >= rabitq.FLT_MAX) | (not prune)] = rabitq.FLT_MAX
    keys, cnt, _ = gi.scan(d["prep"], d["probes"], d["pair_off"], d["pair_ids"], torch.from_numpy(tau).cuda(), k)
    assert route(gi) == (1, int(kernels == 1))
    assert int(cnt.max()) <= keys.shape[1]
    ids, dist = gi.merge(keys, cnt, nq, k, nprobe)
    o_ids, o_d, _ = s.search(c["Q"], k, nprobe, prune=prune, Qr=st["Qr"], tau=tau.astype(np.float64))
    # (1e-4 of the scale of a key, as for the single kernels)
    n_exact = compare_topk(ids.cpu().numpy(), dist.cpu().numpy().astype(np.float64), o_ids, o_d, 1e-4 * scale)
    assert n_exact >= 0.97 * nq
    gi.close()


@pytest.mark.parametrize("name,impl", [("l2_128_b4", 1), ("l2_960_b5", 1), ("l2_960_b5", 4)])
def test_stage_scan_in_a_capture_that_allocates_nothing(name, impl):
    # what the scan makes of the queries beforehand needs memory; in a capture it has to do without
    c = case(name)
    d, k, nprobe, nq = c["dev"], c["k"], c["nprobe"], len(c["Q"])
    warm = upload(c["ix"])
    gi = upload(c["ix"])
    for h in (warm, gi):
        h.set_option("scan_impl", impl)
        h.set_option("split_min_pairs", 0)
        h.set_option("group_min", 0)
    args = (d["prep"], d["probes"], d["pair_off"], d["pair_ids"], d["tau"], k)
    want = warm.merge(*warm.scan(*args)[:2], nq, k, nprobe)
    if impl == 4:
        gi.search(torch.from_numpy(c["Q"]).cuda(), k, nprobe)      # (the descriptors' memory)
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        keys, cnt, _ = gi.scan(*args)
        ids, dist = gi.merge(keys, cnt, nq, k, nprobe)
    assert route(gi) == (int(impl == 4), int(impl == 4))
    for _ in range(3):
        ids.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ids, want[0]) and torch.equal(dist, want[1])
        again = gi.merge(*gi.scan(*args)[:2], nq, k, nprobe)       # eager between the replays, with the memory
        assert torch.equal(again[0], want[0]) and torch.equal(again[1], want[1])
    warm.close()
    gi.close()
