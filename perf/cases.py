"""The work a user of this library has it do, as cases to be timed.

A case is one call of the public interface on one index: a batched search (rabitq_search through ``Index.search``, or the
allocation-free form for serving loops), or the construction of an index and the first batch searched in it.  The indices are of the shapes
that the repository's own workloads have (``paper_2602_23999_amd/synth.py``, ``bench.py``): 128-d image descriptors,
960-d dense descriptors, 96-d unit-norm deep features, 768-d unit-norm embeddings under inner product, and 1-bit codes of
low intrinsic dimension.  Their data is drawn on the device, so that making a case's inputs takes a second at most.
"""
from __future__ import annotations

import math

import torch

from paper_2602_23999_amd import rabitq

# Case keys.  do: "search" (Index.search), "noalloc" (Index.search_noalloc into buffers the caller keeps) or "build"
# (Index.build, then Index.search).  data: recipe of the vectors (_draw_vectors).  n vectors of dim dimensions in nlist lists,
# bits per dimension, metric, center as in Index.build; nq queries, k neighbours, nprobe lists per query.


def listed():
    def c(name, do, data, n, dim, nlist, bits, nq, k, nprobe, metric="l2", center=True):
        return dict(name=name, do=do, data=data, n=n, dim=dim, nlist=nlist, bits=bits, metric=metric,
                    center=center and metric == "l2", nq=nq, k=k, nprobe=nprobe)
    return [
        # one query at a time against the benchmark's index: the latency an interactive service sees
        c("one_query_128", "search", "descriptors", 1_000_000, 128, 1024, 4, 1, 10, 16),
        # the smallest workload of the repository: 10k vectors, 1-bit codes, 100 queries
        c("tiny_1bit_128", "search", "isotropic", 10_000, 128, 64, 1, 100, 10, 8, center=False),
        # a serving loop that may not allocate: a few dozen queries, a batch size that is no multiple of anything
        c("serving_37_queries_128", "noalloc", "descriptors", 1_000_000, 128, 1024, 4, 37, 10, 32),
        # an ordinary medium batch
        c("batch_777_128", "search", "descriptors", 1_000_000, 128, 1024, 4, 777, 10, 16),
        # the benchmark: 10^4 queries, 16 lists each
        c("batch_10k_128", "search", "descriptors", 1_000_000, 128, 1024, 4, 10_000, 10, 16),
        # high recall on the same data: 5 bits (stored in 8-bit fields), 128 lists per query, a long result list
        c("deep_probe_128", "search", "descriptors", 1_000_000, 128, 1024, 5, 3001, 50, 128),
        # deep features: many lists, 3 bits, 100 neighbours
        c("features_96_k100", "search", "unit_wide", 4_000_000, 96, 8192, 3, 10_000, 100, 32, center=True),
        # 960-d descriptors, 5 bits; plain k-means gives this recipe long hub lists
        c("dense_960", "search", "anisotropic", 1_000_000, 960, 1024, 5, 1000, 10, 16),
        # text embeddings, inner product, 8 bits
        c("embeddings_768_ip", "search", "unit_tight", 1_000_000, 768, 2048, 8, 2500, 10, 64, metric="ip"),
        # 1-bit codes larger than the last-level cache, every query in about one list of its own: the codes come from
        # memory once
        c("streaming_1bit_128", "search", "low_rank", 16_000_000, 128, 8192, 1, 6000, 10, 1, center=False),
        # construction of an index and the first batch searched in it
        c("build_250k_128", "build", "descriptors", 250_000, 128, 512, 4, 4096, 10, 32),
    ]


_FAMILIES = [  # data, dims, bits, metric
    ("descriptors", (128,), (2, 3, 4, 5, 6, 8), "l2"),
    ("isotropic", (64, 128, 256), (1, 2, 4), "l2"),
    ("unit_wide", (64, 96), (3, 4, 8), "l2"),
    ("anisotropic", (256, 512, 960), (4, 5, 7), "l2"),
    ("unit_tight", (512, 768), (4, 8), "ip"),
    ("low_rank", (128,), (1,), "l2"),
]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    data, dims, bits, metric = rng.choice(_FAMILIES)
    dim, b = rng.choice(dims), rng.choice(bits)
    n = _log_uniform(rng, 10_000, 4_000_000 if dim <= 128 else 256_000_000 // dim)
    nlist = max(16, min(8192, int(n / _log_uniform(rng, 150, 2000))))
    center = metric == "l2" and rng.random() < 0.7
    build = rng.random() < 0.1
    if build:
        n = min(n, 32_000_000 // dim)
        nlist = max(16, min(nlist, n // 100))
    nprobe = min(_log_uniform(rng, 1, 200), max(1, nlist // 2))
    k = _log_uniform(rng, 1, 100)
    nq = _log_uniform(rng, 1, 10_000)
    # no dearer than the largest listed case (a batch of 10^4 queries, 16 lists of 1000 vectors of 128 dimensions each;
    # the anisotropic recipe's hub lists multiply its work by about ten)
    hubs = 10 if data == "anisotropic" else 1
    nq = max(1, min(nq, int(2.5e10 / (nprobe * (n / nlist) * dim * hubs))))
    # (the allocation-free form works in 64 MiB of scratch: mostly candidate keys, nprobe regions of 128 or 256 per query)
    scratch = nq * (5 * nlist + nprobe * (8 * (128 if k <= 64 else 256) + 20) + 12 * dim)
    do = "build" if build else "noalloc" if nq <= 100 and scratch <= 32 << 20 and rng.random() < 0.3 else "search"
    return dict(do=do, data=data, n=n, dim=dim, nlist=nlist, bits=b, metric=metric, center=center, nq=nq, k=k,
                nprobe=nprobe)


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _rotation(dim, seed):
    """Random orthogonal matrix: QR of a seeded Gaussian matrix (the library takes it as an input)."""
    g = torch.Generator(device="cuda").manual_seed(1_000_003 * seed + dim)
    q, r = torch.linalg.qr(torch.randn((dim, dim), generator=g, device="cuda"))
    return (q * torch.sign(torch.diagonal(r))[None, :]).cpu().numpy()


def _draw_vectors(case, counts, seed):
    """Sets of `counts` vectors each, all from one mixture: base vectors first, queries as fresh draws after them."""
    data, D = case["data"], case["dim"]
    gen = torch.Generator(device="cuda").manual_seed(7_000_003 * seed + 11)
    rn = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    if data == "descriptors":
        # non-negative integer-valued features: 32 modes with a 12-d subspace each, 1024 components inside them
        nc, sub = 1024, 12
        modes = (36.0 + 26.0 * rn(32, D)).clamp_(min=0.0)
        basis = torch.linalg.qr(rn(32, D, sub))[0]
        which = torch.randint(0, 32, (nc,), generator=gen, device="cuda")
        centres = modes[which] + torch.bmm(basis[which], 12.0 * rn(nc, sub, 1)).squeeze(2)
    elif data == "low_rank":
        nc, sub = max(16, case["nlist"]), 8
        centres, basis = 4.0 * rn(nc, D), torch.linalg.qr(rn(64, D, sub))[0]
        which = torch.arange(nc, device="cuda") % 64
    elif data == "isotropic":
        nc = max(16, case["nlist"])
        centres = rn(nc, D)
    elif data == "anisotropic":
        nc = 2 * case["nlist"]
        centres, std = rn(nc, D), torch.rand((nc, D), generator=gen, device="cuda").mul_(0.9).add_(0.1).sqrt_()
    else:  # unit_wide / unit_tight
        nc = case["nlist"] if data == "unit_wide" else max(16, case["nlist"] // 2)
        centres = torch.nn.functional.normalize(rn(nc, D), dim=1)

    def chunk(m):
        comp = torch.randint(0, nc, (m,), generator=gen, device="cuda")
        if data in ("descriptors", "low_rank"):
            std_sub, std_iso = (23.0, 1.5) if data == "descriptors" else (3.0, 0.3)
            z, w = std_sub * rn(m, sub), which[comp]
            x = centres[comp] + std_iso * rn(m, D)
            for j in range(sub):  # (one direction at a time: no [m][D][sub] intermediate)
                x.addcmul_(z[:, j:j + 1], basis[:, :, j][w])
            return x.clamp_(0.0, 255.0).round_() if data == "descriptors" else x
        if data == "isotropic":
            return centres[comp] + 0.3 * rn(m, D)
        if data == "anisotropic":
            return centres[comp] + std[comp] * rn(m, D)
        noise = (0.5 if data == "unit_wide" else 0.15) / math.sqrt(D)
        return torch.nn.functional.normalize(centres[comp] + noise * rn(m, D), dim=1)

    out = []
    for n in counts:
        x = torch.empty((n, D), dtype=torch.float32, device="cuda")
        for s in range(0, n, 1 << 19):
            x[s:s + (1 << 19)] = chunk(min(1 << 19, n - s))
        out.append(x)
    return out


def _build(case, x, rotation):
    return rabitq.Index.build(x, case["nlist"], case["bits"], rotation, metric=case["metric"], kmeans_iters=5,
                              train_size=max(40 * case["nlist"], case["n"] // 10), center=case["center"])


def prepare(case, seed):
    rotation = _rotation(case["dim"], seed)
    x, q = _draw_vectors(case, (case["n"], case["nq"]), seed)
    st = dict(case=case, q=q)
    if case["do"] == "build":
        st.update(x=x, rotation=rotation)
        return st
    st.update(index=_build(case, x, rotation))
    if case["do"] == "noalloc":
        st.update(ids=torch.empty((case["nq"], case["k"]), dtype=torch.int64, device="cuda"),
                  dists=torch.empty((case["nq"], case["k"]), dtype=torch.float32, device="cuda"))
    return st


def run(state):
    case = state["case"]
    if case["do"] == "build":
        return _build(case, state["x"], state["rotation"]).search(state["q"], case["k"], case["nprobe"])
    if case["do"] == "noalloc":
        return state["index"].search_noalloc(state["q"], case["k"], case["nprobe"], state["ids"], state["dists"])
    return state["index"].search(state["q"], case["k"], case["nprobe"])


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    n, D, L, B = case["n"], case["dim"], case["nlist"], case["bits"]
    row = D * B / 8 + 20 if B > 1 else 0  # long code, its two factors, the 1-bit code's third factor, id
    nq, k, p = case["nq"], case["k"], case["nprobe"]
    touched = n * (1.0 - (1.0 - p / L) ** nq)  # vectors of the lists that some query probes
    evaluations = float(nq) * p * n / L
    w = {"bytes": 4.0 * D * (nq + D + L) + touched * (D / 8 + 8) + min(float(nq) * k, touched) * row + 12.0 * nq * k,
         "flops": 2.0 * nq * D * (D + L) + 2.0 * D * evaluations}
    if case["do"] == "build":
        train = min(n, max(40 * L, n // 10))
        w["bytes"] += 4.0 * n * D + n * (D / 8 + 12 + row)
        w["flops"] += 2.0 * n * D * D + 2.0 * D * L * (n + 5 * train)
    return w


def tolerance(case):
    # Measured against the same stages fed with queries rotated in 64 bits: relative error up to 1.5e-5 (1-bit codes; the
    # distances are small differences of 32-bit sums), largest error 5e-5, 7e-4 of the ids (two estimates that tie).
    # A query digit on a rounding boundary that falls the other way moves that query's 1-bit estimates by more.
    return {"rel": 6e-5, "max": 2e-3, "differ": 3e-3}
