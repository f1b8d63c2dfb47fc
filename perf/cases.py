"""What this library's users have it do, as cases that can be timed and compared.

A case is a dict of plain values.  Five kinds of work, one per "kind":

  knn     a query batch against a resident index: probe selection, query ordering, the fused
          scan (distance tables, bound, refine, top-k)
  range   the same with a radius instead of k; results in CSR form
  build   what storing a base set costs once the centroids are trained: list assignment,
          encoding, scan layouts, list summaries
  train   Lloyd's k-means for the PQ codebooks and the coarse lists
  gamma   the relaxation parameter from a confidence level, by sampling

Vectors are seeded Gaussian mixtures of the shapes and laws that synth.py describes (clip255,
aniso01, unit), drawn on the GPU.  An index is trained, encoded and laid out in list order with
the library's own entry points, as a program that keeps one does before it takes queries.
"""
import math

import torch

from paper_2508_17828_amd import trim

DEV = "cuda:0"

# (d, M, law): vector length, subspaces of 8-bit codes, law of the mixture.  The shapes are those of
# the workloads in synth.py and of the data sets in the benchmark spec (100-, 256-dimensional).
SHAPES = ((128, 32, "clip255"), (100, 20, "clip255"), (128, 16, "clip255"), (256, 64, "clip255"),
          (384, 48, "clip255"), (768, 96, "unit"), (960, 120, "aniso01"), (1536, 192, "unit"))


def _knn(name, n, d, M, law, nlist, nprobe, nq, k, gamma, batch=1024, bits=8):
    return dict(name=name, kind="knn", n=n, d=d, M=M, law=law, nlist=nlist, nprobe=nprobe, nq=nq, k=k,
                gamma=gamma, batch=batch, bits=bits)


def _range(name, n, d, M, law, nlist, nprobe, nq, percent, gamma, keep, bits=8):
    return dict(name=name, kind="range", n=n, d=d, M=M, law=law, nlist=nlist, nprobe=nprobe, nq=nq,
                percent=percent, gamma=gamma, keep=keep, bits=bits)


def listed():
    return [
        # one user waits for one answer: latency of the whole call chain
        _knn("knn one query", 1_000_000, 128, 32, "clip255", 1024, 32, 1, 10, 0.45),
        # a service that gathers the requests of a few milliseconds: fewer queries than the chip has CUs
        _knn("knn 67 queries 384d", 500_003, 384, 48, "clip255", 1024, 64, 67, 10, 0.2),
        # word vectors, sub-vectors of five values, a hundred neighbours for a re-ranker
        _knn("knn 100d k=100", 1_180_000, 100, 20, "clip255", 1024, 32, 1000, 100, 0.3),
        # the benchmark's configuration: a large query set over SIFT-like vectors
        _knn("knn 10000 queries 128d", 1_000_000, 128, 32, "clip255", 1024, 32, 10_000, 10, 0.45),
        # the same data with 4-bit codes
        _knn("knn 4-bit codes", 1_000_000, 128, 64, "clip255", 1024, 32, 3001, 10, 0.4, bits=4),
        # text embeddings, long rows
        _knn("knn embeddings 768d", 500_000, 768, 96, "unit", 1024, 64, 2500, 10, 0.6),
        # no lists: every vector is a candidate of every query (GIST-like, ground-truth style)
        _knn("knn exhaustive 960d k=100", 300_000, 960, 120, "aniso01", 0, 0, 500, 100, 0.3, batch=512),
        # a few look-alike searches whose answer size nobody knows beforehand
        _range("range 33 queries 128d", 100_000, 128, 32, "clip255", 128, 16, 33, 0.1, 0.4, False),
        # near-duplicate search over long embeddings, buffers and tables kept between calls
        _range("range embeddings 1536d", 250_000, 1536, 192, "unit", 512, 64, 2000, 0.1, 0.7, True),
        # a base set arrives: assign, encode, lay out
        dict(name="build 1M 128d", kind="build", n=1_000_000, d=128, M=32, law="clip255", nlist=1024, bits=8),
        # centroids are trained (again)
        dict(name="train 128d", kind="train", n=65_536, d=128, M=32, law="clip255", nlist=1024, iters=10, bits=8),
        # the relaxation parameter is calibrated on a sample
        dict(name="gamma 1000 x 10000", kind="gamma", n=100_000, d=128, M=32, law="clip255", rows=1000,
             queries=10_000, p=0.9, bits=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes log-uniform over the ranges above, list counts near sqrt(n) and as odd as
    they come, no more code bytes to scan than the largest listed search."""
    kind = rng.choice(("knn",) * 6 + ("range",) * 2 + ("build", "build", "train", "gamma"))
    d, M, law = rng.choice(SHAPES)
    bits = 8
    if d % 32 == 0 and rng.random() < 0.2:
        bits, M = 4, d // 2
    n = _log(rng, 20_000, min(1_000_000, 500_000_000 // d))
    nlist = max(16, int(math.sqrt(n) * rng.uniform(0.7, 1.4)))
    if kind == "build":
        n = min(n, 128_000_000 // d)
        return dict(kind=kind, n=n, d=d, M=M, law=law, nlist=nlist, bits=bits)
    if kind == "train":
        ns = _log(rng, 4096, min(65_536, 8_388_608 // d))
        return dict(kind=kind, n=ns, d=d, M=M, law=law, nlist=max(16, ns // 64), iters=rng.randint(4, 10), bits=bits)
    if kind == "gamma":
        d, M, law = rng.choice(SHAPES[:6])
        return dict(kind=kind, n=20_000, d=d, M=M, law=law, rows=_log(rng, 100, 1000),
                    queries=min(_log(rng, 500, 10_000), 1_280_000 // d), p=round(rng.uniform(0.5, 0.99), 2), bits=8)
    whole = law == "aniso01" and kind == "knn" and bits == 8
    nprobe = 0 if whole else max(1, min(64, int(nlist * math.exp(rng.uniform(math.log(1 / 64), math.log(1 / 8))))))
    code = (M if bits == 8 else M // 2) + 4
    share = 1.0 if whole else nprobe / nlist
    most = int(1.0e10 / (n * share * code))
    nq = max(1, min(_log(rng, 1, 10_000), most))
    gamma = round(rng.uniform(0.0, 0.6), 2)
    if kind == "range":
        nq = min(nq, 2000, max(1, int(1e9 / (n * share))))
        return dict(kind=kind, n=n, d=d, M=M, law=law, nlist=nlist, nprobe=nprobe, nq=nq,
                    percent=rng.choice((0.01, 0.1)), gamma=gamma, keep=rng.random() < 0.5, bits=bits)
    return dict(kind=kind, n=n, d=d, M=M, law=law, nlist=0 if whole else nlist, nprobe=nprobe, nq=nq,
                k=rng.choice((1, 10, 10, 50, 100)), gamma=gamma, batch=rng.choice((256, 512, 1024, 1024)), bits=bits)


# ---- inputs ----

def _vectors(case, means, count, gen):
    """`count` draws from the mixture, float32 [count][d]."""
    d, law = case["d"], case["law"]
    out = torch.empty((count, d), device=DEV)
    for lo in range(0, count, 131_072):
        z = out[lo:lo + 131_072]
        z.normal_(generator=gen)
        at = torch.randint(0, means.shape[0], (z.shape[0],), device=DEV, generator=gen)
        if law == "clip255":
            z.mul_(20.0).add_(means[at]).clamp_(0.0, 255.0)
        elif law == "aniso01":
            z.mul_(0.1 / torch.arange(1, d + 1, device=DEV).sqrt()).add_(means[at]).clamp_(0.0, 1.0)
        else:
            z.mul_(1.0 / math.sqrt(d)).add_(means[at])
            z.div_(z.norm(dim=1, keepdim=True))
    return out


def _means(case, gen):
    d, law = case["d"], case["law"]
    ncomp = max(16, case["n"] // {"clip255": 1000, "aniso01": 2000, "unit": 4000}[law])
    if law == "unit":
        mu = torch.randn((ncomp, d), device=DEV, generator=gen)
        return mu / mu.norm(dim=1, keepdim=True)
    mu = torch.rand((ncomp, d), device=DEV, generator=gen)
    if law == "clip255":
        return mu * 255.0
    return 0.5 + 0.5 * (2.0 * mu - 1.0) / torch.arange(1, d + 1, device=DEV).sqrt()


def _rows(gen, n, count):
    """`count` distinct row numbers below n, int32."""
    return torch.randperm(n, device=DEV, generator=gen)[:count].to(torch.int32)


def _train_pq(case, train, iters, gen):
    init = _rows(gen, train.shape[0], 256 if case["bits"] == 8 else 16)
    fn = trim.trim_train_pq if case["bits"] == 8 else trim.trim_fs_train_pq
    return fn(train, case["M"], iters, init)


def _encode(case, base, codebooks):
    return (trim.trim_encode if case["bits"] == 8 else trim.trim_fs_encode)(base, codebooks)


def _lay_out(index):
    """The optional scan layouts, where the code length has them (as index_setup.py does)."""
    bytes_per_code = index.codes.shape[1]
    if bytes_per_code % 8 == 0:
        index.scan_head = trim.trim_pack_scan_head(index.codes, index.dlx)
    if bytes_per_code >= 64 and bytes_per_code % 16 == 0:
        index.codes_tiled = trim.trim_pack_codes_tiled(index.codes)
    if index.list_offsets is not None:
        index.list_bounds = trim.trim_pack_list_bounds(index)
    return index


def _in_list_order(base, centroids, nlist):
    """(base in list order, original ids, list offsets, longest list)."""
    at = trim.trim_ivf_probe(base, centroids, 1)[:, 0].long()
    order = torch.argsort(at, stable=True)
    counts = torch.bincount(at, minlength=nlist)
    offsets = torch.zeros((nlist + 1,), dtype=torch.int64, device=DEV)
    offsets[1:] = torch.cumsum(counts, 0)
    return base[order].contiguous(), order.to(torch.int32), offsets, int(counts.max())


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    means = _means(case, gen)
    base = _vectors(case, means, case["n"], gen)
    kind = case["kind"]
    if kind == "train":
        return dict(case=case, train=base, lists=_rows(gen, case["n"], case["nlist"]),
                    rows=_rows(gen, case["n"], 256 if case["bits"] == 8 else 16))
    train = base[:16_384]
    codebooks = _train_pq(case, train, 3, gen)
    if kind == "gamma":
        codes, dlx = _encode(case, base, codebooks)
        return dict(case=case, index=trim.Index(base, codes, dlx, codebooks), rows=_rows(gen, case["n"], case["rows"]),
                    queries=_vectors(case, means, case["queries"], gen))
    nlist, centroids, ids, offsets, longest = case["nlist"], None, None, None, 0
    if nlist:
        sample = base[:max(32 * nlist, 1024)]
        centroids = trim.trim_train_ivf(sample, nlist, 3, _rows(gen, sample.shape[0], nlist))
        base, ids, offsets, longest = _in_list_order(base, centroids, nlist)
    if kind == "build":
        return dict(case=case, base=base, codebooks=codebooks, centroids=centroids, offsets=offsets, ids=ids,
                    longest=longest)
    codes, dlx = _encode(case, base, codebooks)
    index = _lay_out(trim.Index(base, codes, dlx, codebooks, ids=ids, list_offsets=offsets, max_list_len=longest,
                                code_bits=case["bits"]))
    state = dict(case=case, index=index, centroids=centroids, queries=_vectors(case, means, case["nq"], gen))
    if kind == "range":
        # the radius that encloses `percent` of the pairs of a sample
        few = _vectors(case, means, 512, gen)
        many = base[torch.randint(0, case["n"], (8192,), device=DEV, generator=gen)]
        d2 = torch.cdist(few, many).flatten().sort().values
        state["radius"] = float(d2[int(d2.numel() * case["percent"] / 100)])
        # what the answers are collected in for whoever asked
        most = int(8 * case["nq"] * case["n"] * case["percent"] / 100) + 100_000
        state["answer"] = torch.zeros((most,), dtype=torch.int32, device=DEV), torch.zeros((most,), device=DEV)
        if case["keep"]:
            state["capacity"] = most
            most = min(case["n"], case["nprobe"] * longest)
            state["workspace"] = torch.empty((trim.trim_range_workspace_bytes(case["nq"], most),), dtype=torch.uint8,
                                             device=DEV)
            if case["bits"] == 8 and case["M"] > 128:   # tables longer than the LDS are built ahead of the scan
                state["lut"] = torch.empty((case["nq"], case["M"], 256), device=DEV)
    return state


# ---- one pass ----

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "train":
        fn = trim.trim_train_pq if case["bits"] == 8 else trim.trim_fs_train_pq
        return dict(codebooks=fn(state["train"], case["M"], case["iters"], state["rows"]),
                    centroids=trim.trim_train_ivf(state["train"], case["nlist"], case["iters"], state["lists"]))
    if kind == "gamma":
        gamma, each = trim.trim_estimate_gamma(state["index"], state["rows"], state["queries"], case["p"])
        return dict(gamma=gamma, each=each)
    if kind == "build":
        assign = trim.trim_ivf_probe(state["base"], state["centroids"], 1)
        codes, dlx = _encode(case, state["base"], state["codebooks"])
        index = _lay_out(trim.Index(state["base"], codes, dlx, state["codebooks"], ids=state["ids"],
                                    list_offsets=state["offsets"], max_list_len=state["longest"],
                                    code_bits=case["bits"]))
        return dict(assign=assign, codes=codes, dlx=dlx, head=index.scan_head, tiled=index.codes_tiled,
                    bounds=_defined(index.list_bounds, case["nlist"], codes.shape[1]))
    index, queries = state["index"], state["queries"]
    probes = order = None
    if case["nlist"]:
        probes = trim.trim_ivf_probe(queries, state["centroids"], case["nprobe"])
        if case["nq"] > 1:
            order = trim.trim_query_order(probes, case["nlist"])
    if kind == "knn":
        r = trim.trim_search_knn(index, queries, case["k"], case["gamma"], case["batch"], probes=probes,
                                 query_order=order)
        return dict(ids=r["ids"], d2=r["d2"], n_scanned=r["n_scanned"], n_exact=r["n_exact"])
    lut = trim.trim_build_lut(queries, index.codebooks, out=state["lut"]) if "lut" in state else None
    r = trim.trim_search_range(index, queries, state["radius"], case["gamma"], probes=probes, query_order=order,
                               lut=lut, capacity=state.get("capacity", 0), workspace=state.get("workspace"))
    ids, d2 = state["answer"]
    ids[:r["required"]] = r["ids"]
    d2[:r["required"]] = r["d2"]
    return dict(offsets=r["offsets"], ids=ids, d2=d2, n_scanned=r["n_scanned"], n_exact=r["n_exact"])


def _defined(bounds, nlist, code_bytes):
    """The part of the list summaries that the format defines (a record ends in padding)."""
    return bounds.view(nlist, -1)[:, :65 * code_bytes]


def work(case):
    """Bytes and operations of one pass: every input and every result once, one subtraction and one
    multiply-add per coordinate of a distance, one addition per code of a scanned candidate."""
    n, d, M, bits = case["n"], case["d"], case["M"], case["bits"]
    cent = 256 if bits == 8 else 16
    code = M if bits == 8 else M // 2
    books = 4 * d * cent
    kind = case["kind"]
    if kind == "train":
        it, nlist = case["iters"], case["nlist"]
        return dict(bytes=4 * n * d + books + 4 * nlist * d, flops=3.0 * it * n * d * (cent + nlist))
    if kind == "gamma":
        pairs = case["rows"] * case["queries"]
        return dict(bytes=4 * d * (case["rows"] + case["queries"]) + books + case["rows"] * (M + 4), flops=5.0 * pairs * d)
    if kind == "build":
        nlist = case["nlist"]
        layouts = (12 if code % 8 == 0 else 0) + (code if code >= 64 and code % 16 == 0 else 0)
        return dict(bytes=n * (4 * d + code + 8 + layouts) + books + nlist * (4 * d + 65 * code),
                    flops=3.0 * n * d * (cent + nlist))
    nq, nlist = case["nq"], case["nlist"]
    per = n * case["nprobe"] / nlist if nlist else n
    seen = min(n, nq * per)
    results = nq * case["k"] if kind == "knn" else nq * n * case["percent"] / 100
    rows = min(n, results)
    return dict(bytes=seen * (code + 4) + rows * (4 * d + 4) + books + nlist * 4 * d + nq * 4 * d + 8 * results,
                flops=3.0 * nq * d * (cent + nlist) + nq * per * M + 3.0 * results * d)


def tolerance(case):
    """The header fixes every rounding of the searches, the encoder and the training, so their results
    are the same bit for bit; the sampled gamma is binary32 arithmetic in any order."""
    return {"rel": 1e-5, "max": 1e-4} if case["kind"] == "gamma" else "exact"
