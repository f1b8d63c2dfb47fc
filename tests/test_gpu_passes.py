"""The searches in passes (trim_search_knn_ws, trim_search_range_ws with their work space) against the
single kernel (trim_search_knn, trim_search_range), which the other GPU tests hold against the oracle: ids,
distances, counters, offsets and survivor masks are the same bit for bit."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2508_17828_amd import trim
    trim.lib()
    return trim


def built(T, n, d, M, bits, nlist, nq, nprobe, spread, offset, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    means = torch.randn((max(2, n // 300), d), device="cuda", generator=g) * spread

    def draw(count):
        at = torch.randint(0, means.shape[0], (count,), device="cuda", generator=g)
        return (torch.randn((count, d), device="cuda", generator=g) * 0.5 + means[at] + offset).contiguous()

    base, queries = draw(n), draw(nq)
    init = torch.randperm(n, device="cuda", generator=g)[: 256 if bits == 8 else 16].to(torch.int32)
    cb = (T.trim_train_pq if bits == 8 else T.trim_fs_train_pq)(base[:4096].contiguous(), M, 2, init % min(n, 4096))
    ids = offsets = probes = None
    longest = 0
    if nlist:
        cent = base[torch.randperm(n, device="cuda", generator=g)[:nlist]].contiguous()
        at = T.trim_ivf_probe(base, cent, 1)[:, 0].long()
        at[at == 1] = 0                                   # an empty list
        order = torch.argsort(at, stable=True)
        offsets = torch.zeros((nlist + 1,), dtype=torch.int64, device="cuda")
        offsets[1:] = torch.cumsum(torch.bincount(at, minlength=nlist), 0)
        longest = int((offsets[1:] - offsets[:-1]).max())
        base, ids = base[order].contiguous(), order.to(torch.int32)
        probes = T.trim_ivf_probe(queries, cent, nprobe)
        probes[3, 1] = probes[3, 0]                       # a list twice
        probes[5, 0] = nlist + 7                          # no such list
        probes[6, :] = 1                                  # nothing to scan
    codes, dlx = (T.trim_encode if bits == 8 else T.trim_fs_encode)(base, cb)
    ix = T.Index(base, codes, dlx, cb, ids=ids, list_offsets=offsets, max_list_len=longest, code_bits=bits)
    if codes.shape[1] % 8 == 0:
        ix.scan_head = T.trim_pack_scan_head(codes, dlx)
    if nlist:
        ix.list_bounds = T.trim_pack_list_bounds(ix)
    return ix, queries, probes


def single_kernel(T, ix, q, k, gamma, batch, probes, order, lut=None):
    import torch
    nq = q.shape[0]
    ids = torch.full((nq, k), -7, dtype=torch.int32, device="cuda")
    d2 = torch.full((nq, k), -7.0, device="cuda")
    ns, ne = torch.zeros((2, nq), dtype=torch.int32, device="cuda").unbind(0)
    cand, mc = ix._cand(probes)
    mw = (mc + 31) // 32
    mask = torch.zeros((nq, mw), dtype=torch.int32, device="cuda")
    view, stats = ix._view(), T._Stats(ns.data_ptr(), ne.data_ptr(), None)
    p = lambda t: None if t is None else C.c_void_p(t.data_ptr())
    rc = T.lib().trim_search_knn(C.byref(view), p(q), nq, p(lut), C.byref(cand) if cand is not None else None, k, gamma, batch,
                                 p(order), p(ids), p(d2), C.byref(stats), p(mask), mw,
                                 C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    return dict(ids=ids, d2=d2, n_scanned=ns, n_exact=ne, mask=mask)


# every padded sub-vector length; 4-bit codes; with and without lists; result sets of every width;
# batches of a few and of thousands; gamma 0, between, above 1; rows and queries that leave tiles unfilled
CASES = [
    # n, d, M, bits, nlist, nq, nprobe, k, batch, gamma, spread, offset
    (5000, 600, 120, 8, 0, 257, 0, 100, 1, 0.7, 1.0, 3.0),
    (20000, 512, 128, 8, 40, 300, 12, 10, 512, 0.5, 1.0, 0.0),
    (20000, 768, 96, 8, 33, 300, 9, 10, 1024, 0.2, 0.3, 10.0),
    (12000, 800, 160, 8, 20, 270, 7, 100, 300, 0.6, 0.2, 0.0),
    (15000, 768, 96, 8, 0, 260, 0, 100, 512, 0.3, 0.3, 0.0),
    (9000, 512, 32, 8, 16, 290, 16, 300, 4096, 1.5, 0.5, 0.0),
    (6000, 512, 16, 8, 10, 259, 4, 1, 7, 0.0, 0.5, 0.0),
    (10000, 512, 256, 4, 24, 400, 8, 10, 256, 0.4, 0.5, 0.0),
    (7000, 1536, 192, 8, 12, 261, 6, 64, 1000, 0.7, 0.1, 0.0),
    (66000, 528, 44, 8, 0, 261, 0, 10, 512, 0.4, 0.3, 0.0),          # rows for every CU, sub-vectors of 12
    (5000, 544, 136, 8, 5, 300, 4, 10, 512, 0.4, 0.3, 0.0),          # lists of more than one tile, 240 queries each
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_passes_equal_the_single_kernel(T, case):
    import torch
    n, d, M, bits, nlist, nq, nprobe, k, batch, gamma, spread, offset = case
    ix, q, probes = built(T, n, d, M, bits, nlist, nq, nprobe, spread, offset, n + d)
    cand, _ = ix._cand(probes)
    view = ix._view()
    assert T.lib().trim_knn_workspace_bytes(C.byref(view), nq, C.byref(cand) if cand is not None else None, k, batch) > 0
    order = torch.randperm(nq, device="cuda").to(torch.int32)
    order[2] = nq + 5                                    # a query that is not named
    missing = sorted(set(range(nq)) - set(order.tolist()))
    for o in (None, order):
        want = single_kernel(T, ix, q, k, gamma, batch, probes, o)
        out = (torch.full((nq, k), -7, dtype=torch.int32, device="cuda"), torch.full((nq, k), -7.0, device="cuda"))
        got = T.trim_search_knn(ix, q, k, gamma, batch, probes=probes, want_mask=True, out=out, query_order=o)
        rows = np.array([i for i in range(nq) if o is None or i not in missing])
        for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
            a, b = got[name].cpu().numpy(), want[name].cpu().numpy()
            np.testing.assert_array_equal(a[rows], b[rows], err_msg=name)
        np.testing.assert_array_equal(got["ids"].cpu().numpy(), want["ids"].cpu().numpy())


# first batches whose end lies inside a word of marks and at its edge; more passes after them (few vectors for the queries: each pass is measured by itself)
@pytest.mark.parametrize("k,batch", ((1, 4), (1, 3), (10, 40), (10, 39), (8, 1016), (10, 1030), (64, 300), (128, 512), (129, 516), (3, 4096)))
def test_first_batch_with_the_next_pass(T, k, batch):
    test_passes_equal_the_single_kernel(T, (16000, 768, 96, 8, 20, 280, 9, k, batch, 0.4, 0.3, 0.0))


# pick_kernel at the edges of its rule: results and vectors of the batch per result; batches with which the next pass is short and not, largest
# batch, 16 vectors a query (24,960 = 1560 * 16) and one query more; batches of fewer vectors than picks and than results; candidates cut
# before there are as many as picks, and inside the first batch
@pytest.mark.parametrize("k,batch,nq,cut", ((1, 1, 260, 0), (10, 5, 260, 0), (10, 512, 300, 0), (11, 44, 260, 0), (11, 43, 260, 0), (128, 512, 260, 0),
                                            (129, 516, 260, 0), (10, 1013, 260, 0), (10, 1014, 260, 0), (11, 1013, 260, 0),
                                            (10, 1024, 1560, 0), (2, 1024, 260, 0), (10, 1025, 260, 0), (10, 1024, 1561, 0), (10, 600, 260, 1034), (10, 600, 260, 611),
                                            (10, 1024, 260, 70), (100, 400, 260, 170), (9, 512, 260, 23)))
def test_picked_threshold(T, k, batch, nq, cut, monkeypatch):
    if cut:
        plain = T.Index._cand
        monkeypatch.setattr(T.Index, "_cand", lambda self, p, max_candidates=0: plain(self, p, cut))
    for spread, gamma in ((0.3, 0.3), (0.05, 0.1)):
        test_passes_equal_the_single_kernel(T, (24960, 512, 64, 8, 20, nq, 9, k, batch, gamma, spread, 0.0))


@pytest.mark.parametrize("what", ("landmark distances", "rows", "queries", "centroids", "table"))
def test_picked_threshold_with_values_that_are_no_numbers(T, what):
    ix, q, probes = built(T, 24960, 512, 128, 8, 12, 260, 7, 0.5, 0.0, 11)
    ix.list_bounds = None
    table = T.trim_build_lut(q, ix.codebooks) if what == "table" else None
    plant(what, ix, q, table)
    for l in range(12):                       # in the first candidates of every list, whichever comes first
        at = int(ix.list_offsets[l])
        if what == "rows" and at + 400 < 24960:
            ix.base[at + 20:at + 400:37, 3] = float("nan")
            ix.base[at + 25:at + 400:41, 3] = float("inf")
        if what == "landmark distances" and at + 400 < 24960:
            ix.dlx[at + 20:at + 400:37] = float("nan")
            ix.dlx[at + 25:at + 400:41] = float("inf")
    ix.scan_head = T.trim_pack_scan_head(ix.codes, ix.dlx)
    for k, batch in ((1, 20), (1, 512), (10, 1024)):
        want = single_kernel(T, ix, q, k, 0.4, batch, probes, None, table)
        got = T.trim_search_knn(ix, q, k, 0.4, batch, probes=probes, lut=table, want_mask=True)
        for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
            np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=f"{name}, {k}, {batch}")


# no lists and rows enough for 512 queries by 128 rows at a time (measure_kernel): queries that fill a block, leave one idle and begin a
# second, a last tile of a few rows, an uneven number of pairs of slices; the short stretches before take 128 by 128
@pytest.mark.parametrize("n,d,M,nq,batch", ((30000, 528, 44, 320, 64), (30103, 544, 68, 515, 64), (50000, 600, 120, 512, 1024), (28100, 1024, 32, 319, 64)))
def test_many_queries_without_lists(T, n, d, M, nq, batch):
    test_passes_equal_the_single_kernel(T, (n, d, M, 8, 0, nq, 0, 10, batch, 0.3, 0.3, 0.0))


# a last tile of one to four blocks of 32 queries (the filter has a loop for each), rows that leave waves of the last row tile idle,
# an uneven number of code words, sub-vectors of every padded length
@pytest.mark.parametrize("nq", (288, 320, 350, 384))
@pytest.mark.parametrize("d,M,bits,nlist", ((544, 68, 8, 0), (512, 128, 8, 3), (528, 44, 8, 0), (640, 20, 8, 0), (640, 320, 4, 3)))
def test_tiles_of_one_to_four_blocks_of_queries(T, nq, d, M, bits, nlist):
    test_passes_equal_the_single_kernel(T, (2300, d, M, bits, nlist, nq, nlist, 10, 300, 0.3, 0.4, 0.0))


# few queries (bounds by many workgroups, one to settle): one query; first batches measured beside the bounds and not
# (the three largest); codes of every width; table phases; more results than candidates
FEW = [
    (3000, 128, 32, 8, 12, 8, 5, 10, 256, 0.4, 2.0, 0.0),
    (40000, 64, 16, 8, 40, 67, 19, 10, 64, 0.0, 1.0, 0.0),
    (25000, 100, 20, 8, 0, 9, 0, 100, 1, 0.7, 1.0, 3.0),
    (70000, 256, 64, 8, 0, 11, 0, 10, 1024, 0.2, 0.3, 0.0),
    (20000, 768, 96, 8, 33, 30, 9, 10, 1024, 0.2, 0.3, 10.0),
    (9000, 1536, 192, 8, 12, 8, 6, 64, 1000, 0.7, 0.1, 0.0),
    (9000, 512, 32, 8, 16, 100, 16, 300, 3796, 1.5, 0.5, 0.0),
    (6000, 256, 4, 8, 10, 100, 4, 5, 64, 0.3, 0.5, 0.0),
    (10000, 256, 128, 4, 24, 60, 8, 10, 256, 0.4, 0.5, 0.0),
    (2000, 128, 64, 4, 10, 9, 3, 1000, 512, 0.6, 0.5, 0.0),
    (3000, 96, 12, 8, 300, 9, 2, 64, 100, 0.3, 0.5, 0.0),
]


@pytest.mark.parametrize("case", FEW, ids=lambda c: "-".join(map(str, c)))
def test_few_queries_equal_the_single_kernel(T, case):
    import torch
    n, d, M, bits, nlist, nq, nprobe, k, batch, gamma, spread, offset = case
    ix, queries, probes = built(T, n, d, M, bits, nlist, nq, nprobe, spread, offset, n + d)
    cand, _ = ix._cand(probes)
    view = ix._view()
    for count in (nq, 1):
        q = queries[:count].contiguous()
        pr = None if probes is None else probes[:count].contiguous()
        assert T.lib().trim_knn_workspace_bytes(C.byref(view), count, C.byref(cand) if cand is not None else None, k, batch) > 0
        order = torch.randperm(count, device="cuda").to(torch.int32)
        if count > 2:
            order[2] = count + 5
        named = np.array(sorted(set(range(count)) & set(order.tolist())))
        lut = (T.trim_build_lut if bits == 8 else T.trim_fs_build_lut)(q, ix.codebooks) * 0.9
        for o, table in ((None, None), (order, lut)):
            want = single_kernel(T, ix, q, k, gamma, batch, pr, o, table)
            out = (torch.full((count, k), -7, dtype=torch.int32, device="cuda"), torch.full((count, k), -7.0, device="cuda"))
            got = T.trim_search_knn(ix, q, k, gamma, batch, probes=pr, lut=table, want_mask=True, out=out, query_order=o)
            rows = np.arange(count) if o is None else named
            for name in ("n_scanned", "n_exact", "mask"):
                np.testing.assert_array_equal(got[name].cpu().numpy()[rows], want[name].cpu().numpy()[rows], err_msg=name)
            for name in ("ids", "d2"):
                np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)


# few queries over long rows, measured by many workgroups pass by pass: results of every width, passes that begin after 2 and after 4096
# candidates, inside a group of 64 and at its edge, one candidate after the first batch and none; more lookups than without passes; with the
# work space that a search without passes takes, and a byte less than either
@pytest.mark.parametrize("case", [
    (3000, 512, 128, 8, 0, 20, 0, 1, 1, 0.3, 0.3, 0.0),
    (3000, 512, 128, 8, 20, 20, 7, 10, 54, 0.0, 0.3, 0.0),
    (9000, 528, 44, 8, 12, 33, 6, 100, 7, 0.5, 0.3, 3.0),
    (20000, 768, 96, 8, 33, 128, 33, 65, 447, 0.2, 0.2, 0.0),
    (20000, 1536, 192, 8, 0, 9, 0, 300, 1000, 0.1, 0.2, 0.0),
    (9000, 640, 320, 4, 16, 12, 9, 1000, 3096, 0.4, 0.5, 0.0),
    (9000, 640, 320, 4, 16, 12, 14, 1000, 3096, 0.4, 0.5, 0.0),
    (1035, 512, 32, 8, 0, 7, 0, 10, 1024, 0.2, 0.5, 0.0),
    (1034, 512, 32, 8, 0, 7, 0, 10, 1024, 0.2, 0.5, 0.0),
    (40000, 1024, 256, 8, 0, 27, 0, 128, 512, 0.3, 0.2, 0.0),
    (20000, 768, 384, 4, 33, 50, 33, 10, 300, 0.2, 0.2, 0.0),        # (with lists no more lookups than without passes: that many)
], ids=lambda c: "-".join(map(str, c)))
def test_few_queries_over_long_rows(T, case):
    import torch
    test_few_queries_equal_the_single_kernel(T, case)
    n, d, M, bits, nlist, nq, nprobe, k, batch, gamma, spread, offset = case
    ix, q, probes = built(T, n, d, M, bits, nlist, nq, nprobe, spread, offset, n + d)
    cand, _ = ix._cand(probes)
    view = ix._view()
    p = lambda t: None if t is None else C.c_void_p(t.data_ptr())
    pc = C.byref(cand) if cand is not None else None
    need = T.lib().trim_knn_workspace_bytes(C.byref(view), nq, pc, k, batch)
    want = single_kernel(T, ix, q, k, gamma, batch, probes, None)
    for size in (need, need - 1, need // 2, 0):
        ws = torch.full((need + 256,), 0xa5, dtype=torch.uint8, device="cuda")
        ids, d2 = torch.full((nq, k), -7, dtype=torch.int32, device="cuda"), torch.full((nq, k), -7.0, device="cuda")
        rc = T.lib().trim_search_knn_ws(C.byref(view), p(q), nq, None, pc, k, gamma, batch, None, p(ids), p(d2), None, None, 0, p(ws), size,
                                        C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == 0
        assert torch.equal(ids, want["ids"]) and torch.equal(d2, want["d2"]), size
        assert (ws[size:] == 0xa5).all()
    order = torch.arange(nq, dtype=torch.int32, device="cuda")
    order[nq - 1], order[nq // 2] = 0, 1                 # queries twice, at other places than their own; two that are not named
    named = [i for i in range(nq) if i not in (nq - 1, nq // 2)]
    want = single_kernel(T, ix, q, k, gamma, batch, probes, None)
    out = (torch.full((nq, k), -7, dtype=torch.int32, device="cuda"), torch.full((nq, k), -7.0, device="cuda"))
    got = T.trim_search_knn(ix, q, k, gamma, batch, probes=probes, want_mask=True, out=out, query_order=order)
    for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
        assert torch.equal(got[name][named], want[name][named]), name
    for t in out:
        assert (t[nq - 1] == -7).all() and (t[nq // 2] == -7).all()


# survivors few and far between, at the ends of the stretches that are looked at together and of their groups of 64; result sets of
# both block sizes (1024 and 512 threads: other stretches); after results that fill up late
@pytest.mark.parametrize("k,batch", ((10, 64), (300, 100)))
@pytest.mark.parametrize("near", ((16455, 16456, 278599, 278600, 599_999), (8592, 74127, 74128, 300_031, 300_032), ()))
def test_few_survivors_among_many_candidates(T, k, batch, near):
    import torch
    n, d, nq, gamma = 600_000, 16, 2, 0.3
    g = torch.Generator(device="cuda").manual_seed(len(near) + k)
    base = torch.randn((n, d), device="cuda", generator=g) + 20
    base[:k] -= 19
    at = torch.tensor(near, device="cuda", dtype=torch.long)
    base[at] = torch.randn((len(near), d), device="cuda", generator=g) * 0.1
    q = torch.randn((nq, d), device="cuda", generator=g) * 0.1
    cb = T.trim_train_pq(base[:4096].contiguous(), 4, 2, torch.randperm(4096, device="cuda", generator=g)[:256].to(torch.int32))
    codes, dlx = T.trim_encode(base, cb)
    ix = T.Index(base, codes, dlx, cb)
    assert T.lib().trim_knn_workspace_bytes(C.byref(ix._view()), nq, None, k, batch) > 0
    for count in (nq, 1):
        want = single_kernel(T, ix, q[:count], k, gamma, batch, None, None)
        got = T.trim_search_knn(ix, q[:count], k, gamma, batch, want_mask=True)
        for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
            np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)
        assert set(near) <= set(got["ids"][0].tolist())


def single_range(T, ix, q, radius, gamma, probes, order, lut):
    import torch
    nq = q.shape[0]
    ns, ne = torch.zeros((2, nq), dtype=torch.int32, device="cuda").unbind(0)
    cand, mc = ix._cand(probes)
    mw = (mc + 31) // 32
    mask = torch.zeros((nq, mw), dtype=torch.int32, device="cuda")
    offsets = torch.zeros((nq + 1,), dtype=torch.int64, device="cuda")
    required = torch.zeros((1,), dtype=torch.int64, device="cuda")
    view, stats = ix._view(), T._Stats(ns.data_ptr(), ne.data_ptr(), None)
    ws = torch.empty((T.trim_range_workspace_bytes(nq, mc),), dtype=torch.uint8, device="cuda")
    p = lambda t: None if t is None else C.c_void_p(t.data_ptr())
    cap = 8_000_000
    ids = torch.empty((cap,), dtype=torch.int32, device="cuda")
    d2 = torch.empty((cap,), device="cuda")
    rc = T.lib().trim_search_range(C.byref(view), p(q), nq, p(lut), C.byref(cand) if cand is not None else None, radius, gamma,
                                   p(order), p(offsets), p(ids), p(d2), cap, p(required), C.byref(stats), p(mask), mw,
                                   p(ws), ws.numel(), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    r = int(required)
    assert r < cap
    return dict(offsets=offsets, ids=ids[:r], d2=d2[:r], n_scanned=ns, n_exact=ne, mask=mask)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("percent", (0.05, 5.0))
def test_range_in_passes_equals_the_single_kernel(T, case, percent):
    import torch
    n, d, M, bits, nlist, nq, nprobe, _, _, gamma, spread, offset = case
    ix, q, probes = built(T, n, d, M, bits, nlist, nq, nprobe, spread, offset, n + d)
    cand, _ = ix._cand(probes)
    view = ix._view()
    assert T.lib().trim_range_scratch_bytes(C.byref(view), nq, C.byref(cand) if cand is not None else None) > 0
    radius = float(torch.quantile(torch.cdist(q[:64], ix.base).flatten()[:4_000_000].cpu().double(), percent / 100))
    lut = (T.trim_build_lut if bits == 8 else T.trim_fs_build_lut)(q, ix.codebooks)
    other = lut.clone()
    other[4:9] *= 0.75                                   # tables that are not the centroids' distances
    order = torch.randperm(nq, device="cuda").to(torch.int32)
    order[2] = nq + 5
    missing = (set(range(nq)) - set(order.tolist())).pop()
    for o, table in ((None, None), (order, None), (None, lut), (order, other)):
        want = single_range(T, ix, q, radius, gamma, probes, o, table)
        r = want["ids"].shape[0]
        for capacity in (0, r + 3):
            got = T.trim_search_range(ix, q, radius, gamma, probes=probes, lut=table, want_mask=True, query_order=o,
                                      capacity=capacity)
            rows = np.array([i for i in range(nq) if o is None or i != missing])
            for name in ("n_scanned", "n_exact", "mask"):
                np.testing.assert_array_equal(got[name].cpu().numpy()[rows], want[name].cpu().numpy()[rows], err_msg=name)
            for name in ("offsets", "ids", "d2"):
                np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)


@pytest.mark.parametrize("radius", (0.0, 1e-16, 2e15, float("inf")))
def test_range_in_passes_with_radii_that_settle_nothing(T, radius):
    """Squared radii out of the range in which the filter tells who passes for certain; tables made here, the centroids' and others."""
    import torch
    ix, q, probes = built(T, 5000, 1536, 192, 8, 12, 260, 6, 0.3, 0.0, 3)
    q[:200] = ix.base[torch.randperm(5000, device="cuda")[:200]]
    lut = T.trim_build_lut(q, ix.codebooks)
    lut[4:90] *= 0.75
    for table in (None, lut):
        want = single_range(T, ix, q, radius, 0.7, probes, None, table)
        got = T.trim_search_range(ix, q, radius, 0.7, probes=probes, lut=table, want_mask=True)
        for name in ("n_scanned", "n_exact", "mask", "offsets", "ids", "d2"):
            np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)


def host_index(ix):
    """The same stored data for the oracle."""
    from oracle import trim_oracle, trim_oracle_fs
    a = lambda t: None if t is None else np.ascontiguousarray(t.cpu().numpy())
    return (trim_oracle if ix.code_bits == 8 else trim_oracle_fs), \
        (trim_oracle if ix.code_bits == 8 else trim_oracle_fs).Index(a(ix.base), a(ix.codes), a(ix.dlx), a(ix.codebooks), ids=a(ix.ids),
                                                                     list_offsets=a(ix.list_offsets))


# The bounds of a stretch are taken 16,384 candidates at a time where two workgroups share a CU, and a step that marks
# nobody goes on to the next without listing anyone: a few vectors that matter, far behind tens of thousands that do not.
@pytest.mark.parametrize("M,bits", ((32, 8), (256, 4)))
def test_marks_that_begin_late(T, M, bits):
    import torch
    n, d, nq, k, batch, gamma = 70_000, 512, 260, 10, 512, 0.5
    g = torch.Generator(device="cuda").manual_seed(n + M)
    draw = lambda rows, far: (torch.randn((rows, d), device="cuda", generator=g) * 0.1 + far).contiguous()
    near = torch.tensor(list(range(k)) + [17_000, 20_001, 32_767, 32_768, 51_200, 51_201, 69_999], device="cuda")
    base = draw(n, 1.0)
    base[near] = draw(near.numel(), 0.0)
    queries = draw(nq, 0.0)
    train = torch.cat((base[near], base[torch.randperm(n, device="cuda", generator=g)[:4000]])).contiguous()
    init = torch.arange(256 if bits == 8 else 16, device="cuda", dtype=torch.int32)
    cb = (T.trim_train_pq if bits == 8 else T.trim_fs_train_pq)(train, M, 2, init)
    codes, dlx = (T.trim_encode if bits == 8 else T.trim_fs_encode)(base, cb)
    ix = T.Index(base, codes, dlx, cb, code_bits=bits)
    view = ix._view()
    assert T.lib().trim_knn_workspace_bytes(C.byref(view), nq, None, k, batch) > 0
    O, oix = host_index(ix)
    want = O.search_knn(oix, queries.cpu().numpy(), k, gamma, batch, want_mask=True)
    assert want["n_exact"].max() < 2000                    # the far ones are not marked
    got = T.trim_search_knn(ix, queries, k, gamma, batch, want_mask=True)
    for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
        np.testing.assert_array_equal(got[name].cpu().numpy().view(want[name].dtype), want[name], err_msg=name)
    radius = float(np.sqrt(want["d2"][:, -1].max()))
    want = O.search_range(oix, queries.cpu().numpy(), radius, gamma, want_mask=True)
    assert 0 < want["n_exact"].max() < 2000
    got = T.trim_search_range(ix, queries, radius, gamma, want_mask=True)
    for name in ("offsets", "ids", "d2", "n_scanned", "n_exact", "mask"):
        np.testing.assert_array_equal(got[name].cpu().numpy().view(want[name].dtype), want[name], err_msg=name)


# Everyone of a first batch that is measured beside the bounds is a survivor (gamma 0, one landmark for all): the waves that count
# and the one that goes on to sort must agree on how many there are.
@pytest.mark.parametrize("k,batch", ((10, 4086), (64, 4032), (100, 1500), (1000, 3096)))
def test_first_batches_of_many_survivors(T, k, batch):
    import torch
    n, d, M, nq = 5000, 64, 16, 40
    g = torch.Generator(device="cuda").manual_seed(k + batch)
    base = torch.randn((n, d), device="cuda", generator=g)
    queries = torch.randn((nq, d), device="cuda", generator=g)
    cb = torch.zeros((M, 256, d // M), device="cuda")
    codes, dlx = T.trim_encode(base, cb)
    ix = T.Index(base, codes, dlx, cb)
    O, oix = host_index(ix)
    want = O.search_knn(oix, queries.cpu().numpy(), k, 0.0, batch, want_mask=True)
    assert want["n_exact"].max() > 0.9 * n
    for _ in range(3):
        got = T.trim_search_knn(ix, queries, k, 0.0, batch, want_mask=True)
        for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
            np.testing.assert_array_equal(got[name].cpu().numpy().view(want[name].dtype), want[name], err_msg=name)


# Rows so long that the measure pass has no LDS for 256 queries at a time (24,576 values), or for 128 (26,752): the search is
# done with fewer, or by the single kernel.
@pytest.mark.parametrize("d,M", ((24576, 768), (26752, 836)))
def test_the_longest_rows(T, d, M):
    n, nq, nlist, nprobe, k, batch, gamma = 1500, 300, 3, 2, 10, 256, 0.4
    ix, q, probes = built(T, n, d, M, 8, nlist, nq, nprobe, 0.3, 0.0, d)
    for pr in (probes, None):
        want = single_kernel(T, ix, q, k, gamma, batch, pr, None)
        got = T.trim_search_knn(ix, q, k, gamma, batch, probes=pr, want_mask=True)
        for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
            np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)
        radius = float(np.sqrt(want["d2"][:, -1].cpu().numpy()[7:].max()))
        want = single_range(T, ix, q, radius, gamma, pr, None, None)
        got = T.trim_search_range(ix, q, radius, gamma, probes=pr, want_mask=True)
        for name in ("offsets", "ids", "d2", "n_scanned", "n_exact", "mask"):
            np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)


# A GPU without room for the work space: the single kernels do without it.
@pytest.mark.parametrize("nq", (1, 300))
def test_no_memory_for_the_work_space(T, nq, monkeypatch):
    import torch
    ix, queries, probes = built(T, 12000, 512, 128, 8, 70, 300, 12, 0.5, 0.0, 3)
    cent = ix.base[torch.randperm(12000, device="cuda")[:70]].contiguous()
    q, pr = queries[:nq].contiguous(), probes[:nq].contiguous()
    radius = float(torch.cdist(q, ix.base).quantile(0.01, dim=1).max().cpu())
    keep = torch.empty((T.trim_range_workspace_bytes(nq, 12000),), dtype=torch.uint8, device="cuda")

    def all_three():
        r = T.trim_search_range(ix, q, radius, 0.4, probes=pr, workspace=keep, capacity=3_000_000)
        s = T.trim_search_knn(ix, q, 10, 0.4, 512, probes=pr)
        return T.trim_ivf_probe(q, cent, 9), s["ids"], s["d2"], s["n_exact"], r["offsets"], r["ids"], r["d2"]

    assert T.lib().trim_ivf_probe_workspace_bytes(nq, 512, 70, 9) > 0
    want = all_three()
    empty = torch.empty

    def full(*size, **kw):
        if kw.get("dtype") is torch.uint8:
            raise torch.cuda.OutOfMemoryError("no room")
        return empty(*size, **kw)

    monkeypatch.setattr(torch, "empty", full)
    got = all_three()
    monkeypatch.undo()
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())


def test_centroids_far_apart(T):
    """Two groups of vectors 1e23 apart: the scale of the 16-bit operands comes from the distance between them, and its
    square is no binary32 number any more."""
    import torch
    n, d, M, nq, k, batch, gamma = 6000, 512, 128, 300, 10, 256, 0.3
    g = torch.Generator(device="cuda").manual_seed(5)
    base = torch.randn((n, d), device="cuda", generator=g)
    base[1::2] += 1e23
    queries = torch.randn((nq, d), device="cuda", generator=g)
    init = torch.arange(256, device="cuda", dtype=torch.int32)
    cb = T.trim_train_pq(base[:4096].contiguous(), M, 0, init)
    codes, dlx = T.trim_encode(base, cb)
    ix = T.Index(base, codes, dlx, cb)
    O, oix = host_index(ix)
    want = O.search_knn(oix, queries.cpu().numpy(), k, gamma, batch, want_mask=True)
    got = T.trim_search_knn(ix, queries, k, gamma, batch, want_mask=True)
    for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
        np.testing.assert_array_equal(got[name].cpu().numpy().view(want[name].dtype), want[name], err_msg=name)
    radius = float(np.sqrt(want["d2"][:, -1].max()))
    want = O.search_range(oix, queries.cpu().numpy(), radius, gamma, want_mask=True)
    got = T.trim_search_range(ix, queries, radius, gamma, want_mask=True)
    for name in ("offsets", "ids", "d2", "n_scanned", "n_exact", "mask"):
        np.testing.assert_array_equal(got[name].cpu().numpy().view(want[name].dtype), want[name], err_msg=name)


def plant(what, ix, q, table):
    """Infinities, NaN and values out of every 16-bit range where they do harm: among the seeds, in the first batch and later."""
    at = [2, 7, 40, 300, 700, 2000, 4999, 5003, 6000]
    nan, inf = float("nan"), float("inf")
    if what == "landmark distances":            # (as they come out for rows that hold such values)
        ix.dlx[at[0::3]] = nan
        ix.dlx[at[1::3]] = inf
        ix.dlx[at[2::3]] = 1e30
    elif what == "rows":                        # (landmark distances of other rows)
        ix.base[at[0::3], 5] = nan
        ix.base[at[1::3], 6] = inf
        ix.base[at[2::3], 7] = -1e30
    elif what == "queries":
        q[3, 5] = nan
        q[9, 100] = inf
        q[11, 200] = -1e30
        q[12] = 1e25
        q[13] *= 1e-30
    elif what == "centroids":
        ix.codebooks[0, 7] = nan
        ix.codebooks[3, 11, 1] = inf
        ix.codebooks[4, 12, 2] = 1e25
    elif what == "table":
        table[3, 0, ::7] = nan
        table[5, 1, ::9] = inf
        table[8] = inf
        table[9] = nan


SPECIAL = ("landmark distances", "rows", "queries", "centroids", "table")


@pytest.mark.parametrize("lists", (False, True))
@pytest.mark.parametrize("nq", (300, 20))
@pytest.mark.parametrize("what", SPECIAL)
def test_values_that_are_no_numbers(T, what, nq, lists):
    """The passes (300 queries) and the search of few queries against the single kernel, and against the oracle where every
    distance is a number."""
    n, d, M, gamma = 7000, 512, 128, 0.4
    ix, q, probes = built(T, n, d, M, 8, 12 if lists else 0, nq, 7 if lists else 0, 0.5, 0.0, 11)
    ix.list_bounds = None
    table = T.trim_build_lut(q, ix.codebooks) if what == "table" else None
    plant(what, ix, q, table)
    ix.scan_head = T.trim_pack_scan_head(ix.codes, ix.dlx)
    for k, batch in ((10, 512), (100, 3000), (10, 1)):
        want = single_kernel(T, ix, q, k, gamma, batch, probes, None, table)
        if what == "landmark distances" and not lists:
            O, oix = host_index(ix)
            ref = O.search_knn(oix, q.cpu().numpy(), k, gamma, batch, want_mask=True)
            for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
                np.testing.assert_array_equal(want[name].cpu().numpy().view(ref[name].dtype), ref[name], err_msg=name)
        got = T.trim_search_knn(ix, q, k, gamma, batch, probes=probes, lut=table, want_mask=True)
        for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
            np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=f"{name}, {k}, {batch}")
    if nq < 300:
        return
    for radius in (float(np.sqrt(np.nanmedian(want["d2"].cpu().numpy()))), float("inf")):
        want = single_range(T, ix, q, radius, gamma, probes, None, table)
        got = T.trim_search_range(ix, q, radius, gamma, probes=probes, lut=table, want_mask=True)
        for name in ("offsets", "ids", "d2", "n_scanned", "n_exact", "mask"):
            np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=f"{name}, {radius}")


@pytest.mark.parametrize("M,asked", ((44, False), (132, True)))
def test_work_space_beside_a_callers_table(T, M, asked, monkeypatch):
    """Tables of sub-vectors that are not compared with the centroids (12 values) leave the search with the single kernel."""
    import torch
    ix, q, _ = built(T, 3000, 528, M, 8, 0, 300, 0, 0.5, 0.0, 3)
    lut, empty, asked_for = T.trim_build_lut(q, ix.codebooks), torch.empty, []

    def count(*size, **kw):
        if kw.get("dtype") is torch.uint8:
            asked_for.append(size)
        return empty(*size, **kw)

    monkeypatch.setattr(torch, "empty", count)
    got = T.trim_search_knn(ix, q, 10, 0.4, 256, lut=lut)
    assert bool(asked_for) == asked
    ws = empty((T.trim_range_workspace_bytes(300, 3000),), dtype=torch.uint8, device="cuda")
    del asked_for[:]
    T.trim_search_range(ix, q, 1.0, 0.4, lut=lut, workspace=ws)
    assert bool(asked_for) == asked
    monkeypatch.undo()
    want = single_kernel(T, ix, q, 10, 0.4, 256, None, None, lut)
    for name in ("ids", "d2", "n_exact"):
        np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)


def test_work_space_of_the_caller(T, monkeypatch):
    """A buffer of the caller takes the place of an allocation; with too small a one nothing is allocated either."""
    import torch
    ix, q, probes = built(T, 6000, 512, 128, 8, 12, 300, 6, 0.5, 0.0, 3)
    need, more = T.trim_knn_workspace_bytes(ix, 300, 10, 256, probes), T.trim_range_scratch_bytes(ix, 300, probes)
    assert need > 0 and more > 0
    cand, mc = ix._cand(probes)
    rws = torch.empty((T.trim_range_workspace_bytes(300, mc),), dtype=torch.uint8, device="cuda")
    knn = lambda ws: T.trim_search_knn(ix, q, 10, 0.4, 256, probes=probes, want_mask=True, workspace=ws)
    rng = lambda ws: T.trim_search_range(ix, q, 20.0, 0.4, probes=probes, want_mask=True, workspace=rws, scratch=ws)
    want = knn(None), rng(None)
    buffers = [(torch.empty((a,), dtype=torch.uint8, device="cuda"), torch.empty((b,), dtype=torch.uint8, device="cuda"))
               for a, b in ((need, more), (need - 1, more - 1), (0, 0))]
    empty = torch.empty

    def nothing(*size, **kw):
        assert kw.get("dtype") is not torch.uint8
        return empty(*size, **kw)

    monkeypatch.setattr(torch, "empty", nothing)
    for a, b in buffers:
        for got, ref in zip((knn(a), rng(b)), want):
            for name in ref:
                if isinstance(ref[name], torch.Tensor):
                    assert torch.equal(got[name], ref[name]), (name, a.numel())


@pytest.mark.parametrize("case", [CASES[i] for i in (1, 3, 4, 5, 7, 8)], ids=lambda c: "-".join(map(str, c)))
def test_passes_equal_the_oracle(T, case):
    import torch
    n, d, M, bits, nlist, nq, nprobe, k, batch, gamma, spread, offset = case
    ix, q, probes = built(T, n, d, M, bits, nlist, nq, nprobe, spread, offset, n + d)
    if nlist:
        probes[5, 0] = 2                                 # (the oracle takes lists that exist)
    O, oix = host_index(ix)
    hq, hp = q.cpu().numpy(), None if probes is None else np.ascontiguousarray(probes.cpu().numpy())

    def same(got, want, names):
        assert T.trim_knn_workspace_bytes(ix, nq, k, batch, probes) > 0 and T.trim_range_scratch_bytes(ix, nq, probes) > 0
        for name in names:
            np.testing.assert_array_equal(got[name].cpu().numpy(), want[name], err_msg=name)
        mask = got["mask"].cpu().numpy().view(np.uint32)             # (as wide as the longest lists could make it)
        np.testing.assert_array_equal(mask[:, :want["mask"].shape[1]], want["mask"])
        assert not mask[:, want["mask"].shape[1]:].any()

    want = O.search_knn(oix, hq, k, gamma, batch, probes=hp, want_mask=True)
    same(T.trim_search_knn(ix, q, k, gamma, batch, probes=probes, want_mask=True), want, ("ids", "d2", "n_scanned", "n_exact"))
    radius = float(np.sqrt(np.quantile(want["d2"][np.isfinite(want["d2"])], 0.9)))
    want = O.search_range(oix, hq, radius, gamma, probes=hp, want_mask=True)
    assert want["offsets"][-1] > (nq if gamma <= 1.0 else 0)       # (gamma above 1 prunes what is near as well)
    same(T.trim_search_range(ix, q, radius, gamma, probes=probes, want_mask=True), want, ("offsets", "ids", "d2", "n_scanned", "n_exact"))


def test_more_queries_than_one_slab(T):
    """The work space is kept below 8 GiB by splitting the queries: with room for 384,000 candidates each, 2600 at a time."""
    import torch
    n, d, M, nq, k, batch, gamma = 6000, 512, 128, 2800, 10, 256, 0.4
    ix, q, probes = built(T, n, d, M, 8, 12, nq, 7, 0.5, 0.0, 3)
    probes = probes.repeat(1, 9).contiguous()            # (every list nine times)
    order = torch.randperm(nq, device="cuda").to(torch.int32)
    order[2] = nq + 5
    order[2700] = -1
    cand, mc = ix._cand(probes, max_candidates=64 * n)
    view, lut = ix._view(), T.trim_build_lut(q, ix.codebooks)
    need = T.lib().trim_knn_workspace_bytes(C.byref(view), nq, C.byref(cand), k, batch)
    per = T.lib().trim_knn_workspace_bytes(C.byref(view), 300, C.byref(cand), k, batch) / 300
    assert 7 << 30 < need < 9 << 30 and need < (nq - 150) * per        # (more than one slab, the second of some length)
    ws = torch.empty((need,), dtype=torch.uint8, device="cuda")
    p = lambda t: None if t is None else C.c_void_p(t.data_ptr())
    mw = (mc + 31) // 32
    for o, table in ((None, None), (order, None), (order, lut)):
        out = []
        for space, size in ((None, 0), (ws, need)):
            ids = torch.full((nq, k), -7, dtype=torch.int32, device="cuda")
            d2 = torch.full((nq, k), -7.0, device="cuda")
            ns, ne = torch.zeros((2, nq), dtype=torch.int32, device="cuda").unbind(0)
            mask = torch.zeros((nq, mw), dtype=torch.int32, device="cuda")
            stats = T._Stats(ns.data_ptr(), ne.data_ptr(), None)
            rc = T.lib().trim_search_knn_ws(C.byref(view), p(q), nq, p(table), C.byref(cand), k, gamma, batch, p(o), p(ids), p(d2),
                                            C.byref(stats), p(mask), mw, p(space), size,
                                            C.c_void_p(torch.cuda.current_stream().cuda_stream))
            assert rc == 0
            out.append((ids, d2, ns, ne, mask))
        for a, b in zip(*out):
            assert torch.equal(a, b)


# Hardly any candidates: fewer vectors than neighbours wanted, than a word of marks, than a tile; lists that nobody names.
@pytest.mark.parametrize("n", (1, 3, 33, 300))
@pytest.mark.parametrize("nlist", (0, 4))
def test_hardly_any_candidates(T, n, nlist):
    import torch
    d, M, nq, k, batch, gamma = 512, 64, 300, 10, 16, 0.3
    g = torch.Generator(device="cuda").manual_seed(n + nlist)
    base, q = torch.randn((n, d), device="cuda", generator=g), torch.randn((nq, d), device="cuda", generator=g)
    cb = torch.randn((M, 256, d // M), device="cuda", generator=g)
    codes, dlx = T.trim_encode(base, cb)
    offsets = probes = None
    longest = 0
    if nlist:
        offsets = torch.tensor([0, 0, n // 2, n, n], device="cuda")
        probes = torch.randint(-1, nlist + 1, (nq, 3), device="cuda", generator=g).to(torch.int32)
        longest = n - n // 2
    ix = T.Index(base, codes, dlx, cb, list_offsets=offsets, max_list_len=longest)
    every = [probes] if probes is None else [probes, torch.full_like(probes, 3), torch.full_like(probes, -1)]
    for pr in every:
        assert T.trim_knn_workspace_bytes(ix, nq, k, batch, pr) > 0
        want = single_kernel(T, ix, q, k, gamma, batch, pr, None)
        got = T.trim_search_knn(ix, q, k, gamma, batch, probes=pr, want_mask=True)
        for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
            np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)
        for radius in (0.0, 30.0, 35.0):
            want = single_range(T, ix, q, radius, gamma, pr, None, None)
            got = T.trim_search_range(ix, q, radius, gamma, probes=pr, want_mask=True)
            for name in ("offsets", "ids", "d2", "n_scanned", "n_exact", "mask"):
                np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)


# As many lists as are counted in the LDS, and more: one to several vectors each, empty ones, lists named twice and lists that are none.
@pytest.mark.parametrize("nlist", (16384, 16385, 30000))
def test_thousands_of_lists(T, nlist):
    import torch
    n, d, M, nq, nprobe, k, batch, gamma = 40000, 512, 64, 300, 1700, 10, 64, 0.4
    g = torch.Generator(device="cuda").manual_seed(nlist)
    base, q = torch.randn((n, d), device="cuda", generator=g), torch.randn((nq, d), device="cuda", generator=g)
    cb = torch.randn((M, 256, d // M), device="cuda", generator=g)
    codes, dlx = T.trim_encode(base, cb)
    offsets = torch.cat([torch.zeros(1, device="cuda", dtype=torch.int64), torch.randint(0, n, (nlist - 1,), device="cuda", generator=g).sort().values,
                         torch.full((1,), n, device="cuda", dtype=torch.int64)])
    probes = torch.randint(-3, nlist + 3, (nq, nprobe), device="cuda", generator=g).to(torch.int32)
    probes[:, :40] = nlist - 1 - torch.arange(40, device="cuda", dtype=torch.int32)        # (everybody's)
    ix = T.Index(base, codes, dlx, cb, list_offsets=offsets, max_list_len=int((offsets[1:] - offsets[:-1]).max()))
    order = torch.randperm(nq, device="cuda", generator=g).to(torch.int32)
    assert T.trim_knn_workspace_bytes(ix, nq, k, batch, probes) > 0 and T.trim_range_scratch_bytes(ix, nq, probes) > 0
    want = single_kernel(T, ix, q, k, gamma, batch, probes, order)
    got = T.trim_search_knn(ix, q, k, gamma, batch, probes=probes, query_order=order, want_mask=True)
    for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
        np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)
    want = single_range(T, ix, q, 29.0, gamma, probes, order, None)
    got = T.trim_search_range(ix, q, 29.0, gamma, probes=probes, query_order=order, want_mask=True)
    assert 0 < want["ids"].shape[0] < want["n_scanned"].sum()
    for name in ("offsets", "ids", "d2", "n_scanned", "n_exact", "mask"):
        np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)


# A query with more candidates than max_candidates is cut there: inside a list, at its end, before the first batch ends, one candidate after it.
@pytest.mark.parametrize("nq", (300, 20))
@pytest.mark.parametrize("cut", (5, 31, 267, 500, 513, 2000, 2048))
def test_candidates_are_cut(T, cut, nq, monkeypatch):
    import torch
    ix, q, probes = built(T, 9000, 512, 128, 8, 6, nq, 4, 0.5, 0.0, 3)
    plain = T.Index._cand
    monkeypatch.setattr(T.Index, "_cand", lambda self, p, max_candidates=0: plain(self, p, cut))
    k, batch, gamma = 10, 256, 0.4
    assert T.trim_knn_workspace_bytes(ix, nq, k, batch, probes) > 0
    want = single_kernel(T, ix, q, k, gamma, batch, probes, None)
    got = T.trim_search_knn(ix, q, k, gamma, batch, probes=probes, want_mask=True)
    assert int(got["n_scanned"].max()) == cut
    for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
        np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)
    if nq < 300:
        return
    want = single_range(T, ix, q, 20.0, gamma, probes, None, None)
    got = T.trim_search_range(ix, q, 20.0, gamma, probes=probes, want_mask=True)
    for name in ("offsets", "ids", "d2", "n_scanned", "n_exact", "mask"):
        np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)


@pytest.mark.parametrize("nq", (300, 20))
def test_captured_and_replayed(T, nq):
    """Probe selection, ordering, kNN and the range search as one graph (nothing in them allocates outside torch or waits):
    every replay, on other queries, against the eager calls."""
    import torch
    n, d, M, nlist, nprobe, k = 9000, 512, 128, 70, 6, 10
    ix, queries, _ = built(T, n, d, M, 8, nlist, 3 * nq, nprobe, 0.5, 0.0, 9)
    cent = ix.base[torch.arange(0, n, n // nlist, device="cuda")[:nlist]].contiguous()
    cand_max = min(n, nprobe * ix.max_list_len)
    rws = torch.empty((T.trim_range_workspace_bytes(nq, cand_max),), dtype=torch.uint8, device="cuda")
    offsets, required = torch.empty((nq + 1,), dtype=torch.int64, device="cuda"), torch.empty((1,), dtype=torch.int64, device="cuda")
    cap = 400_000
    rids, rd2 = torch.empty((cap,), dtype=torch.int32, device="cuda"), torch.empty((cap,), device="cuda")

    def both(q):
        pr = T.trim_ivf_probe(q, cent, nprobe)
        order = T.trim_query_order(pr, nlist)
        r = T.trim_search_knn(ix, q, k, 0.4, 256, probes=pr, query_order=order, want_mask=True)
        cand, _ = ix._cand(pr)
        view, more = ix._view(), T.trim_range_scratch_bytes(ix, nq, pr)
        sc = torch.empty((max(more, 1),), dtype=torch.uint8, device="cuda")
        rc = T.lib().trim_search_range_ws(C.byref(view), q.data_ptr(), nq, None, C.byref(cand), 22.0, 0.4, order.data_ptr(),
                                          offsets.data_ptr(), rids.data_ptr(), rd2.data_ptr(), cap, required.data_ptr(), None, None, 0,
                                          rws.data_ptr(), rws.numel(), sc.data_ptr(), more, torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        return pr, r["ids"], r["d2"], r["n_scanned"], r["n_exact"], r["mask"]

    x = queries[:nq].clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        both(x)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = both(x)
    for rep in range(4):
        x.copy_(queries[(rep % 3) * nq:(rep % 3 + 1) * nq])
        graph.replay()
        torch.cuda.synchronize()
        total = int(required)
        assert 0 < total <= cap
        got = [t.clone() for t in out] + [offsets.clone(), rids[:total].clone(), rd2[:total].clone()]
        want = list(both(x))
        torch.cuda.synchronize()
        want += [offsets, rids[:total], rd2[:total]]
        for a, b in zip(got, want):
            assert torch.equal(a, b), rep


# one and two result entries per lane at their edges, codes with and without a scan head, query counts at which another block size is
# taken (make_plan): who asks beside them changes nobody's answer, and the first are the oracle's
@pytest.mark.parametrize("d,M,bits", ((100, 20, 8), (128, 16, 8), (128, 32, 8), (384, 48, 8), (128, 64, 4)))
@pytest.mark.parametrize("k,batch", ((1, 512), (10, 100), (64, 256), (65, 100), (128, 512)))
def test_answers_do_not_depend_on_the_number_of_queries(T, d, M, bits, k, batch):
    ix, q, probes = built(T, 20000, d, M, bits, 40, 1100, 9, 1.0, 2.0, d + M + k)
    want = single_kernel(T, ix, q, k, 0.3, batch, probes, None)
    for nq in (20, 256, 257, 512, 513, 768, 769, 1024, 1025):
        got = single_kernel(T, ix, q[:nq], k, 0.3, batch, probes[:nq].contiguous(), None)
        for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
            np.testing.assert_array_equal(got[name].cpu().numpy(), want[name][:nq].cpu().numpy(), err_msg=f"{name} {nq}")
    c = lambda t: t.cpu().numpy()
    from oracle import trim_oracle, trim_oracle_fs
    o = trim_oracle if bits == 8 else trim_oracle_fs
    oix = o.Index(c(ix.base), c(ix.codes), c(ix.dlx), c(ix.codebooks), ids=c(ix.ids), list_offsets=c(ix.list_offsets))
    ref = o.search_knn(oix, c(q[8:28]), k, 0.3, batch, c(probes[8:28]))      # (those before it probe lists that are not there)
    np.testing.assert_array_equal(c(want["ids"][8:28]), ref["ids"])
    np.testing.assert_array_equal(c(want["n_exact"][8:28]), ref["n_exact"])


# 769 to 1024 queries over short codes: four workgroups a CU up to 16,384 candidates or batches of 128, three beyond
@pytest.mark.parametrize("n", (16384, 16385))
@pytest.mark.parametrize("k,batch", ((10, 128), (10, 129), (100, 128), (100, 512)))
def test_queries_that_fit_in_one_go(T, n, k, batch):
    ix, q, _ = built(T, n, 100, 20, 8, 0, 1024, 0, 1.0, 2.0, k)
    want = single_kernel(T, ix, q[:20].contiguous(), k, 0.3, batch, None, None)
    for nq in (769, 1024):
        got = single_kernel(T, ix, q[:nq].contiguous(), k, 0.3, batch, None, None)
        for name in ("ids", "d2", "n_scanned", "n_exact", "mask"):
            np.testing.assert_array_equal(got[name].cpu().numpy()[:20], want[name].cpu().numpy(), err_msg=f"{name} {nq}")


# codes of 16 bytes and more that are no multiple of 8: 16-byte pieces at multiples of 4, what is left of a code (4, 8, 12 bytes), table
# phases, the list summaries without a scan head; one to sixteen result entries per lane
@pytest.mark.parametrize("d,M", ((80, 20), (112, 28), (132, 44), (240, 60), (720, 180)))
@pytest.mark.parametrize("k,batch,nlist", ((10, 1024, 60), (10, 3, 0), (100, 512, 60), (200, 256, 0), (300, 100, 25)))
def test_codes_that_are_no_multiple_of_eight(T, d, M, k, batch, nlist):
    from oracle import trim_oracle
    ix, q, probes = built(T, 30000, d, M, 8, nlist, 12, min(nlist, 20), 1.0, 2.0, d + k)
    got = single_kernel(T, ix, q, k, 0.3, batch, probes, None)
    c = lambda t: None if t is None else t.cpu().numpy()
    oix = trim_oracle.Index(c(ix.base), c(ix.codes), c(ix.dlx), c(ix.codebooks), ids=c(ix.ids), list_offsets=c(ix.list_offsets))
    rows = slice(8, 12)                      # (those before it probe lists that are not there)
    ref = trim_oracle.search_knn(oix, c(q[rows]), k, 0.3, batch, c(probes[rows]) if nlist else None)
    for name in ("ids", "d2", "n_scanned", "n_exact"):
        np.testing.assert_array_equal(c(got[name])[rows], ref[name], err_msg=name)


# The thresholds that count on remaining table minima, and the list summaries, hold for up to 256 additions per table sum: searches over
# longer 4-bit codes go without (nothing is passed over), also where three workgroups would fit a CU; 128 code bytes are the most with them.
@pytest.mark.parametrize("d,M,with_them", ((256, 256, True), (272, 272, False), (320, 320, False), (672, 336, False)))
@pytest.mark.parametrize("k,batch", ((10, 256), (100, 256)))
def test_thresholds_of_long_4_bit_codes(T, d, M, with_them, k, batch):
    from oracle import trim_oracle_fs
    ix, q, probes = built(T, 30000, d, M, 4, 40, 600, 32, 3.0, 0.0, d + k)
    got = T.trim_search_knn(ix, q, k, 0.3, batch, probes=probes, want_work=True)
    skipped = got["work"][:, T.WORK_NAMES.index("skipped")].cpu().numpy()
    assert (skipped.max() > 0) == with_them
    c = lambda t: t.cpu().numpy()
    oix = trim_oracle_fs.Index(c(ix.base), c(ix.codes), c(ix.dlx), c(ix.codebooks), ids=c(ix.ids), list_offsets=c(ix.list_offsets))
    rows = slice(8, 24)                      # (those before it probe lists that are not there)
    ref = trim_oracle_fs.search_knn(oix, c(q[rows]), k, 0.3, batch, c(probes[rows]))
    for name in ("ids", "d2", "n_scanned", "n_exact"):
        np.testing.assert_array_equal(c(got[name])[rows], ref[name], err_msg=name)
