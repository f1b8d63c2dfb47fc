"""Index construction and calibration kernels at the edges of their tiles, against the oracle."""
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


# rows around the 8192-row chunks of the update; clusters that leave a last group partly empty; a row
# longer than one 1024-column slice; one cluster that takes nearly everything; a list of rows that fills several times
@pytest.mark.parametrize("ns,d,nlist", [(8191, 8, 7), (8193, 12, 33), (16385, 4, 130), (9000, 1028, 5), (1, 4, 1), (70001, 4, 2)])
def test_update_of_coarse_centroids(T, oracle, ns, d, nlist):
    import torch
    from oracle import index_build
    rng = np.random.default_rng(ns)
    x = rng.standard_normal((ns, d)).astype(np.float32)
    x[ns // 4:] *= np.float32(0.01)
    init = rng.choice(ns, nlist, replace=False).astype(np.int32)
    want = index_build.train_ivf_fixed(x, nlist, 2, init)
    got = T.trim_train_ivf(torch.from_numpy(x).cuda(), nlist, 2, torch.from_numpy(init).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("ns,d,M,bits", [(8192, 16, 4, 8), (8200, 20, 4, 8), (300, 64, 4, 8), (8300, 8, 4, 4),
                                         (40003, 28, 4, 8), (40001, 24, 8, 4), (257, 132, 4, 8)])
def test_update_of_codebooks(T, oracle, ns, d, M, bits):
    import torch
    from oracle import index_build
    rng = np.random.default_rng(d)
    x = rng.standard_normal((ns, d)).astype(np.float32)
    x[: ns // 2] = x[0]                     # one cluster per subspace takes half of the rows
    K = 256 if bits == 8 else 16
    init = rng.choice(ns, K, replace=False).astype(np.int32)
    fn = T.trim_train_pq if bits == 8 else T.trim_fs_train_pq
    ref = index_build.train_pq_fixed if bits == 8 else index_build.train_pq_fs_fixed
    want = ref(x, M, 3, init)
    got = fn(torch.from_numpy(x).cuda(), M, 3, torch.from_numpy(init).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32))


# vectors whose nearest list the matrix cores leave open (many lists in one place): as many of a workgroup's together as the exact
# rule has widths for, one fewer and one more
@pytest.mark.parametrize("d", (64, 128, 132))
@pytest.mark.parametrize("marked", (1, 2, 3, 4, 5, 8, 9, 11))
def test_nearest_list_of_vectors_left_open(T, oracle, d, marked):
    import torch
    rng = np.random.default_rng(d + marked)
    cent = rng.integers(-40, 41, (150, d)).astype(np.float32)
    cent[30:90:2] = cent[31]
    x = (cent[rng.integers(90, 150, 4100)] + rng.integers(-2, 3, (4100, d))).astype(np.float32)
    at = np.concatenate([7 + np.arange(marked), [300]])
    x[at] = cent[31] + rng.integers(-2, 3, (marked + 1, d)).astype(np.float32)
    got = T.trim_ivf_probe(torch.from_numpy(x).cuda(), torch.from_numpy(cent).cuda(), 1).cpu().numpy()
    np.testing.assert_array_equal(got[:400], oracle.ivf_probe(x[:400], cent, 1))
    assert (got[at] == 30).all()


# long rows, which are added straight from memory: the instance for up to 8192 rows and the other one; a cluster whose rows do not fit the
# list, so that it is filled again after it has been put in order
@pytest.mark.parametrize("ns,d,nlist", [(8192, 1028, 5), (8193, 260, 9), (300, 1028, 40), (40001, 260, 3)])
def test_update_of_coarse_centroids_of_long_rows(T, oracle, ns, d, nlist):
    test_update_of_coarse_centroids(T, oracle, ns, d, nlist)


# the update with work space: chunks of 4096 and 1024 rows that are full, one short and one over, more than 64 of them, rows of every
# kind of sub-vector (four values at a time or one by one, in the LDS or straight from memory), fewer counters than 1024 threads
# have room for, half of the rows in one cluster and none in two; and the same without it, codes, distances and assignments too.  Around the
# work space nothing is written
@pytest.mark.parametrize("ns,d,M,bits", [(32768, 64, 16, 8), (33001, 80, 16, 8), (36863, 128, 16, 8), (45057, 144, 12, 8), (131073, 8, 4, 8),
                                         (26215, 340, 20, 8), (40001, 32, 16, 4), (270001, 16, 4, 8),
                                         (1025, 12, 33, 0), (9300, 8, 20, 0), (5000, 16, 30, 0), (2047, 20, 100, 0), (3072, 24, 7, 0), (262145, 4, 50, 0), (40000, 4, 4990, 0), (70000, 300, 3, 0)])
def test_update_with_work_space(T, oracle, ns, d, M, bits):
    import ctypes as C
    import torch
    from oracle import index_build
    L = T.lib()
    size = L.trim_train_ivf_workspace_bytes if bits == 0 else L.trim_train_pq_workspace_bytes if bits == 8 else L.trim_fs_train_pq_workspace_bytes
    need = size(ns, d, M)
    assert need > 0
    rng = np.random.default_rng(ns + d)
    x = rng.standard_normal((ns, d)).astype(np.float32)
    x[: ns // 2] = x[0]
    K = M if bits == 0 else 256 if bits == 8 else 16
    init = rng.choice(np.arange(ns // 2, ns), K, replace=False).astype(np.int32)
    init[K // 2] = init[K - 1] = init[0]             # (the first of equal centroids takes the rows)
    ref = index_build.train_ivf_fixed if bits == 0 else index_build.train_pq_fixed if bits == 8 else index_build.train_pq_fs_fixed
    want = ref(x, M, 2, init)
    g, gi = torch.from_numpy(x).cuda(), torch.from_numpy(init).cuda()
    fn = T.trim_train_ivf if bits == 0 else T.trim_train_pq if bits == 8 else T.trim_fs_train_pq
    np.testing.assert_array_equal(fn(g, M, 2, gi).cpu().numpy().view(np.uint32), want.view(np.uint32))
    ws = torch.empty((4 + need + 65536,), dtype=torch.uint8, device="cuda")
    p = lambda t: C.c_void_p(t.data_ptr())
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    used = []
    for shift, bytes_ in ((4, need), (0, need - 1)):                  # (the last: the kernel without)
        ws.fill_(0xa5)
        out = torch.empty(want.shape, dtype=torch.float32, device="cuda")
        codes, dlx = torch.zeros((ns * max(M, 4),), dtype=torch.uint8, device="cuda"), torch.zeros((ns,), device="cuda")
        tail = [C.c_void_p(ws.data_ptr() + shift), bytes_, stream]
        if bits == 0:
            rc = L.trim_train_ivf_ws(p(g), ns, d, M, 2, p(gi), p(out), p(codes), *tail)
        elif bits == 8:
            rc = L.trim_train_pq_ws(p(g), ns, d, M, 2, p(gi), p(out), p(codes), p(dlx), *tail)
        else:
            rc = L.trim_fs_train_pq_ws(p(g), ns, d, M, 2, p(gi), p(out), p(codes), *tail)
        assert rc == 0
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))
        used.append((codes, dlx.view(torch.int32)))
        assert (ws[:4] == 0xa5).all() and (ws[4 + need:] == 0xa5).all()
    assert (ws == 0xa5).all()
    for with_it, without in zip(*used):
        assert torch.equal(with_it, without)


@pytest.mark.parametrize("ns,M,bits", [(8192, 32, 8), (300, 32, 8), (20001, 32, 8), (8192, 64, 4), (20001, 64, 4)])
def test_update_of_codebooks_of_long_subvectors(T, oracle, ns, M, bits):
    import torch
    from oracle import index_build
    rng = np.random.default_rng(ns)
    x = rng.standard_normal((ns, 8 * M if bits == 8 else 16 * M)).astype(np.float32)
    x[: ns * 9 // 10] = x[0]                     # (18,000 rows in one cluster; the list holds 16,384)
    x[: ns * 9 // 10, ::8] += np.arange(ns * 9 // 10, dtype=np.float32)[:, None] * np.float32(1e-6)
    K = 256 if bits == 8 else 16
    init = np.concatenate([[0], ns - 1 - np.arange(K - 1)]).astype(np.int32) if ns > K else np.arange(K, dtype=np.int32)
    fn = T.trim_train_pq if bits == 8 else T.trim_fs_train_pq
    ref = index_build.train_pq_fixed if bits == 8 else index_build.train_pq_fs_fixed
    want = ref(x, M, 2, init)
    got = fn(torch.from_numpy(x).cuda(), M, 2, torch.from_numpy(init).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32))


# every sub-vector length with the matrix-core filter and one without; few vectors, with their subspaces dealt out; ties, all-zero centroids, magnitudes outside the filter's range
@pytest.mark.parametrize("dsub,M,n", [(4, 4, 1), (4, 8, 129), (5, 4, 255), (6, 4, 700), (8, 8, 1000), (7, 4, 300),
                                      (4, 4, 131073), (8, 4, 131100)])
def test_encode_filter(T, oracle, dsub, M, n, skew=0):
    import torch
    rng = np.random.default_rng(dsub * 1000 + n)
    d = dsub * M
    x = rng.standard_normal((n, d)).astype(np.float32)
    cb = rng.standard_normal((M, 256, dsub)).astype(np.float32)
    cb[0, 200:] = cb[0, :56]                       # ties: the smaller index wins
    cb[1] = np.round(cb[1] * 2) / 2                # a grid: many ties
    x[: n // 2, dsub: 2 * dsub] = np.round(x[: n // 2, dsub: 2 * dsub] * 2) / 2 + 0.25
    cb[2] = 0 if n % 2 else cb[2] * np.float32(1e-3) + np.float32(100)   # zeros / a far, tight cloud
    cb[3] *= np.float32(1e-20) if n % 3 else np.float32(1e17)
    x[n // 3, :dsub] = 3e6                         # a vector far beyond the centroids
    rc, rd = oracle.encode(x, cb)
    rows = torch.zeros((n * d + skew,), device="cuda")[skew:].view(n, d).copy_(torch.from_numpy(x))
    codes, dlx = T.trim_encode(rows, torch.from_numpy(cb).cuda())
    np.testing.assert_array_equal(codes.cpu().numpy(), rc)
    np.testing.assert_array_equal(dlx.cpu().numpy().view(np.uint32), rd.view(np.uint32))


# workgroups of 256 and of 512 vectors, whole and with the subspaces dealt out: full, one vector short and one over; more than one round
# of the row reader; rows that begin off a 16-byte boundary
@pytest.mark.parametrize("skew", (0, 1))
@pytest.mark.parametrize("dsub,M,n", [(4, 4, 255), (5, 12, 257), (4, 16, 16385), (8, 16, 19968), (6, 16, 20001), (5, 16, 20479),
                                      (4, 8, 57345), (8, 4, 58111), (4, 8, 65537), (5, 8, 66049), (6, 4, 66048), (8, 8, 66047)])
def test_encode_filter_by_workgroup(T, oracle, dsub, M, n, skew):
    test_encode_filter(T, oracle, dsub, M, n, skew)


# the nearest list of many vectors: ragged vector, list and column counts, ties between lists, vectors
# halfway between two lists, lists far from the origin, one far vector, magnitudes that overflow
@pytest.mark.parametrize("n,d,nlist,scale", [(4096, 4, 64, 1), (4099, 128, 1024, 1), (5000, 36, 257, 1), (4353, 100, 300, 1),
                                             (4200, 132, 70, 1e19), (4100, 64, 511, 1e-20), (4097, 768, 90, 1),
                                                 (4096, 64, 129, 1), (4351, 124, 2049, 1), (4100, 68, 65, 1e19), (4100, 128, 64, 1e-3)])
def test_assignment(T, oracle, n, d, nlist, scale):
    import torch
    rng = np.random.default_rng(n)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    cent[nlist // 2:nlist // 2 + 20] = cent[:20]                              # the smaller id wins
    cent[40:60] = cent[20:40] + np.float32(1e-3)                              # nearly the same
    x = cent[rng.integers(0, nlist, n)] + (0.3 * rng.standard_normal((n, d))).astype(np.float32)
    x[:500] = (cent[rng.integers(0, nlist, 500)] + cent[rng.integers(0, nlist, 500)]) / 2
    if nlist == 300:
        cent, x = cent * np.float32(1e-2) + np.float32(10), x * np.float32(1e-2) + np.float32(10)
    x[77] = 1e4
    cent, x = (cent * np.float32(scale)), (x * np.float32(scale)).astype(np.float32)
    want = oracle.ivf_probe(x, cent, 1)
    got = T.trim_ivf_probe(torch.from_numpy(x).cuda(), torch.from_numpy(cent).cuda(), 1).cpu().numpy()
    np.testing.assert_array_equal(got, want)


# the nearest list with work space and without: vectors one short of a workgroup, full and one over, lists around a stage of them (128 of up to
# 64 values, 64 of longer ones), equal lists at one place of as many tiles as are told apart and one more, and at as many places as are
# measured and more
@pytest.mark.parametrize("n,d,nlist", [(4097, 4, 64), (4351, 64, 129), (4352, 60, 128), (4353, 68, 127), (4100, 128, 64), (4120, 128, 65),
                                       (4200, 124, 250), (6000, 128, 1025), (5000, 32, 2050)])
def test_nearest_list_by_work_space(T, oracle, n, d, nlist):
    import ctypes as C
    import torch
    rng = np.random.default_rng(n + d)
    cent = rng.integers(-40, 41, (nlist, d)).astype(np.float32)
    for k, tiles in ((3, 2), (9, 3), (17, 4), (30, 5)):
        cent[k: 32 * tiles + k: 32] = cent[k]
    for k, places in ((5, 2), (40, 12), (64, 20)):
        cent[k: k + places] = cent[min(k, nlist - 1)]
    x = (cent[rng.integers(0, nlist, n)] + rng.integers(-2, 3, (n, d))).astype(np.float32)
    x[50], x[51] = np.nan, 1e30
    xg, cg = torch.from_numpy(x).cuda(), torch.from_numpy(cent).cuda()
    want = oracle.ivf_probe(x, cent, 1)
    np.testing.assert_array_equal(T.trim_ivf_probe(xg, cg, 1).cpu().numpy(), want)
    out = torch.full((n, 1), -7, dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    need = T.lib().trim_ivf_nearest_workspace_bytes(n, d, nlist)
    assert need > 0
    space = torch.full((4 + need + 65536,), 0xa5, dtype=torch.uint8, device="cuda")
    for ws, size in ((None, 0), (space.data_ptr(), need - 1), (space.data_ptr() + 4, need)):
        out.fill_(-7)
        assert T.lib().trim_ivf_probe_ws(C.c_void_p(xg.data_ptr()), n, d, C.c_void_p(cg.data_ptr()), nlist, 1, C.c_void_p(out.data_ptr()),
                                         C.c_void_p(ws), size, C.c_void_p(stream)) == 0
        np.testing.assert_array_equal(out.cpu().numpy(), want)
    assert (space[:4] == 0xa5).all() and (space[4 + need:] == 0xa5).all()


# 4-bit codes: sub-vectors of two values (whole and ragged 32-column slices, odd row counts) and of four
@pytest.mark.parametrize("d,m,n", [(128, 64, 257), (36, 18, 100), (24, 12, 1), (100, 50, 513), (64, 16, 300)])
def test_encode_four_bit(T, d, m, n):
    import torch
    from oracle import trim_oracle_fs
    rng = np.random.default_rng(d + n)
    x = rng.standard_normal((n, d)).astype(np.float32)
    cb = rng.standard_normal((m, 16, d // m)).astype(np.float32)
    cb[0, 8:] = cb[0, :8]
    rc, rd = trim_oracle_fs.encode(x, cb)
    codes, dlx = T.trim_fs_encode(torch.from_numpy(x).cuda(), torch.from_numpy(cb).cuda())
    np.testing.assert_array_equal(codes.cpu().numpy(), rc)
    np.testing.assert_array_equal(dlx.cpu().numpy().view(np.uint32), rd.view(np.uint32))


# one and many queries, an odd vector left over, vectors longer than a half wave's step, values too
# many for two vectors' worth of LDS, and a rank at either end
@pytest.mark.parametrize("S,Q,d,M,p", [(1, 1, 8, 4, 0.5), (3, 7, 128, 32, 1.0), (5, 1000, 260, 20, 0.0),
                                       (2, 16384, 1536, 192, 0.9), (3, 9, 4, 4, 0.6)])
def test_gamma_rank(T, S, Q, d, M, p):
    import torch
    g = torch.Generator(device="cuda").manual_seed(S * 1000 + Q)
    base = torch.randn((50, d), device="cuda", generator=g)
    cb = torch.randn((M, 256, d // M), device="cuda", generator=g)
    q = torch.randn((Q, d), device="cuda", generator=g)
    if S == 3 and Q == 9:
        q[:] = q[0]                          # every value the same
    codes, dlx = T.trim_encode(base, cb)
    rows = torch.arange(S, device="cuda", dtype=torch.int32)
    gamma, each = T.trim_estimate_gamma(T.Index(base, codes, dlx, cb), rows, q, p)
    land = torch.stack([cb[j][codes[:S, j].long()] for j in range(M)], 1).reshape(S, d).double()
    u, w = base[:S].double() - land, q.double()[None] - land[:, None]
    cos = (w * u[:, None]).sum(-1) / (w.norm(dim=-1) * u.norm(dim=-1)[:, None])
    m = min(Q, max(1, int(np.ceil(p * Q))))
    want = (1.0 - cos).sort(dim=1).values[:, Q - m]
    np.testing.assert_allclose(each.cpu().numpy(), want.cpu().numpy(), atol=2e-5)
    assert gamma.item() == max(0.0, each.min().item())


# with work space (bins from the matrix cores, exact values around the rank) the same bits as without: one tile and odd
# remainders of rows, queries and coordinates; more values to evaluate than fit the LDS; vectors in two chunks; rows, queries
# and landmarks that are no numbers, out of the scaled range, or in one place
@pytest.mark.parametrize("S,Q,d,M,p,kind", [
    (32, 256, 16, 4, 0.9, ""), (33, 1001, 100, 20, 0.7, ""), (1, 16384, 128, 16, 0.99, ""), (700, 300, 392, 56, 0.5, ""),
    (40, 5000, 128, 32, 0.0, ""), (5, 5000, 36, 12, 1.0, "same"), (4099, 16300, 4, 4, 0.8, ""), (65, 2000, 64, 16, 0.9, "odd"),
    (65, 3000, 64, 16, 0.3, "tiny"), (65, 3000, 64, 16, 0.3, "huge"), (65, 3000, 64, 16, 0.6, "landmarks"),
    (300, 3000, 64, 16, 0.6, "all landmarks"), (65, 3000, 64, 16, 0.6, "spread")])
def test_gamma_with_work_space(T, S, Q, d, M, p, kind):
    import ctypes
    import torch
    g = torch.Generator(device="cuda").manual_seed(S + Q + d)
    base = torch.rand((max(S, 300), d), device="cuda", generator=g) * 200
    q = torch.rand((Q, d), device="cuda", generator=g) * 200
    cb = torch.rand((M, 256, d // M), device="cuda", generator=g) * 200
    rows = torch.randperm(base.shape[0], device="cuda", generator=g)[:S].int()
    if kind == "same":
        q[:] = q[0]
    if kind == "odd":
        base[rows[:6].long(), 3] = torch.tensor([float("nan"), float("inf"), -float("inf"), 1e20, 3e38, 1e-40], device="cuda")
        q[:9, 5] = torch.tensor([float("nan"), float("inf"), -float("inf"), 1e20, 3e38, 1e-40, -1e14, 1e11, 0.0], device="cuda")
    if kind in ("tiny", "huge"):
        scale = 1e-18 if kind == "tiny" else 1e16
        base, q, cb = base * scale, q * scale, cb * scale
    if kind == "spread":                     # queries' lengths over four decades, sampled rows out of range
        q *= torch.logspace(0, 4, Q, device="cuda")[:, None]
        rows[:2] = torch.tensor([-5, 10**6], device="cuda")
    codes, dlx = T.trim_encode(base, cb)
    if kind == "all landmarks":
        base = torch.stack([cb[j][codes[:, j].long()] for j in range(M)], 1).reshape(-1, d).contiguous()
    if kind == "landmarks":                  # vectors, and queries, at a landmark
        land = torch.stack([cb[j][codes[:, j].long()] for j in range(M)], 1).reshape(-1, d)
        base[rows[:20].long()] = land[rows[:20].long()]
        q[::3] = land[rows[torch.arange(0, Q, 3, device="cuda") % S].long()]
    index = T.Index(base, codes, dlx, cb)
    assert T.lib().trim_estimate_gamma_workspace_bytes(d, S, Q) > 0
    gamma, each = T.trim_estimate_gamma(index, rows, q, p)
    gamma0, each0 = torch.zeros(1, device="cuda"), torch.zeros(S, device="cuda")
    view = index._view()
    assert T.lib().trim_estimate_gamma(ctypes.byref(view), rows.data_ptr(), S, q.data_ptr(), Q, p, each0.data_ptr(),
                                       gamma0.data_ptr(), T._stream()) == 0
    np.testing.assert_array_equal(each.cpu().numpy().view(np.uint32), each0.cpu().numpy().view(np.uint32))
    np.testing.assert_array_equal(gamma.cpu().numpy().view(np.uint32), gamma0.cpu().numpy().view(np.uint32))


# one query to more than a tile of them; lists that leave tiles and columns unfilled; ties; the nearest lists all
# in one column of the selection (8192 lists)
@pytest.mark.parametrize("nq,nlist,d,nprobe", ((1, 64, 4, 2), (1, 1000, 128, 32), (2, 65, 100, 64), (5, 300, 1536, 33),
                                              (9, 4097, 128, 64), (67, 1024, 384, 64), (3, 8192, 96, 32), (4, 8192, 32, 50)))
def test_probe_of_few_queries(T, oracle, nq, nlist, d, nprobe):
    import torch
    assert T.lib().trim_ivf_probe_workspace_bytes(nq, d, nlist, nprobe) > 0
    rng = np.random.default_rng(nlist + d)
    cent = rng.integers(-3, 4, (nlist, d)).astype(np.float32)
    q = rng.integers(-3, 4, (nq, d)).astype(np.float32)
    if nlist == 8192:
        cent[::64] = q[0] + rng.integers(0, 2, (128, d)).astype(np.float32)
    cent[nlist // 2] = cent[3]
    want = oracle.ivf_probe(q, cent, nprobe)
    got = T.trim_ivf_probe(torch.from_numpy(q).cuda(), torch.from_numpy(cent).cuda(), nprobe).cpu().numpy()
    np.testing.assert_array_equal(got, want)


def test_nearest_list_with_centroids_that_are_no_numbers():
    """A centroid that is no number (its list held such a row in training) is nobody's nearest; infinite ones neither.  One
    far out of the scaled range, vectors there, and many lists in one place leave the scores behind as well."""
    import torch
    from paper_2508_17828_amd import trim as T
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((5000, 64), device="cuda", generator=g)
    x[:40] *= 3e3
    cent = torch.randn((70, 64), device="cuda", generator=g)
    cent[50:60] = cent[49]
    for bad in (float("nan"), -float("nan"), float("inf"), 1e6):
        c = cent.clone()
        c[5, 3] = bad
        few = torch.cat([T.trim_ivf_probe(x[i:i + 1000].contiguous(), c, 1) for i in range(0, 5000, 1000)])
        many = T.trim_ivf_probe(x, c, 1)
        assert not (few == 5).any()
        assert torch.equal(many, few)


@pytest.mark.parametrize("d", (36, 128, 132, 516))
@pytest.mark.parametrize("nq", (25_500, 25_700))
def test_nearest_list_of_vectors_that_the_scores_leave_open(nq, d):
    """A workgroup per CU for these, and more than that; all vectors (a centroid is no number), and some of each workgroup's."""
    import torch
    from paper_2508_17828_amd import trim as T
    g = torch.Generator(device="cuda").manual_seed(d)
    x, cent = torch.randn((nq, d), device="cuda", generator=g), torch.randn((77, d), device="cuda", generator=g)
    cent[60:70] = cent[59]
    x[::37] = cent[63]
    x[::101] *= 1e5
    for bad in (0.0, float("nan")):
        cent[5, 3] = bad
        few = torch.cat([T.trim_ivf_probe(x[i:i + 4000].contiguous(), cent, 1) for i in range(0, nq, 4000)])
        assert torch.equal(T.trim_ivf_probe(x, cent, 1), few)


@pytest.mark.parametrize("nq", (1, 3, 20))
def test_probe_of_few_queries_with_values_that_are_no_numbers(nq):
    """The two kernels for few queries and the one for many put NaN and infinite distances in the same places."""
    import ctypes as C
    import torch
    from paper_2508_17828_amd import trim as T
    g = torch.Generator(device="cuda").manual_seed(nq)
    q, cent = torch.randn((nq, 100), device="cuda", generator=g), torch.randn((300, 100), device="cuda", generator=g)
    cent[7, 3] = float("nan")
    cent[0] = float("inf")
    cent[200:210, 5] = float("nan")
    q[nq - 1, 2] = float("inf")
    if nq > 2:
        q[1] = 1e30                           # (no NaN here: which of two a sum keeps, and their signs differ, is nobody's rule)
    for nprobe in (2, 33, 64):
        assert T.lib().trim_ivf_probe_workspace_bytes(nq, 100, 300, nprobe) > 0
        out = torch.empty((nq, nprobe), dtype=torch.int32, device="cuda")
        assert T.lib().trim_ivf_probe(C.c_void_p(q.data_ptr()), nq, 100, C.c_void_p(cent.data_ptr()), 300, nprobe,
                                      C.c_void_p(out.data_ptr()), C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        assert torch.equal(T.trim_ivf_probe(q, cent, nprobe), out)


# the lists a wave keeps in its registers and one more; more equally near lists than are ranked together
@pytest.mark.parametrize("nlist", (1024, 1025, 2049))
@pytest.mark.parametrize("same", (0, 256, 257, 700))
@pytest.mark.parametrize("nprobe", (2, 31, 64))
def test_probe_selection_of_equally_near_lists(T, oracle, nlist, same, nprobe):
    import torch
    rng = np.random.default_rng(nlist + same)
    cent = rng.integers(-9, 10, (nlist, 8)).astype(np.float32)
    q = rng.integers(-9, 10, (3, 8)).astype(np.float32)
    cent[rng.permutation(nlist)[:same]] = q[1] + 1
    assert T.lib().trim_ivf_probe_workspace_bytes(3, 8, nlist, nprobe) == 3 * nlist * 4
    got = T.trim_ivf_probe(torch.from_numpy(q).cuda(), torch.from_numpy(cent).cuda(), nprobe).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.ivf_probe(q, cent, nprobe))


# queries so far away that all their distances agree in the leading bits that the selection looks at first; some of the lists are one
@pytest.mark.parametrize("nlist,same,nprobe", ((1024, 0, 32), (1025, 300, 64), (3000, 500, 2), (300, 299, 33)))
def test_probe_selection_of_queries_far_from_all_lists(T, oracle, nlist, same, nprobe):
    import torch
    rng = np.random.default_rng(nlist)
    cent = rng.uniform(0, 255, (nlist, 128)).astype(np.float32)
    cent[rng.permutation(nlist)[:same]] = 7.0
    q = rng.uniform(0, 255, (3, 128)).astype(np.float32)
    q[1:] += np.float32(1e5)
    bits = ((q[1] - cent) ** 2).sum(axis=1).astype(np.float32).view(np.uint32) >> 12
    assert np.unique(bits).size <= 4
    assert T.lib().trim_ivf_probe_workspace_bytes(3, 128, nlist, nprobe) == 3 * nlist * 4
    got = T.trim_ivf_probe(torch.from_numpy(q).cuda(), torch.from_numpy(cent).cuda(), nprobe).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.ivf_probe(q, cent, nprobe))


# what the selection through the matrix cores takes: lists and values that leave its tiles unfilled, more queries than fit its
# scores at a time, as many probes as it takes; ties, more lists in one place than a query's candidates can be (300 of 1501),
# rows out of the scaled range, and what is no number: the same lists as the kernel that measures every pair
@pytest.mark.parametrize("nq,nlist,d,nprobe", ((40001, 64, 36, 8), (9800, 257, 132, 32), (1700, 1501, 100, 33), (5001, 512, 128, 64),
                                              (1000, 1024, 1000, 8), (120, 8710, 1540, 50), (70001, 1030, 4, 3)))
def test_probe_of_many_queries(nq, nlist, d, nprobe):
    import ctypes as C
    import torch
    from paper_2508_17828_amd import trim as T
    L = T.lib()
    need = L.trim_ivf_probe_workspace_bytes(nq, d, nlist, nprobe)
    assert need > 4 * nlist * min(nq, 60000)
    assert L.trim_ivf_probe_workspace_bytes(nq, d, nlist, 1) == 0          # (one list: the kernels that assign vectors)
    g = torch.Generator(device="cuda").manual_seed(nlist + d)
    q, cent = torch.randn((nq, d), device="cuda", generator=g), torch.randn((nlist, d), device="cuda", generator=g) * 0.7 + 3
    q[: nq // 2] = (2 * q[: nq // 2]).round()              # (whole numbers: ties)
    cent[: nlist // 2] = (2 * cent[: nlist // 2]).round()
    cent[nlist // 2] = cent[3]
    if nlist == 1501:
        cent[600:1200:2] = q[17]
    q[5], q[6], q[7], cent[8, 1], cent[9], cent[10] = 1e30, 3e5, 1e-30, 1e7, float("inf"), 1e-40
    cent[11, 2] = q[nq - 1, 0] = float("nan")
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    want = torch.empty((nq, nprobe), dtype=torch.int32, device="cuda")
    args = (C.c_void_p(q.data_ptr()), nq, d, C.c_void_p(cent.data_ptr()), nlist, nprobe)
    assert L.trim_ivf_probe(*args, C.c_void_p(want.data_ptr()), stream) == 0
    ws = torch.empty((need + 4,), dtype=torch.uint8, device="cuda")
    for shift, size in ((0, need), (4, need), (0, need - 1)):        # (the last: the exact kernels)
        ws.fill_(0xff)
        got = torch.full_like(want, -1)
        assert L.trim_ivf_probe_ws(*args, C.c_void_p(got.data_ptr()), C.c_void_p(ws.data_ptr() + shift), size, stream) == 0
        # (a query with a NaN is equally far from all: which NaN a sum keeps is nobody's rule)
        assert torch.equal(got[:-1], want[:-1])
        assert (got[-1].sort().values.diff() > 0).all()


# of these, `far` are so far from all lists (or no numbers, or equally far) that nearly all lists are candidates: one query, a
# workgroup's eight and one more, more than one turn of the whole grid, several slabs of scores
@pytest.mark.parametrize("nq,nlist,d,nprobe,far", ((2500, 1024, 128, 32, 1), (2500, 1024, 128, 64, 9), (9001, 1030, 36, 3, 9000),
                                                  (3000, 3001, 132, 50, 1025), (70001, 1030, 4, 8, 60000), (120, 8710, 1540, 50, 120),
                                                  (110, 4000, 4096, 50, 55)))
def test_probe_of_many_queries_far_from_all_lists(nq, nlist, d, nprobe, far):
    import ctypes as C
    import torch
    from paper_2508_17828_amd import trim as T
    L = T.lib()
    assert L.trim_ivf_probe_workspace_bytes(nq, d, nlist, nprobe) > 4 * nlist * min(nq, 60000)
    g = torch.Generator(device="cuda").manual_seed(nlist + d)
    q, cent = torch.rand((nq, d), device="cuda", generator=g) * 255, torch.rand((nlist, d), device="cuda", generator=g) * 255
    at = torch.randperm(nq, device="cuda", generator=g)[:far]
    q[at] += 1e5
    if far > 9:
        q[at[::3]], q[at[1::100]] = 1e30, -3e12
        cent[300:700] = cent[299]
    want, got = torch.empty((nq, nprobe), dtype=torch.int32, device="cuda"), T.trim_ivf_probe(q, cent, nprobe)
    assert L.trim_ivf_probe(C.c_void_p(q.data_ptr()), nq, d, C.c_void_p(cent.data_ptr()), nlist, nprobe, C.c_void_p(want.data_ptr()),
                            C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert torch.equal(got, want)


def test_probe_of_many_queries_captured_and_replayed():
    """One graph, other queries on every replay: none, some and all of them far from all lists."""
    import torch
    from paper_2508_17828_amd import trim as T
    nq, nlist, d, nprobe = 3000, 1024, 64, 16
    g = torch.Generator(device="cuda").manual_seed(5)
    cent = torch.rand((nlist, d), device="cuda", generator=g) * 255
    q = torch.rand((nq, d), device="cuda", generator=g) * 255
    assert T.lib().trim_ivf_probe_workspace_bytes(nq, d, nlist, nprobe) > 4 * nq * nlist
    T.trim_ivf_probe(q, cent, nprobe)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = T.trim_ivf_probe(q, cent, nprobe)
    for far in (0, 7, nq, 1, 0):
        new = torch.rand((nq, d), device="cuda", generator=g) * 255
        new[torch.randperm(nq, device="cuda", generator=g)[:far]] += 2e5
        q.copy_(new)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, T.trim_ivf_probe(new, cent, nprobe))


@pytest.mark.parametrize("n", (40, 3000, 200_000))
@pytest.mark.parametrize("dsub,M", ((4, 8), (5, 8), (6, 8), (8, 8), (7, 4), (12, 4)))
def test_encode_values_that_are_no_numbers(T, oracle, dsub, M, n):
    """Rows and centroids with NaN, infinities and values out of the 16-bit range, however the vectors are dealt out: a sub-vector
    without a finite distance takes centroid 0 and makes the landmark distance infinite."""
    import torch
    rng = np.random.default_rng(n + dsub)
    base, cb = rng.normal(size=(n, dsub * M)).astype(np.float32), rng.normal(size=(M, 256, dsub)).astype(np.float32)
    base[3, 1], base[5, 2], base[7, 0], base[9], base[11] = np.nan, np.inf, -1e30, 1e25, np.nan
    cb[1, 7, 0], cb[1, 40, 1], cb[2, 32, 2], cb[3, 9, 3] = np.nan, np.inf, 1e30, -np.inf
    want = oracle.encode(base, cb)
    codes, dlx = T.trim_encode(torch.from_numpy(base).cuda(), torch.from_numpy(cb).cuda())
    np.testing.assert_array_equal(codes.cpu().numpy(), want[0])
    np.testing.assert_array_equal(dlx.cpu().numpy(), want[1])


@pytest.mark.parametrize("n", (40, 3000))
@pytest.mark.parametrize("dsub,M", ((2, 16), (3, 8)))
def test_encode_four_bit_values_that_are_no_numbers(T, dsub, M, n):
    import torch
    from oracle import trim_oracle_fs
    rng = np.random.default_rng(n + dsub)
    base, cb = rng.normal(size=(n, dsub * M)).astype(np.float32), rng.normal(size=(M, 16, dsub)).astype(np.float32)
    base[3, 1], base[5, 2], base[7, 0], base[9] = np.nan, np.inf, -1e30, 1e25
    cb[1, 7, 0], cb[1, 4, 1], cb[3, 9, 1] = np.nan, np.inf, -np.inf
    want = trim_oracle_fs.encode(base, cb)
    codes, dlx = T.trim_fs_encode(torch.from_numpy(base).cuda(), torch.from_numpy(cb).cuda())
    np.testing.assert_array_equal(codes.cpu().numpy(), want[0])
    np.testing.assert_array_equal(dlx.cpu().numpy(), want[1])


@pytest.mark.parametrize("ns", (600, 9000))
def test_training_rows_that_are_no_numbers(T, oracle, ns):
    import torch
    from oracle import index_build
    rng = np.random.default_rng(ns)
    x = rng.standard_normal((ns, 64)).astype(np.float32)
    x[100, 3], x[200, 20], x[300] = np.nan, np.inf, -np.inf
    init = rng.permutation(np.setdiff1d(np.arange(ns), (100, 200, 300)))[:256].astype(np.int32)
    init[9] = 200
    g = lambda a: torch.from_numpy(a).cuda()
    np.testing.assert_array_equal(T.trim_train_pq(g(x), 16, 3, g(init)).cpu().numpy(), index_build.train_pq_fixed(x, 16, 3, init))
    np.testing.assert_array_equal(T.trim_fs_train_pq(g(x), 32, 3, g(init[:16].copy())).cpu().numpy(),
                                  index_build.train_pq_fs_fixed(x, 32, 3, init[:16]))
    # (one iteration: the oracle's lists take what is no number to the first, and stay there once its centroid is none)
    np.testing.assert_array_equal(T.trim_train_ivf(g(x), 70, 1, g(init[:70].copy())).cpu().numpy(),
                                  index_build.train_ivf_fixed(x, 70, 1, init[:70]))


# many short lists and a few long ones (the instances with 256 and with 1024 threads a list); empty lists, one of all the codes
@pytest.mark.parametrize("n,M,nlist", ((3000, 32, 700), (3000, 192, 500), (5000, 4, 90), (3000, 32, 16), (9000, 192, 30), (1, 8, 5)))
def test_list_summaries(T, n, M, nlist):
    import torch
    rng = np.random.default_rng(n + M)
    cuts = np.sort(rng.integers(0, n + 1, nlist - 1))
    cuts[: nlist // 3] = cuts[nlist // 3]                # one long list, empty ones behind it
    lo = np.concatenate([[0], np.sort(cuts), [n]]).astype(np.int64)
    codes = rng.integers(0, 60, (n, M)).astype(np.uint8) * rng.integers(1, 5, M).astype(np.uint8)
    codes[lo[-2]:, 1] = rng.integers(0, 256, n - lo[-2])
    dlx = rng.random(n).astype(np.float32)
    cuda = lambda a: torch.from_numpy(a).cuda()
    ix = T.Index(torch.zeros((n, 4 * M), device="cuda"), cuda(codes), cuda(dlx), torch.zeros((M, 256, 4), device="cuda"), list_offsets=cuda(lo))
    rec = T.trim_pack_list_bounds(ix).cpu().numpy().reshape(nlist, -1)
    for l in range(nlist):
        own, r = codes[lo[l]:lo[l + 1]], rec[l]
        assert r[(M * 65 + 3) // 4 * 4:][:4].view(np.float32)[0] == (dlx[lo[l]:lo[l + 1]].max() if len(own) else 0)
        for j in range(M):
            want, count = np.unique(own[:, j]), r[M * 64 + j]
            if 0 < len(want) <= 64:
                assert count == len(want)
                np.testing.assert_array_equal(r[j * 64:(j + 1) * 64], np.pad(want, (0, 64 - len(want)), constant_values=want[0]))
            else:
                assert count == (255 if len(want) else 0) and not r[j * 64:(j + 1) * 64].any()
