"""CPU-only checks of the boundary: libtrim.so loads, exports every function that
include/trim.h declares, and rejects bad arguments on the host before touching a GPU."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "trim.h")


@pytest.fixture(scope="module")
def L():
    from paper_2508_17828_amd import trim
    if not os.path.exists(trim.LIB_PATH):
        from paper_2508_17828_amd import build
        build.build()
    return trim.lib()


def declared_functions():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(trim_[a-z0-9_]+)\s*\(", src)))


def test_every_declared_function_is_exported(L):
    from paper_2508_17828_amd import trim
    names = declared_functions()
    assert set(names) == set(trim.EXPORTS), (names, trim.EXPORTS)
    for n in names:
        assert getattr(L, n) is not None


def test_header_cites_the_paper_for_each_operation():
    src = open(HEADER).read()
    for name, cite in (("trim_encode", "Section 3.3"), ("trim_build_lut", "Section 3.3"),
                       ("trim_search_knn", "Section 4.2"), ("trim_search_range", "Section 4.2"),
                       ("trim_ivf_probe", "Section 6.1"), ("trim_query_order", "Section 6.1")):
        decl = src.index("int " + name)
        comment = src.rfind("/*", 0, decl)
        assert cite in src[comment:decl], name


def test_host_side_validation(L):
    from paper_2508_17828_amd import trim
    assert L.trim_shape_supported(128, 32) == 1
    assert L.trim_shape_supported(128, 16) == 1
    assert L.trim_shape_supported(960, 120) == 1
    assert L.trim_shape_supported(1536, 192) == 1
    assert L.trim_shape_supported(130, 13) == 0      # d % 4
    assert L.trim_shape_supported(128, 6) == 0       # d % M
    assert L.trim_shape_supported(120, 30) == 0      # M % 4
    assert L.trim_strerror(0) == b"ok"
    assert b"shape" in L.trim_strerror(-2)
    assert L.trim_version().decode().count(".") == 1
    assert L.trim_range_workspace_bytes(100, 10_000) >= 100 * 10_000 // 8
    # null index / bad sizes are refused before any HIP call
    assert L.trim_search_knn(None, None, 1, None, None, 10, 0.0, 64, None, None, None, None, None, 0, None) == -1
    view = trim._IndexView(10, 128, 32, None, None, None, None, None)
    assert L.trim_search_knn(C.byref(view), None, 1, None, None, 10, 0.0, 64, None, None, None, None, None, 0, None) == -1
    view = trim._IndexView(0, 128, 6, None, None, None, None, None)
    assert L.trim_search_knn(C.byref(view), None, 1, None, None, 10, 0.0, 64, None, None, None, None, None, 0, None) == -2
    assert L.trim_encode(None, 5, 128, None, 32, None, None, None) == -1
    assert L.trim_encode(None, 0, 128, None, 32, None, None, None) == 0
    assert L.trim_encode(None, 5, 128, None, 6, None, None, None) == -2
    assert L.trim_build_lut(None, 3, 128, None, 32, None, 0, None) == -1
    assert L.trim_ivf_probe(None, 3, 128, None, 16, 32, None, None) == -1   # nprobe > nlist
    # sizes of caller-owned buffers (pure host functions)
    assert L.trim_list_bounds_bytes(7, 32) == 7 * 2096     # 32 x 64 codes + 32 counts + 4, to 16
    assert L.trim_list_bounds_bytes(0, 32) == 0 and L.trim_list_bounds_bytes(5, 0) == 0
    small, large = L.trim_range_workspace_bytes(10, 1000), L.trim_range_workspace_bytes(10, 100_000)
    assert small % 256 == 0 and large > small >= 10 * 1000 * 4   # a distance slot per candidate
    assert L.trim_codes_tiled_bytes(100, 192) >= 100 * 192
    # the list-summary and ceiling entry points refuse null buffers on the host
    assert L.trim_pack_list_bounds(None, None, 4, None, None) == -1
    assert L.trim_ceiling_lds_gather(0, 1, 1, 0, None, None) == -1
    assert L.trim_ceiling_stream_read(None, 1024, 8, None, None) == -1


def view_of(n, d, M, codebooks=1024):
    from paper_2508_17828_amd import trim
    return trim._IndexView(n, d, M, 1024, 1024, 1024, None, codebooks, None, None, 8)


def cand_of(nlist, nprobe, max_candidates):
    from paper_2508_17828_amd import trim
    return trim._Candidates(nlist, nprobe, 1024, 1024, max_candidates, None)


def test_searches_too_large_for_32_bit_counts_do_not_run_in_passes(L):
    """(query, list) pairs are counted in 32 bits, the operands of the queries addressed by as many."""
    view, cand = view_of(4096, 512, 32), cand_of(2048, 2048, 4096)
    assert L.trim_range_scratch_bytes(C.byref(view), 1_000_000, C.byref(cand)) > 0
    assert L.trim_range_scratch_bytes(C.byref(view), 1_048_576, C.byref(cand)) == 0      # 2^31 pairs
    view = view_of(2048, 20480, 640)
    assert L.trim_range_scratch_bytes(C.byref(view), 1_600_000, None) > 0
    assert L.trim_range_scratch_bytes(C.byref(view), 1_700_000, None) == 0               # 2^32 pieces of operands
    assert L.trim_range_scratch_bytes(C.byref(view_of(10_000_000, 512, 32)), 4_000_000, None) > 0
    assert L.trim_range_scratch_bytes(C.byref(view_of(20_000_000, 512, 32)), 4_000_000, None) == 0      # 2^31 tiles


def test_no_work_space_is_asked_for_where_the_passes_are_refused(L):
    """The size functions ask what the searches ask: centroids, and LDS for every pass at this k and row length."""
    def sizes(view, k):
        return L.trim_knn_workspace_bytes(C.byref(view), 300, None, k, 256), L.trim_range_scratch_bytes(C.byref(view), 300, None)
    assert all(sizes(view_of(4096, 768, 96), 10))
    assert sizes(view_of(4096, 768, 96, codebooks=None), 10) == (0, 0)
    assert all(sizes(view_of(700, 26624, 832), 10))
    assert sizes(view_of(700, 26624, 832), 1000)[0] == 0         # the replay's lists and 1024 result slots
    assert sizes(view_of(700, 26752, 836), 10) == (0, 0)         # the measure pass's means
    # few queries take their bounds from a caller's table as well
    few = view_of(100_000, 100, 20, codebooks=None)
    assert L.trim_knn_workspace_bytes(C.byref(few), 1, None, 10, 256) > 0


def test_product_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2508_17828_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".h", ".hip", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in text.lower() or f == "synth.py", f
    for f in os.listdir(os.path.join(ROOT, "oracle")):
        if f.endswith((".py", ".c")):
            text = open(os.path.join(ROOT, "oracle", f)).read()
            assert "paper_2508_17828_amd" not in text, f


def test_build_refuses_search_kernels_with_static_lds(L):
    """The search kernels address their distance table from LDS address 0.  The build parses the
    compiler's resource remarks and refuses a library in which one of them carries static LDS;
    the built library's own record shows none does."""
    from paper_2508_17828_amd import build
    remarks = ("x.h:1:1: remark: Function Name: _ZN4trim13search_kernelILi0ELi4ELi1ELb0EEEvNS_10SearchArgsE [-R]\n"
               "x.h:1:1: remark:     VGPRs: 80 [-R]\nx.h:1:1: remark:     AGPRs: 0 [-R]\n"
               "x.h:1:1: remark:     ScratchSize [bytes/lane]: 0 [-R]\nx.h:1:1: remark:     Occupancy [waves/SIMD]: 6 [-R]\n"
               "x.h:1:1: remark:     SGPRs Spill: 0 [-R]\nx.h:1:1: remark:     VGPRs Spill: 0 [-R]\n"
               "x.h:1:1: remark:     LDS Size [bytes/block]: %d [-R]\n")
    build.check_resources(build.kernel_resources(remarks % 0))
    with pytest.raises(RuntimeError):
        build.check_resources(build.kernel_resources(remarks % 64))
    rec = [l.split() for l in open(build.RESOURCES)]
    search = [r for r in rec if "search_kernel" in r[0]]
    assert len(search) >= 12 and all("static_lds=0" in r for r in search)


@pytest.mark.parametrize("nq,d,nlist,nprobe,takes", [
    (4097, 128, 16384, 32, True), (4097, 128, 16385, 32, False),         # ivf_probe_kernel's keys fill the LDS
    (4096, 128, 16384, 32, True), (2000, 128, 20000, 32, True), (5000, 128, 65536, 64, False),
    (1000, 2564, 17000, 32, False), (3000, 4096, 16384, 64, True),
    (1 << 31, 128, 1024, 32, False)])
def test_probe_selections_are_refused_whatever_their_work_space(L, nq, d, nlist, nprobe, takes):
    """What trim_ivf_probe refuses and two kernels do not take either is not taken by the third way alone, which needs its
    whole work space: nothing is asked for, and the call is trim_ivf_probe, which refuses on the host."""
    need = L.trim_ivf_probe_workspace_bytes(nq, d, nlist, nprobe)
    assert (need > 0) == takes
    if not takes:        # (no work space is taken, so that nothing is launched on these addresses)
        assert L.trim_ivf_probe_ws(4096, nq, d, 4096, nlist, nprobe, 4096, 4096, 1 << 40, None) in (-1, -2)


def test_which_searches_of_few_queries_are_split(L):
    """More than one query is split over the chip up to a number of lookups that depends on the rows (csrc/trim_api.hip)."""
    def split(n, d, M, nq, k, nlist=0, nprobe=0):
        view = view_of(n, d, M)
        cand = C.byref(cand_of(nlist, nprobe, n)) if nlist else None
        return L.trim_knn_workspace_bytes(C.byref(view), nq, cand, k, 256) > 0
    assert split(1_000_000, 128, 32, 1, 10, 1024, 32) and split(1_000_000, 128, 32, 64, 10, 1024, 32)
    assert not split(1_000_000, 128, 32, 65, 10, 1024, 32)            # 500,000 lookups per value
    assert split(500_003, 384, 48, 67, 10, 1024, 64)
    assert not split(500_003, 384, 48, 71, 10, 1024, 64)              # short rows: 105 million
    assert split(500_000, 768, 96, 96, 10, 1024, 64)                  # long rows: 288 million here
    assert split(30_000, 960, 120, 69, 10) and not split(30_000, 960, 120, 70, 10)      # no lists: 250 million
    assert split(30_000, 128, 32, 128, 10, 173, 8) and not split(30_000, 128, 32, 129, 10, 173, 8)
    assert split(30_000, 128, 32, 256, 100, 173, 8) and not split(30_000, 128, 32, 257, 100, 173, 8)
    assert split(30_000, 768, 96, 128, 100, 173, 8) and not split(30_000, 768, 96, 129, 100, 173, 8)
    assert split(10_000_000, 1536, 192, 1, 10)
