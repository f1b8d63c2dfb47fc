"""CPU-only: the kernels of the update step with work space (csrc/trim_update.h), compiled for the CPU as they stand, a lane per
fiber.  Behind the work space nothing is mapped, so that an access past it ends the run; the sums are those of the rows in row order."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2508_17828_amd", "csrc", "trim_update.h")

# What the kernels use of the device, for lanes that take turns: a barrier (of a wave's lanes, of the workgroup's) lets the others go on.
SHIM = r"""
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <vector>
#include <sys/mman.h>
#include <ucontext.h>
#define __global__
#define __device__
#define __forceinline__ inline
#define __shared__ static
#define __align__(n) alignas(n)
#define __launch_bounds__(n)
#define __restrict__
#define __builtin_amdgcn_fence(order, scope) ((void)0)
struct Dim { unsigned x, y; };
static Dim threadIdx, blockIdx, blockDim;
struct float4 { float x, y, z, w; };
static float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
static unsigned char g_smem[160 * 1024];
struct Lane { ucontext_t at; std::vector<char> stack; long passed[2] = {0, 0}; bool done = false; };
static std::vector<Lane> lanes;
static ucontext_t turns;
static std::function<void()> body;
static unsigned self;
static long long box[1024];
static void yield() {
    const unsigned me = self;
    swapcontext(&lanes[me].at, &turns);
    self = me;
    threadIdx = {me, 0};
}
static void meet(int kind) {          // 0: the wave's lanes, 1: the workgroup's
    const unsigned me = self, lo = kind ? 0 : me & ~63u, hi = kind ? (unsigned)lanes.size() : lo + 64;
    const long mine = ++lanes[me].passed[kind];
    for (;;) {
        bool all = true;
        for (unsigned i = lo; i < hi; ++i) all = all && (lanes[i].done || lanes[i].passed[kind] >= mine);
        if (all) return;
        yield();
    }
}
static void sync_block() { meet(1); }
static void __builtin_amdgcn_wave_barrier() { meet(0); }
template <typename F> static auto exchange(long long v, F read) {
    box[self] = v;
    meet(0);
    const auto r = read(&box[self & ~63u]);
    meet(0);
    return r;
}
static int __shfl_up(int v, int off) {
    const int l = self & 63;
    return exchange(v, [&](long long *b) { return (int)b[l >= off ? l - off : l]; });
}
static int __builtin_amdgcn_readlane(int v, int from) { return exchange(v, [&](long long *b) { return (int)b[from]; }); }
static unsigned long long __ballot(bool v) {
    return exchange(v, [](long long *b) { unsigned long long m = 0; for (int i = 0; i < 64; ++i) m |= (unsigned long long)(b[i] != 0) << i; return m; });
}
static int __popcll(unsigned long long m) { return __builtin_popcountll(m); }
static uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)((uint64_t)a * b >> 32); }
static void enter() { body(); lanes[self].done = true; }
static void launch(unsigned gx, unsigned gy, unsigned threads, std::function<void()> kernel) {
    body = kernel;
    blockDim = {threads, 1};
    for (unsigned y = 0; y < gy; ++y)
        for (unsigned x = 0; x < gx; ++x) {
            blockIdx = {x, y};
            if (lanes.size() != threads) { lanes.clear(); lanes.resize(threads); }
            for (auto &l : lanes) {
                if (l.stack.empty()) l.stack.resize(64 * 1024);
                l.done = false; l.passed[0] = l.passed[1] = 0;
                getcontext(&l.at);
                l.at.uc_stack.ss_sp = l.stack.data(); l.at.uc_stack.ss_size = l.stack.size(); l.at.uc_link = &turns;
                makecontext(&l.at, enter, 0);
            }
            for (bool any = true; any;) {
                any = false;
                for (unsigned i = 0; i < threads; ++i)
                    if (!lanes[i].done) { any = true; self = i; threadIdx = {i, 0}; swapcontext(&turns, &lanes[i].at); }
            }
        }
}
namespace trim { constexpr int kWave = 64, kXcds = 8, kUpdCols = 256; }
"""
MAIN = r"""
using namespace trim;
template <typename T> static T *fenced(size_t count) {        // ends where nothing is mapped
    const size_t page = 4096, bytes = (count * sizeof(T) + page - 1) / page * page;
    char *p = (char *)mmap(nullptr, bytes + page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (p == MAP_FAILED || mprotect(p + bytes, page, PROT_NONE)) abort();
    return (T *)(p + bytes - count * sizeof(T));
}
int main(int argc, char **argv) {
    const int ns = atoi(argv[1]), dim = atoi(argv[2]), K = atoi(argv[3]), loops = atoi(argv[4]), threads = atoi(argv[5]), group = atoi(argv[6]);
    SortArgs a{};
    float *x = fenced<float>((size_t)ns * dim);
    uint32_t *assign = fenced<uint32_t>(ns);
    a.cent = fenced<float>((size_t)K * dim);
    FILE *f = fopen(argv[7], "rb");
    if (fread(x, 4, (size_t)ns * dim, f) + fread(assign, 4, ns, f) + fread(a.cent, 4, (size_t)K * dim, f) != (size_t)ns * dim + ns + (size_t)K * dim) return 2;
    fclose(f);
    a.x = x; a.assign = assign; a.ns = ns; a.stride = dim; a.astride = 1; a.dim = dim; a.K = K; a.ny = 1;
    a.rows = loops * threads; a.nchunk = (ns + a.rows - 1) / a.rows; a.cg_log2 = group;
    while ((1 << a.kbits) < K) ++a.kbits;
    a.starts = fenced<uint16_t>((size_t)a.nchunk * (K + 1));
    a.list = fenced<uint16_t>(ns);
    if (loops == 4) launch(a.nchunk, 1, threads, [&] { kmeans_sort_kernel<4, 4>(a); });
    else launch(a.nchunk, 1, threads, [&] { kmeans_sort_kernel<4, 1>(a); });
    const int groups = (K + (1 << group) - 1) >> group, grid = (groups + kXcds - 1) / kXcds * kXcds;
    if (dim > kShortRow) launch(K, 1, 64, [&] { kmeans_rows_kernel(a); });
    else if (dim % 4) launch(grid, 1, kSumThreads, [&] { kmeans_sums_kernel<0, false>(a); });
    else if (dim == 4) launch(grid, 1, kSumThreads, [&] { kmeans_sums_kernel<4, true>(a); });
    else launch(grid, 1, kSumThreads, [&] { kmeans_sums_kernel<0, true>(a); });
    fwrite(a.cent, 4, (size_t)K * dim, stdout);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("update")
    text = open(HEADER).read().replace("#pragma once", "").replace('#include "trim_aux.h"', "")
    text = text.replace("extern __shared__ __align__(16) unsigned char smem[];", "unsigned char *smem = g_smem;")
    src = d / "update.cpp"
    src.write_text(SHIM + text + MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-w", "-o", str(d / "update"), str(src)], check=True)
    return d


# clusters without a row at all, and without one in the last group of 64 chunks; 1, 63, 64, 65 and 130 chunks, the last of them full, short
# of a row or with one row only; one cluster a workgroup and several; rows of 2 to 20 values
@pytest.mark.parametrize("chunks", (1, 63, 64, 65, 130))
@pytest.mark.parametrize("last", (1, 63, 64))
@pytest.mark.parametrize("dim,K,group", ((4, 9, 0), (4, 40, 3), (8, 5, 0), (12, 33, 2), (16, 9, 1), (2, 7, 0), (20, 6, 0)))
def test_update_stays_within_its_work_space(program, chunks, last, dim, K, group):
    rng = np.random.default_rng(chunks * 100 + last + dim)
    threads = 64
    ns = (chunks - 1) * threads + last
    x = rng.standard_normal((ns, dim)).astype(np.float32)
    assign = rng.integers(0, K - 2, ns).astype(np.uint32)               # (the last two have none)
    assign[64 * threads:] = 1
    assign[assign == 3] = 0                                             # (nor has one in the middle)
    cent = rng.standard_normal((K, dim)).astype(np.float32)
    data = program / "in.bin"
    data.write_bytes(x.tobytes() + assign.tobytes() + cent.tobytes())
    p = subprocess.run([str(program / "update"), *map(str, (ns, dim, K, 1, threads, group)), str(data)], capture_output=True, timeout=60)
    assert p.returncode == 0, p.returncode
    sums = np.zeros((K, dim))
    np.add.at(sums, assign, x.astype(np.float64))
    count = np.bincount(assign, minlength=K)
    want = np.where(count[:, None] > 0, sums / np.maximum(count, 1)[:, None], cent).astype(np.float32)
    np.testing.assert_array_equal(np.frombuffer(p.stdout, np.float32).reshape(K, dim), want)
