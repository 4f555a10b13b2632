"""Host mirror of the group-minima selection (select.hip), around the range arithmetic it is built from.

kth_range.h is compiled for the host as it stands and run inside a sequential model of the block-wide
k-th smallest search, which checks every bin index before it is used. The search is compared with a
sort on values at both ends of the 32-bit range, and then drives a mirror of the minima, bound and
candidate steps, whose candidates must hold the k first jobs in the order (key, arrival, index) and
stay within the count that the ranking kernel's LDS is sized for.
"""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from tests.test_select_paths import data, order

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_09142_amd", "csrc")
WGS, GROUPS, THREADS = 256, 16, 1024

HARNESS = r"""
#define __host__
#define __device__
#include "kth_range.h"
using namespace elis;

// block_kth for one work-group, its barriers as sequence points. Returns the number of counting rounds,
// or -1 for a bin index out of range, -2 for a range turned over, -3 for a part without the k-th value.
extern "C" int kth(const uint32_t* v, uint8_t* act, int n, int* need, int* active, uint32_t* result) {
    KthRange r{0xffffffffu, 0u};
    for (int q = 0; q < n; ++q) {
        if (act[q] && v[q] < r.lo) r.lo = v[q];
        if (act[q] && v[q] > r.hi) r.hi = v[q];
    }
    for (int rounds = 1;; ++rounds) {
        const int shift = r.shift();
        int bin[kKthBins] = {};
        for (int q = 0; q < n; ++q) {
            if (!act[q]) continue;
            const uint32_t b = r.part(v[q], shift);
            if (b >= static_cast<uint32_t>(kKthBins)) return -1;
            ++bin[b];
        }
        int below = 0, found = -1;
        for (int b = 0; b < kKthBins && found < 0; ++b) {
            if (*need <= below + bin[b]) found = b;
            else below += bin[b];
        }
        if (found < 0) return -3;
        *need -= below;
        *active = bin[found];
        for (int q = 0; q < n; ++q) act[q] = act[q] && r.part(v[q], shift) == static_cast<uint32_t>(found);
        r.cut(static_cast<uint32_t>(found), shift);
        *result = r.lo;
        if (shift == 0) return rounds;
        if (r.hi < r.lo) return -2;
    }
}
"""


@pytest.fixture(scope="module")
def kth(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("kth")
    src, lib = str(d / "kth.cpp"), str(d / "kth.so")
    with open(src, "w") as f:
        f.write(HARNESS)
    subprocess.run([cxx, "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
    fn = ctypes.CDLL(lib).kth

    def run(values, act, need):
        """(value, active, rank among the equal ones, their number) of the need-th smallest active value."""
        v = np.ascontiguousarray(values, np.uint32)
        a = np.ascontiguousarray(act, np.uint8)
        nd, ac, res = ctypes.c_int(need), ctypes.c_int(0), ctypes.c_uint32(0)
        rounds = fn(v.ctypes.data_as(ctypes.c_void_p), a.ctypes.data_as(ctypes.c_void_p), len(v), ctypes.byref(nd), ctypes.byref(ac),
                    ctypes.byref(res))
        assert 1 <= rounds <= 4, rounds
        return res.value, a.astype(bool), nd.value, ac.value

    return run


TOP = 0xFFFFFFFF


def value_sets():
    rng = np.random.default_rng(3)
    yield "uniform", rng.integers(0, 1 << 32, 4096, dtype=np.uint64)
    yield "ends", np.array([0, TOP, 1, TOP - 1, 0, TOP], np.uint64)
    yield "one top", np.full(300, TOP, np.uint64)
    yield "one zero", np.zeros(300, np.uint64)
    finite = 0x80000000 | rng.normal(250.0, 100.0, 10).astype(np.float32).view(np.uint32).astype(np.uint64)
    yield "few below many at the top", np.concatenate([finite, np.full(4086, TOP, np.uint64)])
    for span in (1, 1023, 1024, 1025, 4097, (1 << 22) + 5, (1 << 31) + 77):
        for base in (0, TOP - span):
            yield f"span {span} from {base}", base + rng.integers(0, span + 1, 2000, dtype=np.uint64)


def test_kth_smallest_over_the_whole_range(kth):
    rng = np.random.default_rng(5)
    for name, v in value_sets():
        v = v.astype(np.uint32)
        for act in (np.ones(len(v), bool), rng.random(len(v)) < 0.5):
            if not act.any():
                continue
            s = np.sort(v[act])
            for need in sorted({1, 2, 11, len(s) // 2, len(s) - 1, len(s)}):
                if not 1 <= need <= len(s):
                    continue
                got, left, rank, count = kth(v, act, need)
                want = s[need - 1]
                assert got == want, (name, need)
                assert np.array_equal(left, act & (v == want)) and count == left.sum(), (name, need)
                assert rank == need - np.searchsorted(s, want), (name, need)


def order_keys(pred):
    u = pred.view(np.uint32).copy()
    u[u == 0x80000000] = 0
    key = np.where(u & 0x80000000, ~u, u | 0x80000000).astype(np.uint32)
    key[np.isnan(pred)] = TOP
    return key


def layout(n):
    """Group of every job and the most jobs of one group (minima_layout and quad_first)."""
    per_wg = ((n + 15) // 16 + WGS - 1) // WGS
    quads = 4 * per_wg
    sweeps = (quads + THREADS - 1) // THREADS
    lanes = 1
    while lanes * GROUPS < min(quads, THREADS):
        lanes <<= 1
    i = np.arange(n)
    u = ((i >> 4) // WGS) * 4 + ((i & 15) >> 2)  # quad of the job within its work-group
    return ((i >> 4) % WGS) * GROUPS + (u % THREADS) // lanes, lanes * 4 * sweeps


def candidates(kth, pred, arr, k):
    """Jobs that select_filter_kernel lists, by its own steps."""
    n = len(pred)
    key, rank = order_keys(pred), np.empty(n, np.int64)
    full = order(pred, arr)
    rank[full] = np.arange(n)
    group, _ = layout(n)
    first = np.full(WGS * GROUPS, -1)
    for i in full[::-1]:  # the last one written is the group's smallest
        first[group[i]] = i
    act = first >= 0
    if act.sum() < k:
        return np.ones(n, bool)
    a = arr.astype(np.uint64) ^ np.uint64(1 << 63)
    words = [key, (a >> np.uint64(32)).astype(np.uint32), a.astype(np.uint32), np.arange(n, dtype=np.uint32)]
    need, bound = k, []
    for w in words:
        v, act, need, active = kth(np.where(act, w[first], 0), act, need)
        bound.append(v)
        if len(bound) == 1 and active == need:
            return key <= v
    below, equal = np.zeros(n, bool), np.ones(n, bool)
    for w, v in zip(words, bound):
        below |= equal & (w < v)
        equal &= w == v
    return below | equal


KINDS = ["ascending", "clustered", "few", "one", "special", "mostly_nan", "wide_arrivals", "full_arrivals"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [8193, 12288, 20000, 131075])
def test_candidates_hold_the_first_k(kth, n, kind):
    rng = np.random.default_rng(n + len(kind))
    pred, arr = data(kind, n, rng)
    full = order(pred, arr)
    group, most = layout(n)
    assert np.bincount(group).max() <= most
    for k in sorted({1, 11, 64, 512, 2048, len(np.unique(group))}):
        listed = candidates(kth, pred, arr, k)
        assert listed[full[:k]].all(), (kind, k)
        assert listed.sum() <= min(n, k * most), (kind, k)
