"""Width of the packed keys: a candidate of a relaxation is a path plus one
more arc, so it is up to n times the largest weight, and it has to fit the key
as well as every distance does. On the CPU the rule and the packing of the
kernels' header; on the GPU paths on both sides of the rule, against the
oracle."""
import shutil
import subprocess

import numpy as np
import pytest

import oracle
import pins
from gpu_util import assert_same_labels, gpu_labels

MAXD = 2**31 - 2      # the largest distance that a 32-bit key holds

MODEL = r"""
#include <cstdio>
#include <vector>
#include "internal.h"
using namespace chl;

// Trees of a path of n vertices with all weights w, every vertex relaxing
// both its arcs in rounds, with the kernels' packing. Returns 0 if each ends
// within 2n rounds with the right distances.
template <typename K>
int grow(int n, uint64_t w) {
    for (int h = 0; h < n; h++) {
        std::vector<K> key(n, KeyTraits<K>::INF);
        key[h] = pack<K>(0, 1);
        bool more = true;
        for (int round = 0; more; round++) {
            if (round > 2 * n) return 1;
            more = false;
            for (int v = 0; v < n; v++)
                for (int u : {v - 1, v + 1}) {
                    if (u < 0 || u >= n || key[v] == KeyTraits<K>::INF) continue;
                    const K nk = pack<K>((uint64_t)(key[v] >> 1) + w, (uint32_t)(key[v] & 1) & (uint32_t)(u > h));
                    if (nk < key[u]) { key[u] = nk; more = true; }
                }
        }
        for (int v = 0; v < n; v++)
            if ((uint64_t)(key[v] >> 1) != w * (uint64_t)(v > h ? v - h : h - v)) return 2;
    }
    return 0;
}

int main() {
    const int64_t maxd = 2147483646;
    int bad = 0;
    for (int64_t n : {1LL, 2LL, 3LL, 4LL, 66LL, 32768LL, 1048576LL, 2147483646LL})
        for (int64_t w : {(int64_t)1, maxd / n, maxd / n + 1, n > 1 ? maxd / (n - 1) : maxd, maxd + 1}) {
            if (w < 1 || w > 2147483647) continue;
            const int bits = key_bits_for((int32_t)n, (int32_t)w);
            if (bits == 32 && ((pack<uint32_t>((uint64_t)(n * w), 1) >> 1) != (uint64_t)(n * w) ||
                               pack<uint32_t>((uint64_t)(n * w), 1) == KeyTraits<uint32_t>::INF))
                bad++, std::printf("a candidate of n %lld w %lld does not fit\n", (long long)n, (long long)w);
            if (bits != 32 && n * w <= maxd) bad++, std::printf("n %lld w %lld: %d\n", (long long)n, (long long)w, bits);
            if (n > 66) continue;
            if (int r = bits == 32 ? grow<uint32_t>((int)n, w) : grow<uint64_t>((int)n, w))
                bad++, std::printf("path n %lld w %lld: %d\n", (long long)n, (long long)w, r);
        }
    std::printf("keys: %s\n", bad ? "bad" : "ok");
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not found")
def test_candidates_fit_the_key(tmp_path):
    import importlib
    b = importlib.import_module("paper_1907_00140_amd.build")
    src, exe = tmp_path / "model.cpp", str(tmp_path / "model")
    src.write_text(MODEL)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I" + b.CSRC, "-I" + b.INCLUDE,
                    str(src), "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "keys: ok" in r.stdout, r.stdout


# path lengths: a workgroup's smallest trees, and enough vertices for pruning
# levels, teams, groups and the small-tree kernel
@pytest.mark.gpu
@pytest.mark.parametrize("n", [3, 4, 130, 700])
@pytest.mark.parametrize("bits", [32, 64])
def test_paths_at_the_limit(n, bits):
    """All weights the largest that 32 bits hold (a candidate of n * w), or the
    largest whose distances would (n - 1 arcs) but whose candidates do not."""
    w = MAXD // n if bits == 32 else MAXD // (n - 1)
    print("key width", n, bits, w, flush=True)
    row, col, ww = pins.csr_from_edges(n, [(i, i + 1, w) for i in range(n - 1)])
    for order in (np.arange(n, dtype=np.int32), np.arange(n, dtype=np.int32)[::-1].copy(),
                  np.random.default_rng(n).permutation(n).astype(np.int32)):
        ref = oracle.chl(row, col, ww, order)
        for kw in (dict(), dict(delta=1 << 40), dict(prune_hubs=-1), dict(prune_hubs=-1, delta=1 << 40),
                   dict(team_wgs=1, wg_size=64), dict(small=True), dict(hybrid_psi=1), dict(mode="plain")):
            if n > 130 and kw.get("mode"):
                continue
            L, off, hub, dist = gpu_labels(row, col, ww, order, autotune=False, **kw)
            assert_same_labels(off, hub, dist, ref, str((n, bits, kw)))
            assert L.stats()["key_bits"] == bits
            L.free()
