"""The cut of a shared step into chunks (host arithmetic, on the CPU)."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1807_08804_amd", "csrc")

PROG = r"""
#include <initializer_list>
#include <stdio.h>
#include "sgm_share.h"
using namespace sgm;
int main() {
    int64_t bad = 0, runs = 0;
    for (int b = 0; b < 31; ++b)
        for (int64_t d : {-513, -1, 0, 1, 63, 511, 513})
            for (int64_t m : {1, 3, 5, 511}) {
                const int64_t n64 = (m << b) + d;
                if (n64 < 1 || n64 > INT32_MAX) continue;
                for (int32_t h : {0, 1, 4, 63, 64, 511})
                    for (int32_t lo : {64, 512}) {
                        const int32_t n = (int32_t)n64, hi = 8 * lo;
                        const int32_t k = chunk_items(n, h, lo, hi);
                        const int64_t nch = chunk_count(n, k), even = (n64 + h) / (h + 1);
                        ++runs;
                        // every item once, in no more chunks than a claim word counts
                        bool ok = nch <= kMaxChunks && nch * k >= n64 && (nch - 1) * k < n64;
                        // an even share within the limits while they allow it
                        if (n64 <= (int64_t)hi * kMaxChunks)
                            ok = ok && k <= hi && k >= lo && (k == even || k == lo || k == hi ||
                                                              k == chunk_count(n, kMaxChunks));
                        if (!ok && bad++ < 5) printf("n %d helpers %d: %d a chunk\n", n, h, k);
                    }
            }
    printf("%lld runs\n", (long long)runs);
    return bad != 0 || runs < 4000;
}
"""


def test_chunks_of_any_range(tmp_path):
    """Up to the largest range of vertices, a step has at most kMaxChunks
    chunks (a claim word counts 2^20), and even ones below that."""
    src = tmp_path / "share.cpp"
    src.write_text(PROG)
    exe = tmp_path / "share"
    subprocess.run(["g++", "-std=c++17", "-O1", "-ftrapv", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
