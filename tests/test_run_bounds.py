"""Host bounds of the ordered output's work arrays, from the library's own header.

max_runs(n) must hold the runs of any number of accepted samples up to n, and
max_segments(w, points) the segments of any division of up to w accept words among
the points; runs cover the samples, each but the last in full.  Compiled for the
CPU and checked around every change of length.
"""
import os
import subprocess

SRC = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "tkdv_internal.h"
using namespace tkdv;
typedef unsigned long long u64;
int main()
{
    std::vector<u64> at = {0, 1, 2};
    for (int e = 3; e < 44; ++e)
        for (long long d = -2; d <= 2; ++d)
            for (u64 f : {16ull, 17ull, 24ull, 31ull}) at.push_back((f << e) / 16 + d);
    std::sort(at.begin(), at.end());
    for (int K : {8, 32, 64, 128}) {
        u64 most = 0;
        for (u64 n : at) {
            const u64 R = 1ull << run_shift(K, n), r = runs_of(K, n);
            if (r * R < n || (n && (r - 1) * R >= n)) return printf("runs of %llu\n", n), 1;
            if (r > (32 * R > 8192 ? 32 * R : 8192)) return printf("short runs of %llu\n", n), 1;
            if (R >= 128 && r <= 512) return printf("long runs of %llu\n", n), 1;
            most = std::max(most, r);
            if (max_runs(K, n) < most) return printf("max_runs(%llu) = %llu < %llu\n", n, max_runs(K, n), most), 1;
            if (max_runs(K, n) > most + most / 8) return printf("max_runs(%llu) far above %llu\n", n, most), 1;
        }
    }
    for (u64 w : at) {
        if (w > (1ull << 40)) break;
        for (int np : {1, 2, 7, 1000}) {
            // the words spread evenly with one more each, so that every point's last segment is short
            const int sh = seg_shift_for(w);
            const u64 per = w / np, segs = np * ((per + (1ull << sh) - 1) >> sh);
            if (segs > max_segments(w, np)) return printf("max_segments(%llu, %d)\n", w, np), 1;
        }
        // a shorter decided range has no more segments than the whole one may have
        for (u64 v : {w / 2, w / 3, w - w / 100})
            if (((v + (1ull << seg_shift_for(v)) - 1) >> seg_shift_for(v)) > max_segments(w, 1))
                return printf("max_segments(%llu) of %llu\n", w, v), 1;
    }
    return 0;
}
"""


def test_bounds(tmp_path):
    root = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2411_16952_amd", "csrc")
    src = tmp_path / "bounds.cpp"
    src.write_text(SRC)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", root, "-o", str(tmp_path / "bounds"), str(src)], check=True)
    r = subprocess.run([str(tmp_path / "bounds")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
