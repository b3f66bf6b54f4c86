"""Host check of the kernels' array offsets (csrc/carve.h): 64-bit arrays start
at multiples of 8 for even and odd numbers of states, arrays do not overlap,
and the sizes the host launches with hold them."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1701_03038_amd", "csrc")

SOURCE = r"""
#include "carve.h"
#include <algorithm>
#include <cstdio>
using namespace wfst;
int main()
{
    int bad = 0;
    for (int64_t Q : {1, 2, 3, 90, 91, 2000, 2001, 2071, 12000, 12001})
        for (int64_t segs : {0, 1, 2, 77, 361})
            for (int64_t slots : {0, 1, 2, 5, 400}) {
                const int64_t s = std::max<int64_t>(segs, 1), c = std::max<int64_t>(slots, 1);
                const LseCarve l = lse_carve(Q, segs, slots);
                const RestCarve r = rest_carve(Q, segs, slots);
                const bool ok = l.vval % 8 == 0 && l.part % 8 == 0 && l.vkey % 4 == 0 && (int64_t)l.vval >= 8 * (Q + 1) &&
                                (int64_t)(l.part - l.vval) >= 8 * s && (int64_t)(l.vkey - l.part) >= 8 * c &&
                                (int64_t)(l.end - l.vkey) >= 4 * s && r.lse.vval % 8 == 0 && r.lse.part % 8 == 0 &&
                                r.part_s >= r.lse.end && r.part_s % 4 == 0 && (int64_t)(r.marks - r.part_s) >= 4 * c &&
                                (int64_t)(r.end - r.marks) >= 3 * (Q + 1);
                if (!ok) {
                    std::printf("Q=%lld segs=%lld slots=%lld\n", (long long)Q, (long long)segs, (long long)slots);
                    bad = 1;
                }
            }
    return bad;
}
"""


def test_offsets(tmp_path):
    src = tmp_path / "carve.cpp"
    src.write_text(SOURCE)
    exe = str(tmp_path / "carve")
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
