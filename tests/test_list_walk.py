"""The symbolic lists' walk on the CPU: a wave's lanes in step, every read
checked against the members that the row has."""
import shutil
import subprocess

import pytest

from paper_2112_10037_amd import build

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "list_walk.hpp"

// One wave of 64 lanes with R products each over `total` products whose columns
// repeat every `distinct`; member order as the exchanges of a lane-by-lane run
// leave it, `heads` lists.  Returns reads out of range, or -1 for a wrong count.
static int walk(int R, int total, int distinct, int heads) {
    std::vector<int> head(heads, -1), lc(total), lp(total);
    std::vector<int> prev(64 * R, -1), c(64 * R, 0);
    for (int s = 0; s < R; ++s)
        for (int l = 0; l < 64; ++l) {
            const int p = s * 64 + l;
            if (p >= total) continue;
            c[l * R + s] = (int)((unsigned)(p % distinct) * 2654435761u >> 1);
            int& h = head[(unsigned)c[l * R + s] % heads];
            prev[l * R + s] = h;
            lc[p] = c[l * R + s];
            lp[p] = h < 0 ? msp::kListEnd : h;
            h = p;
        }
    int bad = 0, count = 0;
    auto at = [&](const std::vector<int>& v, int m) {
        if (m < 0 || m >= total) { ++bad; return msp::kListEnd; }
        return v[m];
    };
    for (int g = 0; g < R; g += 4) {
        int live[64];
        uint32_t own[64];
        bool any = false;
        for (int l = 0; l < 64; ++l) {
            live[l] = 0;
            own[l] = 0;
            for (int i = 0; i < 4; ++i) {
                own[l] |= (uint32_t)((g + i) * 64 + l < total) << i;
                live[l] |= (prev[l * R + g + i] >= 0) << i;
            }
            any = any || live[l];
        }
        while (any) {
            any = false;
            for (int l = 0; l < 64; ++l) {
                msp::list_step<4>(&c[l * R + g], &prev[l * R + g], live[l], own[l], [&](int m) { return at(lc, m); },
                                  [&](int m) { return at(lp, m); });
                any = any || live[l];
            }
        }
        for (int l = 0; l < 64; ++l) count += __builtin_popcount(own[l]);
    }
    return bad ? bad : (count == (distinct < total ? distinct : total) ? 0 : -1);
}

// the position of product q of an entry that starts at b0 with product `first`
static long long position(long long b0, int first, int q) {
    const long long at = b0 - first;
    return msp::list_position((uint32_t)at, (uint16_t)(at >> 32), q);
}

int main(int n, char** a) {
    if (n == 4) std::printf("%lld\n", position(atoll(a[1]), atoi(a[2]), atoi(a[3])));
    else std::printf("%d\n", walk(atoi(a[1]), atoi(a[2]), atoi(a[3]), atoi(a[4])));
}
"""


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("walk")
    (d / "walk.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wno-unknown-pragmas", "-I", build.CSRC, str(d / "walk.cpp"), "-o",
                    str(d / "walk")], check=True)
    return str(d / "walk")


@pytest.mark.parametrize("R,total,distinct,heads", [
    (8, 512, 512, 64), (8, 511, 100, 64), (8, 1, 1, 64), (16, 1024, 700, 128), (16, 1000, 1, 8), (16, 700, 650, 1024),
    (4, 65, 64, 1),
])
def test_list_walk_stays_inside(harness, R, total, distinct, heads):
    out = subprocess.run([harness, str(R), str(total), str(distinct), str(heads)], capture_output=True, text=True,
                         check=True)
    assert int(out.stdout) == 0


@pytest.mark.parametrize("b0", [0, 5, (1 << 32) - 3, 1 << 32, (1 << 32) + 100, (1 << 37) + 12_345])
@pytest.mark.parametrize("first,q", [(0, 0), (0, 9000), (7, 7), (16_383, 16_383), (9000, 9007)])
def test_list_positions_keep_their_upper_bits(harness, b0, first, q):
    out = subprocess.run([harness, str(b0), str(first), str(q)], capture_output=True, text=True, check=True)
    assert int(out.stdout) == b0 + (q - first)
