"""Index arithmetic of the launches (csrc/work_index.h), compiled for the CPU, at sizes beyond what a test can run."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_05908_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("work_index")
    (d / "main.cpp").write_text("""
#define __host__
#define __device__
#include "work_index.h"
#include <cstdio>
int main()
{
    char what;
    long long a, b, c, d;
    while (std::scanf(" %c %lld %lld %lld %lld", &what, &a, &b, &c, &d) == 5) {
        if (what == 'r') {                                // row d of a launch from row or pair a on; b channels, c rows
            const fftconv::LongRows r = b ? fftconv::long_row_pairs(a, b, c) : fftconv::long_rows(a);
            std::printf("%lld %d\\n", (long long)r.at((uint32_t)d), (int)r.partner((uint32_t)d));
        } else if (what == 'w') {                         // a workgroup's items from a on: every b-th of c; the last one and how many
            int v = (int)a, n = 1;
            for (; fftconv::big_item_follows(v, (int)b, (int)c); v += (int)b) ++n;
            std::printf("%d %d\\n", v, n);
        } else if (what == 'g') {                         // a channels of b items on a chip of c workgroups
            const fftconv::BigSplit g = fftconv::big_split(a, b, c);
            std::printf("%d %d\\n", g.grid, g.nx);
        } else {                                          // a batch rows of b channels
            std::printf("%d 0\\n", (int)fftconv::big_items_fit(a, b));
        }
    }
}
""")
    exe = d / "main"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", CSRC, "-o", str(exe),
                    str(d / "main.cpp")], check=True)
    return str(exe)


def answers(program, lines):
    text = "".join("%s %d %d %d %d\n" % l for l in lines)
    out = subprocess.run([program], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    return [tuple(int(x) for x in l.split()) for l in out if l]


@pytest.mark.parametrize("H,B", [(1, 7), (3, 2), (16, 9), (768, 64), (1 << 17, 65538), (65535, 1 << 18), ((1 << 24) - 1, 1031), (1, 1 << 34)])
def test_rows_of_pairs(program, H, B):
    pairs, rows = (B + 1) // 2 * H, B * H
    ask = set()
    for first in (0, 1, H - 1, H, pairs // 3, pairs // 2, (1 << 32) - 40000, (1 << 32) - 1, 1 << 32, pairs - 65535, pairs - H, pairs - 1):
        for i in (0, 1, H - 1, H, 32767, 40000, 65534):
            if 0 <= first and 0 <= i < 65535 and first + i < pairs:
                ask.add((first, i))
    ask = sorted(ask)
    assert len(ask) > 3
    want = [2 * ((f + i) // H) * H + (f + i) % H for f, i in ask]
    assert answers(program, [("r", f, H, rows, i) for f, i in ask]) == [(w, int(w + H < rows)) for w in want]


def test_single_rows(program):
    ask = [(0, 0), (5, 65534), ((1 << 33) + 7, 40000)]
    assert [a for a, _ in answers(program, [("r", f, 0, 0, i) for f, i in ask])] == [sum(a) for a in ask]


@pytest.mark.parametrize("step", [1, 32, 255, 512])
@pytest.mark.parametrize("items", [1, 2, 511, 512, 513, 100000, (1 << 31) - 600, (1 << 31) - 512, (1 << 31) - 9])
def test_items_of_a_workgroup(program, items, step):
    first = [f for f in (0, 1, 31, items - 1, items - step, items - 2 * step + 1, items - 5 * step) if 0 <= f < items and (items - f) // step < 10 ** 6]
    got = answers(program, [("w", f, step, items, 0) for f in first])
    assert got == [(f + (items - 1 - f) // step * step, (items - 1 - f) // step + 1) for f in first]


def test_item_limits(program):
    fits = [(1, 1), ((1 << 31) - 2, 1), ((1 << 31) - 10, 2), (2, (1 << 31) - 9), (5, 30000)]
    not_ = [((1 << 31) - 1, 1), (1 << 32, 1), ((1 << 32) + 4, 1), ((1 << 31) - 9, 2), (2, (1 << 31) - 8), (1 << 20, 1 << 20)]
    assert answers(program, [("f", B, H, 0, 0) for B, H in fits]) == [(1, 0)] * len(fits)
    assert answers(program, [("f", B, H, 0, 0) for B, H in not_]) == [(0, 0)] * len(not_)


def test_split_of_items(program):
    """As few steps of a workgroup as all the chip's workgroups allow, channels dealt to the dies where that takes no more; H = 37 and 65 took two steps."""
    shapes = [(H, pairs, resident) for H in (1, 2, 7, 8, 9, 15, 16, 17, 37, 40, 64, 65, 100, 255, 256, 257, 300, 768, 1032)
              for pairs in (1, 2, 3, 8, 17, 32, 255) for resident in (256, 512, 304, 4)]
    for (H, pairs, resident), (grid, nx) in zip(shapes, answers(program, [("g", H, p, r, 0) for H, p, r in shapes])):
        items = H * pairs
        best = -(-items // min(items, resident))
        assert 1 <= grid <= min(items, resident) and (nx == 1 or (nx == 8 and grid % 8 == 0))
        # die x: channels x, x + nx, ...; its workgroups take its items in turn
        steps = max(-(-len(range(x, H, nx)) * pairs // (grid // nx)) for x in range(nx))
        assert steps == best, (H, pairs, resident, grid, nx)
        if nx == 1 and resident >= 8 and items >= 8:
            each = min(items, resident) // 8
            assert -(-(-(-H // 8) * pairs) // each) > best
