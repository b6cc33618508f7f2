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
    long long first, H, rows, i;
    while (std::scanf("%lld %lld %lld %lld", &first, &H, &rows, &i) == 4) {
        const fftconv::LongRows r = H ? fftconv::long_row_pairs(first, H, rows) : fftconv::long_rows(first);
        std::printf("%lld %d\\n", (long long)r.at((uint32_t)i), (int)r.partner((uint32_t)i));
    }
}
""")
    exe = d / "main"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", CSRC, "-o", str(exe),
                    str(d / "main.cpp")], check=True)
    return str(exe)


@pytest.mark.parametrize("H,B", [(1, 7), (3, 2), (16, 9), (768, 64), (1 << 17, 65538), (65535, 1 << 18), ((1 << 24) - 1, 1031), (1, 1 << 34)])
def test_rows_of_pairs(program, H, B):
    pairs, rows = (B + 1) // 2 * H, B * H
    ask = set()
    for first in (0, 1, H - 1, H, pairs // 3, pairs // 2, (1 << 32) - 40000, (1 << 32) - 1, 1 << 32, pairs - 65535, pairs - H, pairs - 1):
        for i in (0, 1, H - 1, H, 32767, 40000, 65534):
            if 0 <= first and 0 <= i < 65535 and first + i < pairs:
                ask.add((first, i))
    ask = sorted(ask)
    text = "".join("%d %d %d %d\n" % (f, H, rows, i) for f, i in ask)
    out = subprocess.run([program], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    assert len(ask) > 3
    for (f, i), line in zip(ask, out):
        j = f + i
        want = 2 * (j // H) * H + j % H
        assert line == "%d %d" % (want, want + H < rows), (f, i)


def test_single_rows(program):
    ask = [(0, 0), (5, 65534), ((1 << 33) + 7, 40000)]
    out = subprocess.run([program], input="".join("%d 0 0 %d\n" % a for a in ask), capture_output=True, text=True, check=True).stdout.split("\n")
    assert [int(l.split()[0]) for l in out[:3]] == [sum(a) for a in ask]
