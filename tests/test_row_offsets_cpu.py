"""The rule by which kernels form byte offsets within a row in 32 bits: where it
holds, the last byte of the row has an offset below 2^32, and the next longer row
of the same elements that it refuses does not."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1108_2651_amd", "csrc")


@pytest.fixture(scope="module")
def fits(tmp_path_factory):
    d = tmp_path_factory.mktemp("offsets")
    (d / "t.cpp").write_text('#include "limits.h"\n#include <cstdio>\n#include <cstdlib>\n'
                             "int main(int c, char** v)\n{\n"
                             "    for (int k = 1; k + 1 < c; k += 2)\n"
                             '        std::printf("%d\\n", (int)lbem::offsets32(std::atoll(v[k]), std::atoll(v[k + 1])));\n'
                             "}\n")
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t")], check=True)

    def ask(pairs):
        out = subprocess.run([str(d / "t")] + [str(x) for p in pairs for x in p], check=True, capture_output=True, text=True)
        return [line == "1" for line in out.stdout.split()]
    return ask


def test_rule_is_where_the_offsets_wrap(fits):
    pairs = [(n, b) for b in (2, 4, 8) for n in (1, 100, 2 ** 28, 2 ** 29 - 1, 2 ** 29, 2 ** 29 + 1, 2 ** 29 + 192,
                                                2 ** 30 - 1, 2 ** 30)]
    for (n, b), ok in zip(pairs, fits(pairs)):
        last = (n - 1) * b + b - 1
        assert ok == (last == last % 2 ** 32), (n, b)


def test_every_accepted_fp32_row_fits(fits):
    """Rows have at most 2^30 cells, so only FP64 needs wider offsets."""
    assert fits([(2 ** 30, 4), (2 ** 30, 8)]) == [True, False]
