"""The candidates of a ranking's sample (csrc/topk_sample.hpp): inside the table, none twice, and of all phases of a period."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2211_12281_amd", "csrc")


@pytest.fixture(scope="module")
def sample(tmp_path_factory):
    d = tmp_path_factory.mktemp("sample")
    (d / "s.cpp").write_text('#include "topk_sample.hpp"\n#include <cstdio>\n#include <cstdlib>\n'
                             "int main(int, char **a) { long n = atol(a[1]), t = atol(a[2]); TopkSample s = topk_sample(n, t);\n"
                             "for (long i = 0; i < t; ++i) for (int r = 0; r < 32; ++r) { int c = s.first(r) + (int)s.place((uint32_t)i);\n"
                             "fwrite(&c, 4, 1, stdout); } }\n")
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "s.cpp"), "-o", str(d / "s")], check=True)
    return lambda n, tiles: np.frombuffer(subprocess.run([str(d / "s"), str(n), str(tiles)], capture_output=True, check=True).stdout, np.int32)


@pytest.mark.parametrize("n,tiles", [(4097, 128), (8191, 128), (8192, 255), (15_871, 128), (15_872, 247), (31_743, 300), (31_744, 300), (39_050, 610),
                                     (179_343, 2724), (1 << 20, 900), (1_000_003, 1), (5_701_914, 3000), (2**31 - 1, 6770), (2**31 - 1, 2**16 + 1)])
def test_no_candidate_twice_and_none_outside(sample, n, tiles):
    c = sample(n, tiles)
    assert c.size == 32 * tiles and c.min() >= 0 and c.max() < n
    assert np.unique(c).size == c.size
    # every 64th of the table has its share: one more or less per part that it touches, and the gaps between parts are a 32nd of the table in all
    if tiles >= 128:
        share = np.histogram(c, 64, (0, n))[0] / (c.size / 64)
        assert 0.7 < share.min() and share.max() < 1.6


@pytest.mark.parametrize("n,tiles", [(1 << 20, 900), (1 << 20, 2048), (1_000_000, 2000), (262_144, 512)])
def test_all_phases_of_a_period(sample, n, tiles):
    c = sample(n, tiles)
    for period in (2, 8, 32, 1024, n // 1000, n // 32):
        bins = min(period, 16)
        share = np.histogram(c % period, bins, (0, period))[0] / (c.size / bins)
        assert 0.7 < share.min() and share.max() < 1.3, (period, share)
