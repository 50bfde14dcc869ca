"""The roundings that the ranking's check counts (csrc/topk_bound.hpp) against the scan's arithmetic in its worst case."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2211_12281_amd", "csrc")


@pytest.fixture(scope="module")
def units(tmp_path_factory):
    d = tmp_path_factory.mktemp("bound")
    (d / "u.cpp").write_text('#include "topk_bound.hpp"\n#include <cstdio>\n#include <cstdlib>\n'
                             "int main(int, char **a) { int d = atoi(a[1]); bool b = a[2][0] == '1';\n"
                             'printf("%d %d", topk_product_units(d, b), topk_distance_units(d, b)); }\n')
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "u.cpp"), "-o", str(d / "u")], check=True)
    return lambda dim, bf16: tuple(map(int, subprocess.run([str(d / "u"), str(dim), str(int(bf16))], capture_output=True, text=True,
                                                           check=True).stdout.split()))


def _toward_zero(x):
    """fp64 -> fp32, truncated."""
    y = np.float32(x)
    return np.nextafter(y, np.float32(0)) if abs(np.float64(y)) > abs(x) else y


def _pieces(x):
    e = 14 - int(np.floor(np.log2(np.abs(x).max())))
    y = np.ldexp(x.astype(np.float64), e)
    hi = y.astype(np.float16).astype(np.float64)
    return hi, (y - hi).astype(np.float16).astype(np.float64), e


def _error_units(a, b, bf16):
    """Error of the scan's sum of a . b in units of 2^-23 |a| |b|: one sum after the other, every one truncated."""
    acc = np.float32(0)
    if bf16:
        terms, e = [x * y for x, y in zip(a.astype(np.float64), b.astype(np.float64))], 0
    else:
        (ah, al, ea), (bh, bl, eb) = _pieces(a), _pieces(b)
        terms, e = [t for i in range(len(a)) for t in (ah[i] * bl[i], al[i] * bh[i], ah[i] * bh[i])], ea + eb
    for t in terms:
        acc = _toward_zero(np.float64(acc) + t)
    a64, b64 = a.astype(np.float64), b.astype(np.float64)
    return abs(np.ldexp(np.float64(acc), -e) - a64 @ b64) / (2.0 ** -23 * np.linalg.norm(a64) * np.linalg.norm(b64))


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d", [8, 16, 128, 256])
def test_every_sum_of_the_scan_is_counted(units, d, bf16):
    """One large product and many small ones of the other sign, each of whose sums takes a truncated sum down by a last bit; elements that lose
    their last bit in two pieces; and rows at random."""
    g = np.random.default_rng(d)
    products, distances = units(d, bf16)
    lose = np.float32(1 + 2.0 ** -12 + 2.0 ** -23)
    small = np.full(d, 2.0 ** -19 * (1 + 2.0 ** -12), np.float32)
    a, b = small.copy(), -small
    a[0] = b[0] = 1
    cases = [(a, b), (np.full(d, lose), np.full(d, lose))] + [tuple(g.normal(size=(2, d)).astype(np.float32)) for _ in range(20)]
    cases += [(x, np.abs(x) * np.exp2(g.integers(-12, 1, d)).astype(np.float32)) for x in g.normal(size=(5, d)).astype(np.float32)]
    for x, y in cases:
        if bf16:
            x, y = ((v.view(np.uint32) & 0xFFFF0000).view(np.float32) for v in (np.ascontiguousarray(x), np.ascontiguousarray(y)))
        u = _error_units(x, y, bf16)
        assert u <= products
        # 2 q.t as a part of units of 2^-22 (|q| + |t|)^2, which is 4 |q| |t| at least; a quarter of them and more is left for the norms
        assert u / 4 <= 0.75 * distances
