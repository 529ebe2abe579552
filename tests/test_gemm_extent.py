"""Host check of the GEMM tiles' buffer descriptors (gemm_extent.h): every
element of an operand can be read through them and nothing outside it,
whatever the leading dimension and wherever a slice lies in its matrix."""
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_05275_amd", "csrc")

SRC = """
#include "gemm_extent.h"
#include <cstdio>
int main() {
  long long kind, n, first, r, ld;
  while (scanf("%lld %lld %lld %lld %lld", &kind, &n, &first, &r, &ld) == 5)
    printf("%lld\\n", (long long)(kind ? ld::mc_extent(n, r, ld) - ld::mc_offset(first, ld) : ld::kc_extent(n, first, ld)));
}
"""


@pytest.fixture(scope="module")
def extents(tmp_path_factory):
    d = tmp_path_factory.mktemp("extent")
    (d / "x.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", f"-I{CSRC}", str(d / "x.cpp"), "-o", str(d / "x")], check=True)

    def ask(cases):
        text = "\n".join(" ".join(map(str, c)) for c in cases)
        out = subprocess.run([str(d / "x")], input=text, capture_output=True, text=True, check=True).stdout.split()
        return [int(v) for v in out]
    return ask


def _clamped(vals):
    """As dma_make_rsrc takes them: a negative size is none."""
    return [max(0, v) for v in vals]


def test_mn_contiguous_reads_stay_in_the_operand(extents):
    """A step fetches k rows k0..k0+63 and 256 columns from r0, 16 bytes (8
    elements) per lane, from X + k0 ld; a piece is read where its end is within
    the descriptor.  Read pieces end at or before the operand's last element
    and every element of its rows is read."""
    cases = [(1, K, k0, R, ld) for K, R, pad in itertools.product((1, 2, 7, 8, 63, 64, 65, 130), (8, 248, 256, 264, 520),
                                                                  (0, 8, 248, 256, 4096))
             for ld in (R + pad,) for k0 in range(0, K + 64, 64)]
    for (_, K, k0, R, ld), ext in zip(cases, _clamped(extents(cases))):
        last = (K - 1) * ld + R                       # elements from X to the operand's end
        for k in range(k0, k0 + 64):
            for r0 in range(0, R, 256):
                for m in range(r0, r0 + 256, 8):
                    read = ((k - k0) * ld + m + 8) * 2 <= ext
                    if read:
                        assert k * ld + m + 8 <= last, (K, k0, R, ld, k, m)
                    if k < K and m < R:
                        assert read, (K, k0, R, ld, k, m)


def test_k_contiguous_reads_stay_in_the_operand(extents):
    """Rows r0..r0+255, pieces of 8 k below K only: those of rows past R start
    at or past the descriptor's end, the others are within it."""
    cases = [(0, R, r0, 0, K + pad) for R, K, pad in itertools.product((1, 8, 255, 256, 300), (8, 64, 72), (0, 8, 4096))
             for r0 in range(0, R, 256)]
    for (_, R, r0, _, ld), ext in zip(cases, _clamped(extents(cases))):
        for r in range(r0, r0 + 256):
            assert ((r - r0) * ld * 2 >= ext) if r >= R else ((r - r0 + 1) * ld * 2 <= ext)


def test_nothing_is_read_of_an_empty_operand(extents):
    empty = [(1, 0, 0, 512, 0), (1, 0, 0, 512, 512), (1, 64, 64, 512, 512), (1, 8, 64, 8, 8), (0, 0, 0, 0, 64)]
    assert _clamped(extents(empty)) == [0] * 5
