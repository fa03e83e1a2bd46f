"""The long accumulator (long_sum.h) compiled for the host: what a double adds to its words is that double."""
import os
import random
import struct
import subprocess
from fractions import Fraction

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include "long_sum.h"
#include <stdio.h>
int main() {
    unsigned long long bits;
    printf("%d %d\n", LONG_WORDS, LONG_SHIFT);
    while (scanf("%llx", &bits) == 1) {
        printf("%d", (int)long_fits(bits));
        for (uint32_t i = 0; i < LONG_WORDS; ++i) printf(" %lld", (long long)long_word(bits, i));
        printf("\n");
    }
}
"""


def test_words_add_up_to_the_double(tmp_path):
    src, exe = tmp_path / "long.cpp", tmp_path / "long"
    src.write_text(MAIN)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", os.path.join(ROOT, "paper_2605_01989_amd", "csrc"), "-o", str(exe), str(src)])
    rng = random.Random(1)
    # every exponent of a sum of squares of floats, the ends of its range and what lies outside
    fit = [s * m * 2.0 ** e for e in range(-298, 272) for s in (1, -1) for m in (1.0, 2 - 2.0 ** -52, 1 + rng.random())]
    top = (3.4028234663852886e38) ** 2 * 65535
    fit += [top, -top, 2.0 ** -298]
    out = [0.0, -0.0, float("inf"), float("-inf"), float("nan"), 5e-324, 2.0 ** -320, 1e300]
    bits = [struct.unpack("<Q", struct.pack("<d", x))[0] for x in fit + out]
    done = subprocess.run([str(exe)], input="\n".join(f"{b:x}" for b in bits), capture_output=True, text=True, check=True).stdout.splitlines()
    words, shift = map(int, done[0].split())
    for x, line in zip(fit, done[1:]):
        fits, *w = map(int, line.split())
        assert fits and len(w) == words and all(abs(v) < 2 ** 32 for v in w)
        assert sum(Fraction(v) * Fraction(2) ** (32 * i - shift) for i, v in enumerate(w)) == Fraction(x)
    assert [int(line.split()[0]) for line in done[1 + len(fit):]] == [0] * len(out)
