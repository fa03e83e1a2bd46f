"""Where the gather reads a packet (packet_units.h), compiled for the host and walked exhaustively."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WALK = r"""
#include "packet_units.h"
#include <stdio.h>
// Every payload length up to `most`, cut into pieces of np KB: returns the number of units that hold payload and are
// read elsewhere than they lie, or outside their descriptor or the packet, and of units without payload that are read.
template <uint32_t LEAD> static long walk(uint32_t most, uint32_t np) {
    long bad = 0;
    for (uint32_t len = 1; len <= most; ++len) {
        const int64_t end = 8 + 4ll * len, stride = (end + 15) / 16 * 16;
        const uint32_t units = (len + LEAD + 3) / 4;            // units that hold payload
        for (uint32_t u = 0; u < (units + 64 * np - 1) / (64 * np) * 64 * np; ++u) {
            const uint32_t skip = u / (64 * np) * (np * 1024), l = u - skip / 16;
            const int64_t off = unit_offset<LEAD>(len, skip, l), have = unit_have<LEAD>(len, skip), at = unit_base<LEAD>(skip) + off;
            bool ok;
            if (u >= units) ok = off >= have || off < 0;       // zeros, nothing asked of memory
            else {
                const bool tail = !LEAD && 4 * u + 4 > len;    // fewer than four floats: the 16 bytes that end with them
                const int64_t want = tail ? (len > 2 ? end - 16 : 0) : 16ll * u + (LEAD ? 0 : 8);
                ok = off >= 0 && off + 16 <= have && at == want && at >= 0 && at + 16 <= stride;
            }
            if (!ok && bad++ < 3) fprintf(stderr, "LEAD %u np %u len %u unit %u: offset %ld of %ld, byte %ld of %ld\n", LEAD, np, len, u, (long)off, (long)have, (long)at, (long)stride);
        }
    }
    return bad;
}
int main() {
    long bad = 0;
    for (uint32_t np = 1; np <= 5; ++np) bad += walk<0>(4200, np) + walk<2>(20000, np);
    return bad ? 1 : 0;
}
"""


def test_every_unit_of_every_packet_length_is_read_where_it_lies(tmp_path):
    """All lengths up to 4200 floats with units counted from the payload and up to 20000 counted from the packet,
    in pieces of 1 to 5 KB: each unit that holds payload lies whole inside its piece's descriptor and the packet."""
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_01989_amd", "csrc"), "-o", str(exe), str(src)])
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
