"""Where the gather reads a packet and how it shares a range out (packet_units.h), compiled for the host and walked."""
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

TURNS = r"""
#include <initializer_list>
#include "packet_units.h"
#include <stdio.h>
// The groups of all turns and blocks, in that order, cover the range once and in order, are no longer than r_max and
// start on steps; a block without a group has none in later turns; no block is given more steps than needed.
static int check(uint32_t n_seq, uint32_t blocks, uint32_t r_max, uint32_t step) {
    const BurstTurns s(n_seq, blocks, r_max, step);
    uint64_t at = 0, given = 0;
    for (uint32_t k = 0; k < s.turns; ++k) {
        if (s.size(k) == 0 || s.size(k) > r_max || s.size(k) % step) return 1;
        given += s.size(k);
        for (uint32_t b = 0; b < blocks; ++b) {
            const uint32_t f = s.first(k, b);
            if (f == n_seq) { if (at < n_seq || s.first(k + 1, b) != n_seq) return 1; continue; }
            if (f != at || f % step) return 1;
            at += s.size(k);
        }
    }
    for (uint32_t b = 0; b < blocks; ++b) if (s.first(s.turns, b) != n_seq) return 1;
    const uint64_t row = (uint64_t)step * blocks;
    return at < n_seq || given != ((uint64_t)n_seq + row - 1) / row * step || s.turns != (given + r_max - 1) / r_max;
}
int main() {
    for (uint32_t step : {1u, 8u})
        for (uint32_t blocks : {1u, 3u, 256u})
            for (uint32_t m = 1; m <= 32; m = m * 3 / 2 + 1)
                for (uint32_t n = 1; n < 200000; n = n < 300 ? n + 1 : n * 9 / 8 + n % 7)
                    if (check(n, blocks, m * step, step)) { fprintf(stderr, "n %u blocks %u r_max %u step %u\n", n, blocks, m * step, step); return 1; }
    for (uint32_t n : {0xFFFFFFFEu, 0xFFFFFF00u, 0x80000001u}) {        // as large as a round can be: the ends only
        const BurstTurns s(n, 256, 256, 8);
        if (s.first(0, 0) != 0 || s.first(s.turns, 0) != n || s.first(s.turns - 1, 0) >= n) return 1;
    }
    // Rounds up to the largest, batches that end before the round does: a group's numbers stay inside the round, so
    // that the last of them fits 32 bits, and but for the round's end a group is whole steps.
    for (uint32_t pkts : {0xFFFFFFFEu, 0xFFFFFF01u, 0xFFFFFF00u, 70000u, 70001u, 9u})
        for (uint32_t step : {1u, 8u})
            for (uint32_t lo : {0u, pkts / 16 * 8})
                for (uint32_t short_of : {0u, 1u, 5u, 8u}) {
                    const uint32_t n = pkts - lo - (short_of < pkts - lo ? short_of : 0u);
                    const BurstTurns s(n, 256, 32 * step, step);
                    for (uint32_t k = s.turns < 3 ? 0 : s.turns - 3; k < s.turns; ++k)
                        for (uint32_t b = 0; b < 256; ++b) {
                            const uint32_t at = s.first(k, b);
                            if (at >= n) continue;
                            const uint32_t seq0 = lo + at, c = s.count(k, pkts - seq0);
                            if (c == 0 || c > s.size(k) || (uint64_t)seq0 + c > pkts || (c != s.size(k) && (uint64_t)seq0 + c != pkts)) {
                                fprintf(stderr, "round of %u from %u on, %u numbers: group at %u holds %u\n", pkts, lo, n, seq0, c);
                                return 1;
                            }
                        }
                }
    return 0;
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


def test_groups_of_a_burst_cover_the_range_once(tmp_path):
    """Ranges of 1 to 200 k sequence numbers over 1, 3 and 256 blocks, groups of 1 to 256; the ends of the largest rounds."""
    src, exe = tmp_path / "turns.cpp", tmp_path / "turns"
    src.write_text(TURNS)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_01989_amd", "csrc"), "-o", str(exe), str(src)])
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
