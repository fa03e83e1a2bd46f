// A sum of doubles that is the same in whatever order they are added: a long accumulator (U. Kulisch), a fixed-point
// number wide enough for all of them.  Without device code.
#ifndef DBLP_LONG_SUM_H
#define DBLP_LONG_SUM_H

#include <stdint.h>

// LONG_WORDS integers of 64 bits, word i in units of 2^(32 i - LONG_SHIFT).  A double adds its 53 bits to three neighbours, 32
// bits to each, so that a word takes 2^31 of them before it could overflow.  The doubles here are sums of squares of floats: multiples of
// 2^-298 below 2^272 (65535 squares of the largest float), whose last bits weigh 2^-350 at least and 2^219 at most.
#define LONG_WORDS 20
#define LONG_SHIFT 352

// Of the double with these bits: position of its last bit above the accumulator's.
constexpr uint32_t long_at(uint64_t bits) { return (uint32_t)(bits >> 52 & 0x7FFu) - (1075u - LONG_SHIFT); }
// Whether it can be added (zero, infinities and NaN cannot).
constexpr bool long_fits(uint64_t bits) { return long_at(bits) < 32u * (LONG_WORDS - 2); }
// What it adds to word i.
constexpr uint64_t long_word(uint64_t bits, uint32_t i) {
    const uint64_t m = (bits & 0xFFFFFFFFFFFFFull) | 0x10000000000000ull;
    const uint32_t s = long_at(bits) & 31u, k = i - (long_at(bits) >> 5);
    const uint64_t part = k == 0 ? (uint32_t)(m << s) : k == 1 ? (uint32_t)(m >> (32 - s)) : k == 2 ? (uint32_t)((m >> 32) >> (32 - s)) : 0u;
    return bits >> 63 ? 0 - part : part;
}

#endif
