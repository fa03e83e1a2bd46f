// Where the gather reads a packet: plain integer rules, without device code.
#ifndef DBLP_PACKET_UNITS_H
#define DBLP_PACKET_UNITS_H

#include <stdint.h>

// A packet is read in 16-byte units, one per lane, cut into pieces of whole KB: a piece starts `skip` bytes into
// the units.  Each worker's piece is read through a buffer descriptor that starts unit_base() bytes into the
// packet and is unit_have() bytes long; what lies outside reads as zeros.  Units count from the packet's start
// (LEAD 2: the header takes two floats of unit 0; the last unit may hold padding) or from the payload's
// (LEAD 0: a last unit of fewer than four floats is read as the 16 bytes that end with the payload and turned
// into place when it is stored; those bytes may begin before the piece does, so the descriptor starts with the
// packet and `skip` is part of the offset).

// Bytes from the packet's start to the end of what is read of a payload of `len` floats.
template <uint32_t LEAD>
constexpr uint32_t unit_end(uint32_t len) { return LEAD ? ((len + 2 + 3) >> 2) * 16 : len > 2 ? 8 + 4 * len : 16; }

template <uint32_t LEAD>
constexpr uint32_t unit_base(uint32_t skip) { return LEAD ? skip : 0; }

template <uint32_t LEAD>
constexpr uint32_t unit_have(uint32_t len, uint32_t skip) {
    return unit_end<LEAD>(len) > unit_base<LEAD>(skip) ? unit_end<LEAD>(len) - unit_base<LEAD>(skip) : 0;
}

// Offset in the descriptor of the piece's l-th unit.
template <uint32_t LEAD>
constexpr int unit_offset(uint32_t len, uint32_t skip, uint32_t l) {
    return LEAD ? (int)(16 * l) : (len & 3u) && skip / 16 + l == len >> 2 ? (int)(unit_end<LEAD>(len) - 16) : (int)(skip + 16 * l + 8);
}

#endif
