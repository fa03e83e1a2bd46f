// Where the gather reads a packet, and which packets a block of the gather in bursts takes: plain integer rules,
// without device code.
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

// A range of n_seq sequence numbers, shared out over n_blocks blocks in turns: in each turn every block takes one
// group of consecutive numbers, of at most r_max (a multiple of r_step, the smallest group).  As few turns as r_max
// allows, and every block is given the same number of steps, over its groups as evenly as whole steps go: the
// first n_long turns have groups of r_long, the others one step less.
struct BurstTurns {
    uint32_t n_seq, n_blocks, r_step, turns, r_long, n_long;
    constexpr BurstTurns(uint32_t n_seq_, uint32_t n_blocks_, uint32_t r_max, uint32_t r_step_)
        : n_seq(n_seq_), n_blocks(n_blocks_), r_step(r_step_), turns(0), r_long(0), n_long(0) {
        const uint32_t row = r_step * n_blocks, steps = (uint32_t)(((uint64_t)n_seq + row - 1) / row), most = r_max / r_step;
        turns = (steps + most - 1) / most;
        const uint32_t a = (steps + turns - 1) / turns;
        r_long = a * r_step;
        n_long = steps - turns * (a - 1);
    }
    constexpr uint32_t size(uint32_t turn) const { return turn < n_long ? r_long : r_long - r_step; }
    // Numbers of a group that exist where `left` of the round are left from its first on: the last group may reach
    // past the round, where a number need not fit 32 bits.  (Past the range it stays whole: a group owns whole bytes of
    // the bitmap.)
    constexpr uint32_t count(uint32_t turn, uint32_t left) const { return left < size(turn) ? left : size(turn); }
    // First number of the block's group in that turn; none (n_seq): the block has no more.
    constexpr uint32_t first(uint32_t turn, uint32_t block) const {
        const uint64_t before = (uint64_t)turn * r_long - (turn > n_long ? (uint64_t)(turn - n_long) * r_step : 0u);
        const uint64_t at = before * n_blocks + (uint64_t)block * size(turn);
        return turn < turns && at < n_seq ? (uint32_t)at : n_seq;
    }
};

// Whether a batch of `cand` packets in a range of n_seq sequence numbers has enough of them per number for bursts.  Each
// turn of a burst has a part that does not overlap with its loads, and a step has room for several workers' pieces:
// where few workers delivered a packet, neither is made up for by the stores.  So many packets per number: 3.2 where the
// blocks take up to six turns; where they take more, 1 for packets in pieces, 1.9 for those of one KB (`kb`), 1.6 for
// the others; and where there are few workers, four in five of them.  us of a pass, gather_stream and bursts, by the
// share of the packets that arrived in one batch over the round: 2 workers x 150 M elements in 1472-byte packets (15 turns)
// half 297, 387, 0.6 330, 365, 0.8 384, 351; 8 x 124 M (13) 0.13 311, 353, 0.2 361, 361, a quarter 399, 369; 8 x 60 M in 528-byte ones (7)
// 0.13 308, 392, 0.2 342, 364, a quarter 365, 345; 8 x 25.6 M (3) 0.2 80, 93, a third 100, 103, half 131, 128; 16 x 34 M (4) 0.13 116,
// 128, a quarter 166, 166, half 287, 267; 5 x 60 M in 2816-byte ones (6) half 171, 184, 0.8 244, 245, all 294, 283; 16 x 100 M in
// 4112-byte ones (12) 0.13 282, 261; 8 x 124 M in 8992-byte ones (13) 0.13 201, 200, 0.16 245, 225.
constexpr bool burst_pays(uint64_t cand, uint64_t n_seq, uint32_t n_workers, uint32_t n_blocks, uint32_t r_max, uint32_t kb) {
    uint32_t tenths = n_seq <= 6ull * r_max * n_blocks ? 32 : kb > 4 ? 10 : kb == 1 ? 19 : 16;
    if (tenths > 8 * n_workers) tenths = 8 * n_workers;
    return cand * 10 >= n_seq * tenths;
}

#endif
