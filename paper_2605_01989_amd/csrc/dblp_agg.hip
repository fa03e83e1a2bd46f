// Receiver-side bounded-loss gradient aggregation of DBLP on gfx950 (MI355X).
// Kernels and the C-ABI declared in include/dblp_agg.h.
//
// Data flow of one arrival batch (Alg. "DBLP_RECV", chunk-arrival branch):
//   index_arrivals   one thread per arrival: header parse, validation, and an atomicMin of
//                    (arrival rank << 32 | slot) into the arrival index `pending[w][seq]`, so the
//                    earliest copy of a packet in the batch wins; per-block tallies (stale, invalid,
//                    candidates, touched seq range) that every gather block adds up for itself
//   gather_stream (dense batches, or both kinds and the blocks decide)
//                    organised by OUTPUT packet: a block takes a group of consecutive sequence
//                    numbers, reads the index entries of all workers, drops copies of packets
//                    that an earlier batch delivered, sets the bitmap bits, then streams the
//                    payloads of each packet from every delivering worker (16-byte loads,
//                    worker order) into registers and writes the accumulator span once.
//   gather_burst     the same for large dense batches of two workers and more, with the spans of many packets stored together.
//   gather_list      batches of few packets, from a list that the index pass makes of them (gather_few, which gather_stream
//                    uses too where its blocks find that a larger batch of few packets is sparse).
// Every payload byte is read exactly once and the accumulator is written once per batch that
// touches it; there are no floating-point atomics, so the sum is independent of the arrival
// permutation.  The accumulator may exist in two copies placed in different thirds of the HBM
// address space (classify_rw measures which copy a packet buffer should be paired with); a
// per-packet byte map records where each span lives.
//
// The probe (Sec. "Dynamically Changing Loss Tolerance"): probe_all for short rounds (prefix sums of the bitmap in LDS), probe_once
// (popcount of bitmap words + DPP wave reduction, list lengths that the blocks tell each other, ordered compaction), or loss_count
// and emit_retx where blocks are many.  The mean of Alg. "Server" is formed as the payloads are summed when
// W is a power of two (the division is exact), and the gather kernels keep the sum of squares of
// what they store, so finalize_pass only writes zeros where nothing arrived (and moves or copies
// spans where the result is wanted elsewhere); for other W it divides and squares itself.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <time.h>

#include <new>
#include <vector>

#include "../../include/dblp_agg.h"
#include "packet_units.h"
#include "long_sum.h"

typedef unsigned long long u64;
typedef uint32_t u32;

#define NONE64 0xFFFFFFFFFFFFFFFFull
#define WAVE 64

// device counters (u64 each)
enum { C_ACCEPTED = 0, C_STALE, C_INVALID, C_CANDIDATES, C_COUNT };
#define M_PROBE_GAVE_UP 2        // word of the host mailbox: a block of probe_once has waited long enough

struct Geo {
    const u32* first_seq;   // [B+1]
    const u64* b_off;       // [B]
    const u64* b_cnt;       // [B]
    const u32* hint;        // bucket of sequence number 64 i, [ceil(n_pkts / 64) + 1]; null where first_seq fits LDS
    u32 B, P, W;
    u32 n_pkts;
    u32 stride;             // bytes
    u32 units;              // stride / 16
    u64 words_pw;           // bitmap words per worker
};

// ------------------------------------------------------------------------------------------
// wave-level primitives (64 lanes): DPP moves, reductions and scans
// ------------------------------------------------------------------------------------------
#define DPP_ROW_SHR(n) (0x110 + (n))
#define DPP_ROW_BCAST15 0x142
#define DPP_ROW_BCAST31 0x143

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ u32 dpp_u32(u32 identity, u32 v) {
    return (u32)__builtin_amdgcn_update_dpp((int)identity, (int)v, CTRL, ROW_MASK, 0xF, false);
}

struct OpAdd { static __device__ __forceinline__ u32 id() { return 0u; } static __device__ __forceinline__ u32 f(u32 a, u32 b) { return a + b; } };
struct OpMin { static __device__ __forceinline__ u32 id() { return 0xFFFFFFFFu; } static __device__ __forceinline__ u32 f(u32 a, u32 b) { return a < b ? a : b; } };
struct OpMax { static __device__ __forceinline__ u32 id() { return 0u; } static __device__ __forceinline__ u32 f(u32 a, u32 b) { return a > b ? a : b; } };
struct OpOr { static __device__ __forceinline__ u32 id() { return 0u; } static __device__ __forceinline__ u32 f(u32 a, u32 b) { return a | b; } };

// Inclusive scan over the 64 lanes; all lanes must be active.  Lane 63 ends with the total.
template <class Op>
__device__ __forceinline__ u32 wave_scan_incl(u32 v) {
    v = Op::f(v, dpp_u32<DPP_ROW_SHR(1), 0xF>(Op::id(), v));
    v = Op::f(v, dpp_u32<DPP_ROW_SHR(2), 0xF>(Op::id(), v));
    v = Op::f(v, dpp_u32<DPP_ROW_SHR(4), 0xF>(Op::id(), v));
    v = Op::f(v, dpp_u32<DPP_ROW_SHR(8), 0xF>(Op::id(), v));
    v = Op::f(v, dpp_u32<DPP_ROW_BCAST15, 0xA>(Op::id(), v));
    v = Op::f(v, dpp_u32<DPP_ROW_BCAST31, 0xC>(Op::id(), v));
    return v;
}

template <class Op>
__device__ __forceinline__ u32 wave_reduce(u32 v) {
    return (u32)__builtin_amdgcn_readlane((int)wave_scan_incl<Op>(v), 63);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double v) {
    u64 bits = (u64)__double_as_longlong(v);
    u32 lo = dpp_u32<CTRL, ROW_MASK>(0u, (u32)bits);
    u32 hi = dpp_u32<CTRL, ROW_MASK>(0u, (u32)(bits >> 32));
    return __longlong_as_double((long long)(((u64)hi << 32) | lo));   // identity 0.0 = all-zero bits
}

// Sum of a double over the 64 lanes (all active); every lane gets the total.
__device__ __forceinline__ double wave_sum_f64(double v) {
    v += dpp_f64<DPP_ROW_SHR(1), 0xF>(v);
    v += dpp_f64<DPP_ROW_SHR(2), 0xF>(v);
    v += dpp_f64<DPP_ROW_SHR(4), 0xF>(v);
    v += dpp_f64<DPP_ROW_SHR(8), 0xF>(v);
    v += dpp_f64<DPP_ROW_BCAST15, 0xA>(v);
    v += dpp_f64<DPP_ROW_BCAST31, 0xC>(v);
    u64 bits = (u64)__double_as_longlong(v);
    u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)bits, 63);
    u32 hi = (u32)__builtin_amdgcn_readlane((int)(u32)(bits >> 32), 63);
    return __longlong_as_double((long long)(((u64)hi << 32) | lo));
}

typedef float f4v __attribute__((ext_vector_type(4)));

// 16-byte store with the non-temporal hint (the sender's packets are not read again by the sender).
typedef u32 u4v __attribute__((ext_vector_type(4)));
typedef u4v u4v_a4 __attribute__((aligned(4)));      // a 16-byte access at a 4-byte aligned address
__device__ __forceinline__ void st_stream4(uint4* p, uint4 v) {
    const u4v t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, (u4v*)p);
}

__device__ __forceinline__ u32 uniform(u32 v) { return (u32)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ u64 uniform(u64 v) { return ((u64)uniform((u32)(v >> 32)) << 32) | uniform((u32)v); }

__device__ __forceinline__ u32 lane_id() { return threadIdx.x & (WAVE - 1); }

// ------------------------------------------------------------------------------------------
// geometry helpers
// ------------------------------------------------------------------------------------------
// Largest b with first_seq[b] <= seq (seq < n_pkts); fs is first_seq or its copy in LDS.  A table that does not
// fit LDS is searched between two entries of the hint table, which stays in the caches (4 bytes per 64
// packets): the whole search is a chain of 13 and more loads from L2 (index pass over 7.7 M arrivals of
// 120 k buckets 538 -> 436 us).
__device__ __forceinline__ u32 find_bucket(const Geo& g, const u32* __restrict__ fs, u32 seq) {
    u32 lo = 0, hi = g.B;
    if (g.hint) { lo = g.hint[seq >> 6]; hi = g.hint[(seq >> 6) + 1] + 1; }
    while (hi - lo > 1) {
        u32 mid = (lo + hi) >> 1;
        if (fs[mid] <= seq) lo = mid; else hi = mid;
    }
    return lo;
}

// First element and float count of packet `seq`, which lies in bucket b.
__device__ __forceinline__ void packet_span(const Geo& g, u32 seq, u32 b, u64* elem, u32* len) {
    u64 start = (u64)(seq - g.first_seq[b]) * g.P;
    u64 left = g.b_cnt[b] - start;
    *elem = g.b_off[b] + start;
    *len = left < g.P ? (u32)left : g.P;
}

#define ACCEPT_ROWS 8192   // >= blocks of any gather launch (n_cus * blocks per CU)
// Long accumulators that a list's gather shares out over its blocks, up to 1024: atomics on one word take turns, about 12 ns each.
#define LONG_COPIES 32u
#define LONG_PITCH 32u
#define LONG_ALL (LONG_COPIES * LONG_PITCH)

// ------------------------------------------------------------------------------------------
// small utility kernels
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void fill_u64(u64* __restrict__ p, u64 n, u64 v) {
    u64 stride = (u64)gridDim.x * blockDim.x;
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// What a round counts in: the long accumulators (LONG_ALL words) and right behind them the delivery bitmap, the gather kernels'
// per-block rows (accepted packets, sums of squares: [ACCEPT_ROWS] each, in one piece), the counters.  A context keeps two of
// them.  The finalize of a round clears the one that is not in use while it is about it, and the next begin_round changes
// over to that and launches nothing.  A launch cost the host 2.6 us before it could make the next, and small rounds are chains
// of launches and waits (us of a pass: 4 x 1 M elements in 1040-byte packets 45.1, 43.3; 3 x 5.3 M 102.0, 98.6; 1 x 25.6 M
// 111.2, 108.6).
struct RoundState { u64* bitmap; u64* rows; u64* counters; u32 rows_used, listed; };    // rows_used: of the rows, those that may not be zero; listed: whether a list was gathered

// Start of a round where no finalize has cleared the other state, in one launch: all of it to zero.  words: accumulators and bitmap.
__global__ __launch_bounds__(256) void reset_round(u64* __restrict__ words, u64 n_words, u64* __restrict__ rows, u64 n_rows,
                                                   u64* __restrict__ counters) {
    const u64 stride = (u64)gridDim.x * blockDim.x;
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n_words + n_rows; i += stride) {
        if (i < n_words) words[i] = 0; else rows[i - n_words] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x < C_COUNT) counters[threadIdx.x] = 0;
}

// counters[C_ACCEPTED] = sum of the per-block rows written by the gather kernels.  One block.
__global__ __launch_bounds__(256) void fold_accept_rows(const u64* __restrict__ rows, u32 n, u64* __restrict__ counters) {
    __shared__ u64 sh[256];
    u64 a[8] = {0, 0, 0, 0, 0, 0, 0, 0};          // eight loads in flight per thread
    for (u32 i = threadIdx.x; i < n; i += 256 * 8) {
        #pragma unroll
        for (u32 j = 0; j < 8; ++j) {
            const u32 k = i + j * 256;
            a[j] += k < n ? rows[k] : 0;
        }
    }
    sh[threadIdx.x] = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    __syncthreads();
    for (u32 d = 128; d > 0; d >>= 1) {
        if (threadIdx.x < d) sh[threadIdx.x] += sh[threadIdx.x + d];
        __syncthreads();
    }
    if (threadIdx.x == 0) counters[C_ACCEPTED] = sh[0];
}

// ------------------------------------------------------------------------------------------
// sender: gradient -> wire packets
// ------------------------------------------------------------------------------------------
// One wave writes one packet (write_packet; short ones several at once, write_packets below): lane l builds 16-byte units l, l + 64, ... (header in the first 8
// bytes of unit 0, zero padding after the payload) and stores them aligned.  A unit inside the payload is
// one 16-byte load at the gradient's own (4-byte) alignment (two 8-byte loads where it was even and four
// single ones elsewhere: 25.6 M elements, 205 MB moved, ten sets of buffers in turn 48.3 -> 45.8 us, one set 37.8 ->
// 37.7; a list of 56 k packets 63.3 -> 57.0 and 48.6 -> 45.8); the first and the last unit go float by float.  All loads of a packet are issued before the
// first store; the stores carry the non-temporal hint (+11 %), the loads do not (with it: -8 %, neighbouring
// units share lines).  PK_UNITS = units per lane kept in registers (packets of up to PK_UNITS KB go in
// one pass, longer ones in several).
#define PK_UNITS 5
__device__ __forceinline__ void write_packet(const float* __restrict__ src, u32 len, u32 seq, u32 round, u32 units,
                                             uint4* __restrict__ dst, u32 lane) {
    const u32 hdr1 = (round & 0xFFFFu) | (len << 16);
    for (u32 u0 = 0; u0 < units; u0 += PK_UNITS * WAVE) {
        uint4 q[PK_UNITS];
        #pragma unroll
        for (int k = 0; k < PK_UNITS; ++k) {
            const u32 u = u0 + k * WAVE + lane;            // packet float positions 4u .. 4u+3 = payload floats 4u-2 .. 4u+1
            q[k] = make_uint4(0u, 0u, 0u, 0u);
            if (u >= units) continue;
            const u32 p0 = 4 * u;
            if (p0 >= 2 && p0 + 1 < len) {
                const u4v_a4 t = *(const u4v_a4*)(src + (p0 - 2));
                q[k] = make_uint4(t.x, t.y, t.z, t.w);
            } else {
                if (p0 >= 2 && p0 - 2 < len) q[k].x = __float_as_uint(src[p0 - 2]);
                if (p0 >= 2 && p0 - 1 < len) q[k].y = __float_as_uint(src[p0 - 1]);
                if (p0 < len) q[k].z = __float_as_uint(src[p0]);
                if (p0 + 1 < len) q[k].w = __float_as_uint(src[p0 + 1]);
            }
            if (u == 0) { q[k].x = seq; q[k].y = hdr1; }
        }
        #pragma unroll
        for (int k = 0; k < PK_UNITS; ++k) {
            const u32 u = u0 + k * WAVE + lane;
            if (u < units) st_stream4(dst + u, q[k]);
        }
    }
}

// Several short packets by one wave, whose units lie one after the other over its lanes: lane j < n_k holds packet j (dst null: it is
// skipped), and a unit's lane asks that one for what it needs.  A wave for each packet leaves lanes of its last pass empty, has few
// bytes in flight where packets are short, and searches the bucket once per packet where here up to 64 lanes search at the same time.
// 60 M elements, 161 buckets, slots in order and by a map (us, a wave for each packet -> several):
//   payload of 14 floats 1148 -> 103, 1304 -> 239; 64: 314 -> 100, 380 -> 186; 126: 174 -> 91, 212 -> 116; 254: 96.9 -> 91.2, 125 -> 113;
//   300: 117 -> 95.4, 142 -> 120; 366: 94.2 -> 87.8, 119 -> 114; 430: 89.1 -> 88.6, 115 -> 113; 500: 91.7 -> 89.3, 118 -> 118;
//   lists of 3 % of eight workers' packets 126: 60.8 -> 41.8, 366: 42.1 -> 40.1, 500: 40.1 -> 39.2.
// 4 passes of 64 units: with 5 most of this was 30 % slower (payload 64 132 us, 254 116), with 2 and 3 packets of 300 to 500 floats
// fill the passes worse (300: 124 and 97.9, 500: 92.1 and 93.3).  Packets of which two don't fit go one by one.
#define SENDER_PASSES 4
struct SentPacket { const float* src; u32 len, seq; uint8_t* dst; };
struct SenderSplit { u32 k, inv; };              // packets per wave (0: one, by write_packet); unit f of a wave belongs to its packet f * inv >> 16 (exact for f < 256)
__device__ __forceinline__ u64 lane_value(u64 v, u32 from) { return ((u64)(u32)__shfl((int)(u32)(v >> 32), (int)from) << 32) | (u32)__shfl((int)(u32)v, (int)from); }
__device__ __forceinline__ void write_packets(const SentPacket& mine, u32 n_k, u32 inv, u32 round, u32 units, u32 lane) {
    uint4 q[SENDER_PASSES];
    uint4* out[SENDER_PASSES];
    const u32 all = n_k * units;
    #pragma unroll
    for (int p = 0; p < SENDER_PASSES; ++p) {
        out[p] = nullptr;
        q[p] = make_uint4(0u, 0u, 0u, 0u);
        if (p * WAVE >= all) continue;                      // the same in all lanes
        const u32 f = p * WAVE + lane, j = f < all ? f * inv >> 16 : 0u, u = f - j * units;
        const float* const src = (const float*)lane_value((u64)mine.src, j);
        uint8_t* const dst = (uint8_t*)lane_value((u64)mine.dst, j);
        const u32 len = (u32)__shfl((int)mine.len, (int)j), seq = (u32)__shfl((int)mine.seq, (int)j);
        if (f >= all || !dst) continue;
        out[p] = (uint4*)dst + u;
        const u32 p0 = 4 * u;
        if (p0 >= 2 && p0 + 1 < len) {
            const u4v_a4 t = *(const u4v_a4*)(src + (p0 - 2));
            q[p] = make_uint4(t.x, t.y, t.z, t.w);
        } else {
            if (p0 >= 2 && p0 - 2 < len) q[p].x = __float_as_uint(src[p0 - 2]);
            if (p0 >= 2 && p0 - 1 < len) q[p].y = __float_as_uint(src[p0 - 1]);
            if (p0 < len) q[p].z = __float_as_uint(src[p0]);
            if (p0 + 1 < len) q[p].w = __float_as_uint(src[p0 + 1]);
        }
        if (u == 0) { q[p].x = seq; q[p].y = (round & 0xFFFFu) | (len << 16); }
    }
    #pragma unroll
    for (int p = 0; p < SENDER_PASSES; ++p)
        if (out[p]) st_stream4(out[p], q[p]);
}

// *bad (host memory, mapped) becomes 1 when an entry has to be skipped: the host reads it after the wait it
// needs anyway, where a counter in device memory cost a copy back (10 us of a 77 us retransmission).
//
// Sender, a range of sequence numbers of one worker: packet first_seq + i -> slot slot_map[i] (or
// slot_base + i).  The bucket boundaries are searched in LDS when the table fits (TABLE_IN_LDS).
template <bool TABLE_IN_LDS, bool SHORT>
__global__ __launch_bounds__(256) void packetize_kernel(Geo g, SenderSplit split, u32 w, u32 round, const float* __restrict__ grad,
                                                        u64 elem_base, u32 first_seq, u32 n, const u32* __restrict__ slot_map,
                                                        u64 slot_base, u64 n_slots, uint8_t* __restrict__ packets,
                                                        uint16_t* __restrict__ src_worker, u64* __restrict__ bad) {
    extern __shared__ u32 fs_lds[];
    const u32* fs = g.first_seq;
    if (TABLE_IN_LDS) {
        for (u32 i = threadIdx.x; i <= g.B; i += blockDim.x) fs_lds[i] = g.first_seq[i];
        __syncthreads();
        fs = fs_lds;
    }
    u32 lane = lane_id();
    u32 wave = (blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
    u32 n_waves = gridDim.x * blockDim.x / WAVE;
    if (SHORT) {
        const u32 k = split.k;
        for (u64 i0 = (u64)wave * k; i0 < n; i0 += (u64)n_waves * k) {
            const u32 n_k = n - i0 < k ? (u32)(n - i0) : k;
            SentPacket mine = {nullptr, 0, 0, nullptr};
            if (lane < n_k) {
                const u32 seq = first_seq + (u32)i0 + lane;
                const u64 slot = slot_map ? (u64)slot_map[i0 + lane] : slot_base + i0 + lane;
                if (slot >= n_slots) *bad = 1;
                else {
                    const u32 b = find_bucket(g, fs, seq);
                    const u64 start = (u64)(seq - fs[b]) * g.P, left = g.b_cnt[b] - start;
                    mine.src = grad + (g.b_off[b] + start - elem_base);
                    mine.len = left < g.P ? (u32)left : g.P;
                    mine.seq = seq;
                    mine.dst = packets + slot * g.stride;
                    src_worker[slot] = (uint16_t)w;
                }
            }
            write_packets(mine, n_k, split.inv, round, g.units, lane);
        }
        return;
    }
    for (u32 i = wave; i < n; i += n_waves) {
        u32 seq = first_seq + i;
        u64 slot = slot_map ? (u64)slot_map[i] : slot_base + i;
        if (slot >= n_slots) {
            if (lane == 0) *bad = 1;
            continue;
        }
        u32 b = find_bucket(g, fs, seq);
        const u64 start = (u64)(seq - fs[b]) * g.P;
        const u64 left = g.b_cnt[b] - start;
        const u64 elem = g.b_off[b] + start;
        const u32 len = left < g.P ? (u32)left : g.P;
        write_packet(grad + (elem - elem_base), len, seq, round, g.units, (uint4*)(packets + slot * g.stride), lane);
        if (lane == 0) src_worker[slot] = (uint16_t)w;
    }
}

struct GradPtrs { const float* p[DBLP_MAX_WORKERS]; };

// List entry i (w << 32 | seq): worker w's packet seq -> slot slot_base + i.  A wave takes one entry, or several at once (SHORT).
template <bool TABLE_IN_LDS, bool SHORT>
__global__ __launch_bounds__(256) void packetize_list_kernel(Geo g, SenderSplit split, GradPtrs grads, u32 round, const u64* __restrict__ list,
                                                             u64 n, u64 slot_base, uint8_t* __restrict__ packets,
                                                             uint16_t* __restrict__ src_worker, u64* __restrict__ bad) {
    extern __shared__ u32 fs_lds[];
    const u32* fs = g.first_seq;
    if (TABLE_IN_LDS) {
        for (u32 i = threadIdx.x; i <= g.B; i += blockDim.x) fs_lds[i] = g.first_seq[i];
        __syncthreads();
        fs = fs_lds;
    }
    const u32 lane = lane_id();
    const u64 wave = ((u64)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
    const u64 n_waves = (u64)gridDim.x * blockDim.x / WAVE;
    if (SHORT) {
        const u32 k = split.k;
        for (u64 i0 = wave * k; i0 < n; i0 += n_waves * k) {
            const u32 n_k = n - i0 < k ? (u32)(n - i0) : k;
            SentPacket mine = {nullptr, 0, 0, nullptr};
            if (lane < n_k) {
                const u64 e = list[i0 + lane], slot = slot_base + i0 + lane;
                const u32 w = (u32)(e >> 32), seq = (u32)e;
                if (w >= g.W || seq >= g.n_pkts) *bad = 1;
                else {
                    const u32 b = find_bucket(g, fs, seq);
                    const u64 start = (u64)(seq - fs[b]) * g.P, left = g.b_cnt[b] - start;
                    mine.src = grads.p[w] + (g.b_off[b] + start);
                    mine.len = left < g.P ? (u32)left : g.P;
                    mine.seq = seq;
                    mine.dst = packets + slot * g.stride;
                    src_worker[slot] = (uint16_t)w;
                }
            }
            write_packets(mine, n_k, split.inv, round, g.units, lane);
        }
        return;
    }
    for (u64 i = wave; i < n; i += n_waves) {
        const u64 e = list[i];
        const u32 w = (u32)(e >> 32), seq = (u32)e;
        if (w >= g.W || seq >= g.n_pkts) {
            if (lane == 0) *bad = 1;
            continue;
        }
        const u32 b = find_bucket(g, fs, seq);
        const u64 start = (u64)(seq - fs[b]) * g.P;
        const u64 left = g.b_cnt[b] - start;
        const u64 elem = g.b_off[b] + start;
        const u32 len = left < g.P ? (u32)left : g.P;
        write_packet(grads.p[w] + elem, len, seq, round, g.units, (uint4*)(packets + (slot_base + i) * g.stride), lane);
        if (lane == 0) src_worker[slot_base + i] = (uint16_t)w;
    }
}

// ------------------------------------------------------------------------------------------
// receiver step 1: index the arrivals
// ------------------------------------------------------------------------------------------
struct ArrivalList {
    u64* entries;           // per arrival: bucket << 32 | sequence number, NONE64 of one that is not valid; null: none is made
    u32* first;             // per sequence number: the batch's first arrival with it; all-ones between batches
    u32 n;
};

// Grid-stride over arrivals.  Per-thread tallies are reduced per wave (DPP) and per block
// (LDS) and written to the block's row of block_tallies; fold_index_tallies adds the rows up.
// No global atomics on shared counters: atomics of many waves (or even of a few thousand
// blocks) on one address serialise in L2 at about 12 ns each.
//
// `few`: the batch is a small one that gather_few will take (below).
//
// TABLE_IN_LDS: the block first copies the bucket boundaries (first_seq, B + 1 words of dynamic
// shared memory) into LDS, so the ten dependent steps of the bucket search stay inside the CU.
// FROM_QUEUE: arrival k is the descriptor queue[k] = slot | worker << 32 (one coalesced 8-byte
// load) instead of order[k], mask bit[slot] and src_worker[slot]; the latter two are random
// accesses, and src_worker[slot] alone costs half as much as the header line it sits beside.
template <bool TABLE_IN_LDS, bool FROM_QUEUE>
__global__ __launch_bounds__(256) void index_arrivals(Geo g, const uint8_t* __restrict__ packets,
                                                      const uint16_t* __restrict__ src_worker, u64 n_slots,
                                                      const u64* __restrict__ mask, const u32* __restrict__ order,
                                                      const u64* __restrict__ queue,
                                                      u64 n_arrivals, u32 cur_round, u64* __restrict__ pending,
                                                      u32* __restrict__ block_tallies, u64* __restrict__ any, ArrivalList few) {
    __shared__ u32 sh[4][5];    // per wave: stale, invalid, candidates, lowest seq, highest seq + 1
    extern __shared__ u32 fs_lds[];
    u32 n_stale = 0, n_inv = 0, n_cand = 0;
    u32 seq_lo = 0xFFFFFFFFu, seq_hi = 0;
    const u64 stride = (u64)gridDim.x * blockDim.x;
    // Arrival k: its slot, worker and header.  live: neither lost nor outside the buffer.
    u64 slot = 0;
    uint2 hdr = make_uint2(0u, 0u);
    u32 w = 0;
    bool live = false;
    auto fetch = [&](u64 k) {
        live = k < n_arrivals;
        if (!live) return;
        if (FROM_QUEUE) {
            const u64 e = queue[k];
            slot = e & 0xFFFFFFFFull;
            w = (u32)(e >> 32);             // bits 48..63 must be zero: w >= W below catches them
        } else slot = order ? (u64)order[k] : k;
        if (slot >= n_slots) { ++n_inv; live = false; return; }
        // lost packets are never looked at
        if (!FROM_QUEUE && mask && !((mask[slot >> 6] >> (slot & 63)) & 1ull)) { live = false; return; }
        hdr = *(const uint2*)(packets + slot * g.stride);
        if (!FROM_QUEUE) w = src_worker[slot];
    };
    // The first arrival is on its way while the table is: a short batch is one chain of loads (4 x 1 M elements in
    // 1040-byte packets 4.0, 3.7 us).
    u64 k = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    fetch(k);
    const u32* fs = g.first_seq;
    if (TABLE_IN_LDS) {
        for (u32 i = threadIdx.x; i <= g.B; i += blockDim.x) fs_lds[i] = g.first_seq[i];
        __syncthreads();
        fs = fs_lds;
    }
    for (; k < n_arrivals; k += stride, fetch(k)) {
        if (few.entries) few.entries[k] = NONE64;
        if (!live) continue;
        const u32 seq = hdr.x, round = hdr.y & 0xFFFFu, len = hdr.y >> 16;
        if (round != cur_round) { ++n_stale; continue; }
        if (w >= g.W || seq >= g.n_pkts) { ++n_inv; continue; }
        const u32 b = find_bucket(g, fs, seq);
        u32 want = g.P;         // every packet of a bucket but its last one is full
        if (seq + 1 == fs[b + 1]) { u64 elem; packet_span(g, seq, b, &elem, &want); }
        if (len != want) { ++n_inv; continue; }
        ++n_cand;
        atomicMin(&pending[(u64)w * g.n_pkts + seq], (k << 32) | slot);
        if (few.entries) {
            few.entries[k] = (u64)b << 32 | seq;
            atomicMin(&few.first[seq], (u32)k);
        }
        seq_lo = seq < seq_lo ? seq : seq_lo;
        seq_hi = seq + 1 > seq_hi ? seq + 1 : seq_hi;
    }
    // loops above have lane-dependent trip counts; all 64 lanes are back here
    n_stale = wave_reduce<OpAdd>(n_stale); n_inv = wave_reduce<OpAdd>(n_inv);
    n_cand = wave_reduce<OpAdd>(n_cand);
    seq_lo = wave_reduce<OpMin>(seq_lo); seq_hi = wave_reduce<OpMax>(seq_hi);
    const u32 wave = threadIdx.x / WAVE;
    if (lane_id() == 0) {
        sh[wave][0] = n_stale; sh[wave][1] = n_inv; sh[wave][2] = n_cand;
        sh[wave][3] = seq_lo; sh[wave][4] = seq_hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        u32 t[3] = {0, 0, 0}, lo = 0xFFFFFFFFu, hi = 0;
        for (int i = 0; i < 4; ++i) {
            for (int j = 0; j < 3; ++j) t[j] += sh[i][j];
            lo = sh[i][3] < lo ? sh[i][3] : lo;
            hi = sh[i][4] > hi ? sh[i][4] : hi;
        }
        u32* row = block_tallies + (u64)blockIdx.x * 5;
        row[0] = t[0]; row[1] = t[1]; row[2] = t[2]; row[3] = lo; row[4] = hi;
        if (any && t[2]) *any = 1;
    }
}

// What the gather kernels need to know about the batch: the touched sequence range and the number
// of candidates.  Every block of a gather launch adds up the index launch's per-block tallies
// itself (n_rows rows of 5 words, read from L2), which saves a launch between the two passes; the
// block that `owner` names also adds the totals to the round's counters (one block of one launch
// per batch).  All threads of the block must call this; sh holds 5 words per wave.
struct BatchInfo { u64 lo, hi, cand; };
__device__ __forceinline__ BatchInfo fold_index_tallies(const u32* __restrict__ block_tallies, u32 n_rows, u64* __restrict__ counters,
                                                        bool owner, u32* sh) {
    u32 t0 = 0, t1 = 0, t2 = 0, lo = 0xFFFFFFFFu, hi = 0;
    for (u32 b = threadIdx.x; b < n_rows; b += blockDim.x) {
        const u32* row = block_tallies + (u64)b * 5;
        t0 += row[0]; t1 += row[1]; t2 += row[2];
        lo = row[3] < lo ? row[3] : lo;
        hi = row[4] > hi ? row[4] : hi;
    }
    t0 = wave_reduce<OpAdd>(t0); t1 = wave_reduce<OpAdd>(t1); t2 = wave_reduce<OpAdd>(t2);
    lo = wave_reduce<OpMin>(lo); hi = wave_reduce<OpMax>(hi);
    const u32 wave = threadIdx.x / WAVE, n_waves = blockDim.x / WAVE;
    if (lane_id() == 0) { sh[wave * 5 + 0] = t0; sh[wave * 5 + 1] = t1; sh[wave * 5 + 2] = t2; sh[wave * 5 + 3] = lo; sh[wave * 5 + 4] = hi; }
    __syncthreads();
    u64 s0 = 0, s1 = 0, s2 = 0;
    u32 l = 0xFFFFFFFFu, h = 0;
    for (u32 i = 0; i < n_waves; ++i) {
        s0 += sh[i * 5 + 0]; s1 += sh[i * 5 + 1]; s2 += sh[i * 5 + 2];
        l = sh[i * 5 + 3] < l ? sh[i * 5 + 3] : l;
        h = sh[i * 5 + 4] > h ? sh[i * 5 + 4] : h;
    }
    __syncthreads();                                // sh may be reused by the caller
    if (owner && threadIdx.x == 0) {
        counters[C_STALE] += s0;
        counters[C_INVALID] += s1;
        counters[C_CANDIDATES] += s2;
    }
    BatchInfo bi;
    bi.cand = s2; bi.lo = s2 ? (u64)l : NONE64; bi.hi = s2 ? (u64)h : 0;
    return bi;
}

// ------------------------------------------------------------------------------------------
// receiver step 2: gather payloads per output packet and accumulate
// ------------------------------------------------------------------------------------------
#define NONE32 0xFFFFFFFFu

// A batch is sparse when it holds fewer than one packet per SPARSE_DIV (worker, seq) pairs of the
// sequence range it touches (retransmission batches), or one packet.  Sparse batches go through gather_stream in a
// way of their own (below); where the host cannot tell, the launch holds both and its blocks decide.
#define SPARSE_DIV 8
enum { TOLD_DENSE = 0, TOLD_SPARSE, TOLD_BURST };       // what a launch that decides on the device tells its trace group
__device__ __forceinline__ bool batch_is_sparse(const BatchInfo& bi, u32 W) {
    return bi.cand == 1 || bi.cand * SPARSE_DIV < (bi.hi - bi.lo) * W;
}

// A block takes a group of `sub` = 16 (8 to 1 in short ranges, 32 in sparse batches, where a single wave may take one)
// consecutive sequence numbers: every wave reads the group's arrival index (64 / sub workers x sub packets per load; of many workers
// its share), ballots which packets are new, and keeps their slots in LDS; after a barrier the first wave resets the index
// entries and sets the bitmap, whose bytes the group owns (8, 16 or 32 bits: a plain store, where one
// memory-side atomic per worker and group took up to a microsecond of a small group's time).  The
// waves then share the group's packets, cut into pieces of NP KB when they are longer than 5 KB.
//
// What bounds it is the memory system, so the loop is there to keep it asked: a step loads G workers'
// pieces of one packet (16 bytes per lane and KB), D steps are in flight in registers, and a packet's
// stores are issued between the loads of later steps.  The loads are the same in every step, without
// branches or masks, so the compiler can wait for exactly the oldest step (s_waitcnt vmcnt counts in
// order): each worker's piece is a buffer descriptor of its own (base and length in scalar registers),
// of length zero for a worker that delivered nothing, and lanes beyond the length read zeros without
// asking memory.  Any packet length goes this way: the sums stay in registers and leave them as
// 16-byte stores at the span's own (4-byte) alignment.
//
// Measured against the kernel it replaces (reader waves, LDS, a writer wave per block; packets above
// 12 KB went to the direct kernel), us per launch, algorithmic TB/s in brackets:
//   8 workers x 8992-byte packets, 4.5 GB       1430 -> 930  (3.1 -> 4.8)
//   16 x 4112 B, 23.8 GB                         4740 -> 4630 (5.0 -> 5.1)
//   8 x 1472 B, 0.92 GB                           194 -> 177  (4.7 -> 5.2)
//   8 x 1472 B, 4.5 GB                            912 -> 892  (4.9 -> 5.0)
//   1 x 1472 B, 0.2 GB (as much written as read)   94 -> 45   (2.2 -> 4.6)
//   4 x 1040 B, 21 MB                              19 -> 12
//
// SPARSE (retransmissions): a step is one worker's 2 KB, two in flight, and the last step of a packet
// loads the span's old contents with it (they were a second trip to memory after the payload's), again
// through a descriptor, of length zero where the span is new.  Most waves have one to three steps, so none
// is empty and little code is run through once (four steps in flight, empty ones among them, and eight
// index rows: 1.5 to 2 us more for a few packets of a round of 4096).  Against a kernel whose waves of a
// block took whole packets one after the other, us per launch:
//   524 k packets of a round of 546 k x 32, 1472 B      722 -> 460
//   14 k of 340 k x 8, 1472 B                            114 -> 46
//   10 of 3740 x 4, 64 KB                                 72 -> 22
//   57 k in three runs of 355 k x 16, 4016 B             345 -> 186
typedef f4v f4v_a4 __attribute__((aligned(4)));      // a 16-byte access at a 4-byte aligned address

#define GS_WAVES 4           // waves per block
// Cache policy of the payload's buffer loads: non-temporal.  The payload is read exactly once and should
// not displace the accumulator and index lines that are being written (measured: 8 % off the payload
// pass).  Headers are NOT loaded this way in the index pass: their lines are read again by the gather.
#define BUF_NT 2
#define BUF_RAW 0x00020000   // word 3 of a raw buffer descriptor: 32-bit data format, no swizzle
#define GS_TEAM_LDS(W, sub_log2) ((((W) + (WAVE >> (sub_log2)) - 1) >> (6 - (sub_log2)) << (6 - (sub_log2))) * ((1u << (sub_log2)) + 1u))

// Orders the LDS accesses of one wave (a wave's LDS operations execute in order; this keeps the
// compiler from moving them across).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double squares(f4v v) {
    return (((double)v.x * (double)v.x + (double)v.y * (double)v.y) + (double)v.z * (double)v.z) + (double)v.w * (double)v.w;
}

// Unit u (16 bytes) of a packet of `len` floats in the grid that LEAD says: which of its floats are payload.
template <u32 LEAD>
struct SpanUnit {
    u32 u, n_tail;              // n_tail: floats of a last unit that is not full
    bool head, full, part;      // head: two header words, then the first two floats
    bool v0, v1, v2, v3;        // floats of a unit that is not full
    bool past_end;
    __device__ __forceinline__ SpanUnit(u32 u_, u32 len) : u(u_) {
        const u32 past = len + LEAD;
        n_tail = past & 3u;
        head = LEAD && u == 0;
        full = !head && 4 * u + 4 <= past;
        part = !head && n_tail && u == past >> 2;
        v0 = part; v1 = part && n_tail > 1; v2 = head ? len > 0 : part && n_tail > 2; v3 = head && len > 1;
        past_end = n_tail && !head && 4 * u + 4 > past;
    }
    // The unit's floats in place, zeros where there is no payload.
    __device__ __forceinline__ f4v take(f4v r, u32 len) const {
        if (head) {
            r.x = r.y = 0.f;
            if (!v3) r.w = 0.f;
        }
        if (past_end) {
            if (LEAD) r = f4v{v0 ? r.x : 0.f, v1 ? r.y : 0.f, v2 ? r.z : 0.f, 0.f};
            else {
                const u32 first = len > 1 ? 4 - n_tail : 2;
                r = f4v{v0 ? (first == 1 ? r.y : first == 2 ? r.z : r.w) : 0.f, v1 ? (first == 1 ? r.z : r.w) : 0.f, v2 ? r.w : 0.f, 0.f};
            }
        }
        return r;
    }
    // What is stored of a unit that is not full.
    __device__ __forceinline__ f4v floats(const float* o) const {
        return f4v{v0 ? o[0] : 0.f, v1 ? o[1] : 0.f, v2 ? o[2] : 0.f, v3 ? o[3] : 0.f};
    }
    template <class T>
    __device__ __forceinline__ void store(T* o, f4v r) const {
        if (full) *(f4v_a4*)o = r;
        else {
            if (v0) o[0] = r.x;
            if (v1) o[1] = r.y;
            if (v2) o[2] = r.z;
            if (v3) o[3] = r.w;
        }
    }
};

// Sequence numbers (log2) that a block of the gather takes at a time, where n of them hold packets: 16; 8 while such
// groups fit the chip at once, three blocks per CU (4 x 1024 B, 4096 packets: 11.7 against 12.6 us; 5600: 12.2 against
// 13.2; 6600: 14.7 against 13.2; far above that groups of 8 pay for the shorter rows of the index: 8 x 1472 B, 340 k
// packets, 920 against 893 us), for packets in pieces only when they are fewer still (64 KB datagrams, 3740 packets:
// 224 us with 16, 232 with 8).  4, 2 or 1 where one sequence number is heavy, whatever gives every CU a group: with 128
// KB or more from all workers (2) below 8 per CU (32 workers, 340 datagrams: 161 us against 650 with 16; 32 x 8992 B,
// 900 packets: 58 against 104), with 64 KB (1) below 4 (8 x 25.6 M elements of 8992 B in 60 steps: 1514 us with 8, 1042
// with 1; 1600 packets at once: 29.6 with 8, 31.0 with 4); light packets are not worth the atomics on the shared bytes
// of the bitmap (3 x 4112 B, 420 packets: 24 us with 1, 12 with 8).
__host__ __device__ static inline u32 group_log2(u64 n, u32 cus, bool pieces, u32 heavy) {
    if (n >= (pieces ? 12u : 24u) * cus) return 4;
    if (heavy == 0 || n >= (heavy == 1 ? 4u : 8u) * cus) return 3;
    return n >= 4u * cus ? 2 : n >= 2u * cus ? 1 : 0;
}

// What a gather launch is given for one regime: sequence numbers per group (log2), pieces per packet, blocks.
struct GatherShape { u32 sub_log2, n_piece, blocks; };

// The gather of one batch by blocks 0 .. s.blocks - 1 of the launch.  fs: the bucket boundaries.
// MANY (more than 16 workers, whose index is several trips to memory, one after the other): the block's waves share a group's
// rows of the index out instead of each reading all of them.  us of index pass and gather, rows read by all and shared
// out: 32 workers x 82 k numbers of 1472 B, 78 k packets late 90, 82, 210 k late 140, 131; 64 x 33 k, 63 k late 72, 62, 168 k late
// 118, 107.  Whole rounds: in blocks of 16 waves 64 x 200 of 2416 B 24.8, 24.0, 33 x 200 of 4096 B 22.4, 21.5, 24 x 150 of 14.8 KB 25.6,
// 24.9; 64 x 300 of 272 B 27.6, 26.2, 64 x 1500 of 4112 B 85.9, 83.3, 64 x 6000 of 1472 B 114.9, 115.0; but 17 x 400 of 4112 B 19.9, 20.8, 32 x 300
// of 8992 B 30.6, 31.4: 0.4 % over 55 shapes, more the more workers.  With fewer workers the waves' waiting for each other is all
// that it gives: 4 x 4096 packets of 1040 B 14.4, 15.8; 16 x 5465, 2.6 k late 17.7, 18.2.
template <int NP, int G, int D, int NW, bool SPARSE, u32 LEAD, bool MANY>
__device__ __forceinline__ void gather_groups(const Geo& g, const BatchInfo& bi, const GatherShape& s, const u32* fs, u32* sh_slots,
                                              const uint8_t* __restrict__ packets, u64* __restrict__ pending, u64* __restrict__ bitmap,
                                              float* acc0, float* acc1, uint8_t* __restrict__ home, u32 pick,
                                              u64* __restrict__ accept_rows, double* __restrict__ sumsq_rows, float inv_w) {
    __shared__ u32 sh_accepted[NW];
    __shared__ double sh_sq[NW];
    __shared__ u32 sh_tile[4];      // sparse: groups of the tile that hold an arrival; groups left to the whole block
    __shared__ u32 sh_any[3][2];    // MANY: of three groups in turn, packets with a new copy; packets with contents
    if (blockIdx.x >= s.blocks) return;
    u32 turn = 0, f = 0;            // MANY: groups that the block has taken together, modulo 2 and 3
    if (MANY) {
        if (threadIdx.x < 6) sh_any[0][threadIdx.x] = 0;
        __syncthreads();
    }
    const u32 lane = lane_id();
    const u32 wave = uniform(threadIdx.x / WAVE);
    const u32 sub_log2 = s.sub_log2, n_piece = s.n_piece, n_blocks = s.blocks;
    const u32 W = g.W, sub = 1u << sub_log2, wpl = WAVE >> sub_log2, pitch = sub + 1;
    const u64 lo = bi.lo, hi = bi.hi;
    const u32 s_lane = lane & (sub - 1), w_sub = lane >> sub_log2;
    const u64 submask = NONE64 >> (WAVE - sub);
    const u32 grp_lo = (u32)__builtin_amdgcn_readfirstlane((int)(u32)(lo >> sub_log2));
    const u32 grp_end = (u32)__builtin_amdgcn_readfirstlane((int)(u32)((hi + sub - 1) >> sub_log2));
    constexpr int J = 4;                            // index loads in flight
    u32 accepted = 0;
    double sq = 0.0;      // change of the sum of squares of the stored values caused by this lane's packets

    // The block's groups (grid-stride), up to 64 at a time.  Where most of them hold no arrival (a small
    // retransmission batch over a long round: fewer than one candidate per 64 sequence numbers), the block
    // first looks through their index entries, eight loads in flight per wave, and then takes the groups
    // that hold one (26 against 46 us for a few packets in a round of 589 k x 8; 15.0 against 16.7 for 56 of
    // 187 k, six groups per block; with fewer than three groups to look through it costs what it saves).
    const bool skim = SPARSE && bi.cand * 64 < hi - lo;
    constexpr u32 TILE = SPARSE ? 64 : 1;
    for (u64 tile = (u64)grp_lo + blockIdx.x; tile < grp_end; tile += (u64)TILE * n_blocks) {
    const u32 tile_left = SPARSE ? (grp_end - (u32)tile + n_blocks - 1) / n_blocks : 1, n_tile = tile_left < TILE ? tile_left : TILE;
    u64 todo = NONE64 >> (64 - n_tile);
    // A sparse batch's groups go to single waves (`solo`), every NW-th to one, unless the average group holds
    // more than solo_max pieces; a wave leaves a group of more than twice that to the whole block, which takes those
    // afterwards.  A group is a chain of about 6 us whatever it holds (index, payload, store), so what counts is
    // how many are in hand.  Against blocks as teams, us: 4 x 1.9 M packets of 136 bytes, 22 k lost 267 -> 90; 8 x
    // 340 k of 1472 B, 14 k lost 102 -> 46; 32 x 340 k, 3 k lost 110 -> 61 and 217 k lost 276 -> 210; 16 x 355 k
    // of 4016 B, 57 k lost in three runs 265 -> 186.  Whole blocks win where groups are full (32 x 540 k, 527 k lost
    // in bursts, 33 a group: 478 against 501), or fewer than the waves (two groups a block, 16 x 60 k of 416 B, 10 a
    // group: 36 against 46), and with packets of three and more pieces (2 x 45 k of 8992 B, 1786 lost: 32 against 40).
    const u32 solo_max = n_piece > 2 ? 0 : n_piece == 2 ? (n_tile > 2 ? 10 : 0) : n_tile > 2 ? 24 : 8;
    const bool look = skim && n_tile >= 3;
    bool solo = SPARSE && n_tile > 1 && (bi.cand << sub_log2) * n_piece <= (hi - lo) * solo_max;
    if (solo || look) {
        __syncthreads();                            // the tile before is done with sh_tile
        if (threadIdx.x < 4) sh_tile[threadIdx.x] = 0;
        __syncthreads();
    }
    if (look) {
        const u32 rows = (W + wpl - 1) >> (6 - sub_log2);
        u32 k = 0, r = wave;                        // group k of the tile, index row r of the group
        u64 found = 0;
        while (k < n_tile) {
            u64 e[8];
            u32 kk[8];
            #pragma unroll
            for (int j = 0; j < 8; ++j) {
                while (r >= rows && k < n_tile) { r -= rows; ++k; }
                const u32 w = (r << (6 - sub_log2)) + w_sub, seq = ((u32)(tile + (u64)k * n_blocks) << sub_log2) + s_lane;
                kk[j] = k;
                e[j] = k < n_tile && w < W && seq < g.n_pkts ? pending[(u64)w * g.n_pkts + seq] : NONE64;
                r += NW;
            }
            #pragma unroll
            for (int j = 0; j < 8; ++j)
                if (__ballot(e[j] != NONE64)) found |= 1ull << kk[j];
        }
        if (lane == 0 && found) { atomicOr(&sh_tile[0], (u32)found); atomicOr(&sh_tile[1], (u32)(found >> 32)); }
        __syncthreads();
        todo = uniform(((u64)sh_tile[1] << 32) | sh_tile[0]);
    }
    if (solo) for (u32 i = 0; i < wave; ++i) todo &= todo - 1;
    for (;;) {
        if (todo == 0) {
            if (!solo) break;
            solo = false;
            __syncthreads();
            todo = uniform(((u64)sh_tile[3] << 32) | sh_tile[2]);
            if (todo == 0) break;
        }
        const u32 at = (u32)__builtin_ctzll(todo);
        const u64 grp = tile + (u64)at * n_blocks;
        for (u32 i = 0; i < (solo ? NW : 1); ++i) todo &= todo - 1;
        const bool leader = solo || wave == 0;
        bool heavy = false;
        // ---- arrival index -> slots of the group's new packets, bitmap bits, spans
        const u32 seq0 = (u32)grp << sub_log2, seq_l = seq0 + s_lane;
        const u32 word = seq0 >> 6, shift = seq0 & 63;
        u64 elem_l = 0, new_any = 0, old_any = 0;
        u32 len_l = 0, home_l = pick;
        const bool split = MANY && !solo;       // a row is read by one wave only
        u32* const slots = sh_slots + (split ? turn : wave) * GS_TEAM_LDS(W, sub_log2);
        const u32 w_step = split ? NW * wpl : wpl, w_first = split ? wave * wpl : 0;
        for (u32 w0 = w_first; w0 < W || (MANY && w0 == w_first); w0 += J * w_step) {
            u64 p[J], bits[J], nb[J];
            #pragma unroll
            for (int j = 0; j < J; ++j) {
                const u32 w = w0 + j * w_step + w_sub;
                p[j] = NONE64; bits[j] = 0;
                if (w < W && seq_l < g.n_pkts) {
                    p[j] = pending[(u64)w * g.n_pkts + seq_l];
                    bits[j] = bitmap[(u64)w * g.words_pw + word];
                }
            }
            if (w0 == w_first && lane < sub && seq_l < g.n_pkts) {
                const u32 b = find_bucket(g, fs, seq_l);
                const u64 start = (u64)(seq_l - fs[b]) * g.P;
                const u64 left = g.b_cnt[b] - start;
                elem_l = g.b_off[b] + start;
                len_l = left < g.P ? (u32)left : g.P;
                home_l = home[seq_l];                       // only meaningful (and only used) for spans written before
            }
            #pragma unroll
            for (int j = 0; j < J; ++j) {
                nb[j] = 0;
                if (w0 + j * w_step >= W) continue;
                const u32 w = w0 + j * w_step + w_sub;
                const bool had = (bits[j] >> (shift + s_lane)) & 1ull;      // delivered by an earlier batch
                const bool fresh = p[j] != NONE64 && !had;                  // a copy of a delivered packet is dropped
                nb[j] = __ballot(fresh);
                slots[w * pitch + s_lane] = fresh ? (u32)p[j] : NONE32;
                u64 n = nb[j], o = __ballot(had);
                new_any |= n; old_any |= o;
                for (u32 k = 1; k < wpl; ++k) { n >>= sub; o >>= sub; new_any |= n; old_any |= o; }
            }
            if (SPARSE && solo) {
                if (w0 == 0) {       // judged by the first J * wpl workers, before an entry of the group is reset
                    u32 n = 0;
                    #pragma unroll
                    for (int j = 0; j < J; ++j) n += (u32)__popcll(nb[j]);
                    heavy = n * n_piece * ((W + J * wpl - 1) / (J * wpl)) > 2 * solo_max;
                    if (heavy) {
                        if (lane == 0) atomicOr(&sh_tile[2 + (at >> 5)], 1u << (at & 31));
                        break;
                    }
                }
            } else if (!split) __syncthreads();     // every wave of the block has read the index before the first one resets it
            if (leader || split) {
                #pragma unroll
                for (int j = 0; j < J; ++j) {
                    const u32 w = w0 + j * w_step + w_sub;
                    if (p[j] != NONE64) pending[(u64)w * g.n_pkts + seq_l] = NONE64;   // leave the index empty
                    const u64 mine = (nb[j] >> (w_sub << sub_log2)) & submask;
                    // a group owns its 1, 2, 4 or 8 bytes of the bitmap: no atomics
                    if (s_lane == 0 && mine) {
                        uint8_t* bp = (uint8_t*)(bitmap + (u64)w * g.words_pw) + (seq0 >> 3);
                        const u64 both = mine | ((bits[j] >> shift) & submask);
                        if (sub_log2 == 4) *(uint16_t*)bp = (uint16_t)both;
                        else if (sub_log2 == 3) *bp = (uint8_t)both;
                        else if (sub_log2 == 5) *(u32*)bp = (u32)both;
                        else atomicOr(&bitmap[(u64)w * g.words_pw + word], mine << shift);   // shorter groups share a byte
                    }
                    accepted += (u32)__popcll(nb[j]);
                }
            }
        }
        new_any = uniform(new_any & submask); old_any = uniform(old_any & submask);
        if (split) {
            if (lane == 0 && new_any) atomicOr(&sh_any[f][0], (u32)new_any);
            if (lane == 0 && old_any) atomicOr(&sh_any[f][1], (u32)old_any);
            __syncthreads();                    // and all waves are done with the group before
            new_any = uniform(sh_any[f][0]); old_any = uniform(sh_any[f][1]);
            const u32 z = f == 0 ? 2 : f - 1;
            if (threadIdx.x < 2) sh_any[z][threadIdx.x] = 0;        // the words of the group before are those of the group after the next
            turn ^= 1; f = f == 2 ? 0 : f + 1;
        }
        if (heavy || new_any == 0) continue;
        if (lane < sub && !((old_any >> lane) & 1u)) {
            home_l = pick;
            if (leader && ((new_any >> lane) & 1u)) home[seq_l] = (uint8_t)pick;
        }
        wave_lds_fence();

        // ---- payloads: items = pieces of NP KB of the group's packets; G workers' pieces make one
        // step, D steps are in flight
        const u32 n_team = solo ? 1 : NW;
        u32 t_gen = 0, piece_gen = 0, t_next = 0, piece_next = solo ? 0 : wave;   // item the generator is at: piece of packet t_gen; (t_next, piece_next) comes after it
        u64 left_gen = 0;               // its workers still to be loaded
        u32 slot32 = NONE32;            // lane w: slot of worker w's copy of packet t_gen
        f4v v[D][G][NP], old[D][NP];    // old: what earlier batches left in the span (SPARSE: loaded with the last step's payloads)
        u32 tag[D];                     // t | piece << 8 | last << 30 | valid << 31
        f4v a[NP];
        #pragma unroll
        for (int q = 0; q < NP; ++q) a[q] = f4v{0.f, 0.f, 0.f, 0.f};

        // the next step's packet, piece and workers; false when the wave has no more
        auto next = [&]() {
            if (left_gen == 0) {
                for (;;) {
                    while (piece_next >= n_piece) { piece_next -= n_piece; ++t_next; }
                    if (t_next >= sub) break;
                    t_gen = t_next; piece_gen = piece_next;
                    piece_next += n_team;
                    if (((new_any >> t_gen) & 1u) && piece_gen * (NP * 256u) < (u32)__builtin_amdgcn_readlane((int)len_l, (int)t_gen) + LEAD) {
                        slot32 = lane < W ? slots[lane * pitch + t_gen] : NONE32;
                        left_gen = uniform((u64)__ballot(slot32 != NONE32));
                        break;
                    }
                }
            }
            return left_gen != 0;
        };
        auto issue = [&](int d) {
            const u32 len = (u32)__builtin_amdgcn_readlane((int)len_l, (int)t_gen);
            const u32 skip = piece_gen * (NP * 1024u);
            const u32 have = unit_have<LEAD>(len, skip);
            int off[NP];
            #pragma unroll
            for (int q = 0; q < NP; ++q) off[q] = unit_offset<LEAD>(len, skip, q * WAVE + lane);
            u32 tg = left_gen ? 0x80000000u : 0u;
            #pragma unroll
            for (int j = 0; j < G; ++j) {
                const bool any = left_gen != 0;
                const u32 w = any ? (u32)__builtin_ctzll(left_gen) : 0u;
                left_gen &= left_gen - 1;
                const u32 slot = any ? (u32)__builtin_amdgcn_readlane((int)slot32, (int)w) : 0u;
                // a buffer of `have` bytes (none for a worker without one): lanes beyond it read zeros and ask
                // memory for nothing, so every step issues the same loads; packet_units.h says where it lies
                __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                    (void*)(packets + uniform((u64)slot * g.stride + unit_base<LEAD>(skip))), 0, (int)uniform(any ? have : 0u), BUF_RAW);
                #pragma unroll
                for (int q = 0; q < NP; ++q)
                    v[d][j][q] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r, off[q], 0, BUF_NT));
            }
            if (left_gen == 0) tg |= 0x40000000u;
            if (SPARSE) {
                // the 16-byte units that lie in the span whole (and the first four floats for unit 0)
                const bool upd = tg >> 30 == 3u && ((old_any >> t_gen) & 1u);
                const u64 elem = ((u64)(u32)__builtin_amdgcn_readlane((int)(u32)(elem_l >> 32), (int)t_gen) << 32) |
                                 (u32)__builtin_amdgcn_readlane((int)(u32)elem_l, (int)t_gen);
                const u32 h = (u32)__builtin_amdgcn_readlane((int)home_l, (int)t_gen);
                __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                    (void*)uniform((u64)((h ? acc1 : acc0) + elem)), 0, (int)uniform(upd ? 4 * len : 0u), BUF_RAW);
                #pragma unroll
                for (int q = 0; q < NP; ++q) {
                    const u32 u = (piece_gen * NP + q) * WAVE + lane;
                    const bool whole = !LEAD ? u < len >> 2 : u == 0 ? len >= 4 : 4 * u + 2 <= len;
                    old[d][q] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r, !whole ? 0x40000000 : u == 0 ? 0 : (int)(16 * u - 4 * LEAD), 0, 0));
                }
            }
            tag[d] = tg | t_gen | (piece_gen << 8);
        };
        auto consume = [&](int d) {
            #pragma unroll
            for (int j = 0; j < G; ++j)
                #pragma unroll
                for (int q = 0; q < NP; ++q) a[q] += v[d][j][q];
            if ((tag[d] & 0xC0000000u) == 0xC0000000u) {
                const u32 t = tag[d] & 0xFFu, piece = (tag[d] >> 8) & 0x3FFFFFu;
                const u32 len = (u32)__builtin_amdgcn_readlane((int)len_l, (int)t);
                const u64 elem = ((u64)(u32)__builtin_amdgcn_readlane((int)(u32)(elem_l >> 32), (int)t) << 32) |
                                 (u32)__builtin_amdgcn_readlane((int)(u32)elem_l, (int)t);
                const u32 h = (u32)__builtin_amdgcn_readlane((int)home_l, (int)t);
                const bool rmw = (old_any >> t) & 1u;
                // float position i of the unit grid -> dst[i]; the payload is positions LEAD .. LEAD + len - 1
                float* dst = (h ? acc1 : acc0) + elem - LEAD;
                #pragma unroll
                for (int q = 0; q < NP; ++q) {
                    const SpanUnit<LEAD> su((piece * NP + q) * WAVE + lane, len);
                    float* o = dst + 4 * su.u;
                    f4v r = su.take(a[q] * inv_w, len);
                    if (rmw) {                                        // result = old value + this batch's sum
                        f4v ov = {0.f, 0.f, 0.f, 0.f};
                        if (SPARSE) {
                            ov = old[d][q];
                            if (su.head) ov = f4v{0.f, 0.f, ov.x, ov.y};
                        } else if (su.full) ov = *(const f4v_a4*)o;
                        if (su.part || (su.head && (!SPARSE || len < 4))) ov = su.floats(o);
                        sq -= squares(ov);
                        r = ov + r;
                    }
                    sq += squares(r);
                    su.store(o, r);
                    a[q] = f4v{0.f, 0.f, 0.f, 0.f};
                }
            }
        };
        if (SPARSE) {
            // two steps in flight and none of them empty: most waves have one to three
            static_assert(!SPARSE || (G == 1 && D == 2), "sparse: one worker per step, two steps");
            if (next()) {
                issue(0);
                for (;;) {
                    if (!next()) { consume(0); break; }
                    issue(1); consume(0);
                    if (!next()) { consume(1); break; }
                    issue(0); consume(1);
                }
            }
        } else {
            #pragma unroll
            for (int d = 0; d < D; ++d) { next(); issue(d); }
            for (;;) {
                bool more = false;
                #pragma unroll
                for (int d = 0; d < D; ++d) {
                    consume(d);
                    next(); issue(d);
                    more = more || (tag[d] >> 31);
                }
                if (!more) break;
            }
        }
    }
    }
    // accepted packets and sum-of-squares change of this block: plain adds to the block's own rows
    sq = wave_sum_f64(sq);
    if (lane == 0) { sh_accepted[wave] = accepted; sh_sq[wave] = sq; }
    __syncthreads();
    if (threadIdx.x == 0) {
        u32 total = 0;
        double t = 0.0;
        #pragma unroll
        for (int i = 0; i < NW; ++i) { total += sh_accepted[i]; t += sh_sq[i]; }
        if (total) { accept_rows[blockIdx.x] += total; sumsq_rows[blockIdx.x] += t; }
    }
}

// A retransmission of few packets is a chain of memory trips, whatever bandwidth there is, and by groups it is long: the
// tallies, the index of whole groups looked through for the entries, the entries again, the payload, and in
// a group with several packets the packets one after the other by one wave.  Where a batch holds at most FEW_MAX arrivals, and at most
// one per FEW_DIV sequence numbers of the round, the index pass also lists what it found, and a wave takes entries of the list, one output packet
// each: the entry; what its number leads to (all workers' index entries and bitmap words, the span); the payloads
// and the span's old contents; the store.  Several arrivals of one number are one output packet, taken by the one that the
// index pass noted as the first.  Packets of three and more pieces are taken by the block's waves together.  The sums and
// their order are those of the groups; a wave adds up the squares of its part of a packet, and these sums go into a long
// accumulator, so that the norm does not depend on the order of arrival either.
//
// A batch that turns out to be dense goes by groups after all: neighbours in the bitmap are set by atomics here, one
// after the other.  It pays the list, 0 to 0.6 us of 14 to 20.  us of index pass and gather, by groups and by the list:
//                                spread evenly              in runs of 20 of one worker
//   8 x 70 k of 1472 B, 273       18.5 -> 11.5               30 -> 11
//     4.4 k                       27 -> 17                   46 -> 16
//     17 k                        41 -> 34                   59 -> 31
//   4 x 312 k of 272 B, 39 k      63 -> 38                  111 -> 36
//     78 k                        91 -> 68                  133 -> 63
//   8 x 27 k of 8992 B, 1.7 k     34 -> 22                   59 -> 21
//   4 x 3.7 k of 64 KB, 465       53 -> 29                   71 -> 28
//   16 x 29 k of 4112 B, 7.3 k    37 -> 29                   47 -> 28
// and by the list where it holds as many arrivals as every second number: 1 x 35 k 40 -> 53, 8 x 35 k 50 -> 60.
#define FEW_DIV 4u
#define FEW_MAX 131072u      // more are as a rule a step of a round in chunks, whose index pass would pay a second atomic for each (78 k of 272 B 25, 26 us)
#define FEW_DEPTH(np) ((np) == 1 ? 8 : (np) == 2 ? 4 : 2)    // workers' pieces that a step loads
#define FEW_TEAM(g, np) ((g).units > 2u * (np) * WAVE)       // packets of three and more pieces

// What a sequence number of the list leads to; lane w: worker w's.
struct FewFound { u64 p, bits; u32 seq, home, fs; u64 off, cnt; };
__device__ __forceinline__ FewFound few_look_up(const Geo& g, u64 e, const u64* pending, const u64* bitmap, const uint8_t* home) {
    FewFound f;
    const u32 lane = lane_id(), b = (u32)(e >> 32);
    f.seq = (u32)e;
    f.p = NONE64; f.bits = 0;
    if (lane < g.W) {
        f.p = pending[(u64)lane * g.n_pkts + f.seq];
        f.bits = bitmap[(u64)lane * g.words_pw + (f.seq >> 6)];
    }
    f.home = home[f.seq];
    f.fs = g.first_seq[b]; f.off = g.b_off[b]; f.cnt = g.b_cnt[b];
    return f;
}

// Entry of the list that a lane of a team takes, from k0 on (below); NONE64 behind the last one.
template <bool TEAM, int NW>
__device__ __forceinline__ u64 few_entry(const ArrivalList& few, u64 k0, u32 n_blocks) {
    const u64 k = k0 + (u64)lane_id() * (TEAM ? n_blocks : n_blocks * NW);
    return k < few.n ? few.entries[k] : NONE64;
}
template <bool TEAM, int NW>
__device__ __forceinline__ u32 few_team() { return TEAM ? blockIdx.x : blockIdx.x * NW + uniform(threadIdx.x / WAVE); }

template <int NP, int NW, u32 LEAD, bool TEAM>
__device__ __forceinline__ void gather_few(const Geo& g, const uint8_t* __restrict__ packets, u64* __restrict__ pending, u64* __restrict__ bitmap,
                                           float* acc0, float* acc1, uint8_t* __restrict__ home, u32 pick, const ArrivalList& few, u64 e, u32 n_blocks,
                                           u64* __restrict__ accept_rows, double* __restrict__ sumsq_rows, float inv_w) {
    __shared__ u32 sh_accepted[NW];
    __shared__ u64 sh_long[NW][LONG_WORDS];     // per wave: a long accumulator of its changes of the sum of squares
    __shared__ double sh_odd[NW];               // and the infinities and NaN, which that does not take
    const u32 lane = lane_id(), wave = uniform(threadIdx.x / WAVE);
    constexpr int D = FEW_DEPTH(NP);
    constexpr u32 team = TEAM ? NW : 1;
    const u32 n_teams = TEAM ? n_blocks : n_blocks * NW;
    const bool leader = !TEAM || wave == 0;
    u32 accepted = 0;
    if (lane < LONG_WORDS) sh_long[wave][lane] = 0;
    if (lane == 0) sh_odd[wave] = 0.0;
    auto take = [&](const FewFound& f) {
        const u32 seq = f.seq;
        const bool had = (f.bits >> (seq & 63)) & 1ull;             // delivered by an earlier batch
        const bool fresh = f.p != NONE64 && !had;                   // a copy of a delivered packet is dropped
        const u64 new_w = uniform((u64)__ballot(fresh)), old_w = uniform((u64)__ballot(had));
        const u32 slot32 = (u32)f.p;
        if (TEAM) __syncthreads();      // every wave of the block has read the entries before they are reset
        if (leader) {
            if (f.p != NONE64) pending[(u64)lane * g.n_pkts + seq] = NONE64;    // leave the index empty
            if (fresh) atomicOr(&bitmap[(u64)lane * g.words_pw + (seq >> 6)], 1ull << (seq & 63));
            if (lane == 0) {
                few.first[seq] = NONE32;
                if (new_w && !old_w) home[seq] = (uint8_t)pick;
            }
            accepted += (u32)__popcll(new_w);
        }
        if (!new_w) return;
        const u64 start = (u64)(seq - f.fs) * g.P, left_in = uniform(f.cnt) - start;
        const u32 len = uniform(left_in < g.P ? (u32)left_in : g.P);
        const u32 h = uniform(old_w ? f.home & 1u : pick);
        float* const span = (h ? acc1 : acc0) + uniform(f.off + start);
        float* const dst = span - LEAD;             // float position i of the unit grid -> dst[i]
        double sq = 0.0;        // change of the sum of squares of the stored values
        for (u32 piece = TEAM ? wave : 0; piece * (NP * 256u) < len + LEAD; piece += team) {
            const u32 skip = piece * (NP * 1024u), have = unit_have<LEAD>(len, skip);
            int off[NP];
            f4v a[NP], old[NP];
            #pragma unroll
            for (int q = 0; q < NP; ++q) { off[q] = unit_offset<LEAD>(len, skip, q * WAVE + lane); a[q] = f4v{0.f, 0.f, 0.f, 0.f}; }
            {   // the 16-byte units that lie in the span whole (and the first four floats for unit 0)
                __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)uniform((u64)span), 0, (int)uniform(old_w ? 4 * len : 0u), BUF_RAW);
                #pragma unroll
                for (int q = 0; q < NP; ++q) {
                    const u32 u = (piece * NP + q) * WAVE + lane;
                    const bool whole = !LEAD ? u < len >> 2 : u == 0 ? len >= 4 : 4 * u + 2 <= len;
                    old[q] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r, !whole ? 0x40000000 : u == 0 ? 0 : (int)(16 * u - 4 * LEAD), 0, 0));
                }
            }
            for (u64 left = new_w; left;) {
                f4v v[D][NP];
                #pragma unroll
                for (int d = 0; d < D; ++d) {
                    if (d && left == 0) {
                        #pragma unroll
                        for (int q = 0; q < NP; ++q) v[d][q] = f4v{0.f, 0.f, 0.f, 0.f};
                        continue;
                    }
                    const u32 w = (u32)__builtin_ctzll(left);
                    left &= left - 1;
                    const u32 slot = (u32)__builtin_amdgcn_readlane((int)slot32, (int)w);
                    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                        (void*)(packets + uniform((u64)slot * g.stride + unit_base<LEAD>(skip))), 0, (int)uniform(have), BUF_RAW);
                    #pragma unroll
                    for (int q = 0; q < NP; ++q)
                        v[d][q] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r, off[q], 0, BUF_NT));
                }
                #pragma unroll
                for (int d = 0; d < D; ++d)
                    #pragma unroll
                    for (int q = 0; q < NP; ++q) a[q] += v[d][q];
            }
            #pragma unroll
            for (int q = 0; q < NP; ++q) {
                const SpanUnit<LEAD> su((piece * NP + q) * WAVE + lane, len);
                float* o = dst + 4 * su.u;
                f4v r = su.take(a[q] * inv_w, len);
                if (old_w) {                                        // result = old value + this batch's sum
                    f4v ov = old[q];
                    if (su.head) ov = f4v{0.f, 0.f, ov.x, ov.y};
                    if (su.part || (su.head && len < 4)) ov = su.floats(o);
                    sq -= squares(ov);
                    r = ov + r;
                }
                sq += squares(r);
                su.store(o, r);
            }
        }
        sq = wave_sum_f64(sq);
        const u64 bits = (u64)__double_as_longlong(sq);
        if (long_fits(bits)) { if (lane < LONG_WORDS) sh_long[wave][lane] += long_word(bits, lane); }
        else if (lane == 0) sh_odd[wave] += sq;
    };

    // A team's entries lie n_teams apart, so that the first ones of a number, which a list sorted by worker has
    // at its beginning, fall to all teams; 64 of them at a time, one per lane.
    for (u64 k0 = few_team<TEAM, NW>();;) {
        auto look_up = [&](u32 i) {
            return few_look_up(g, (u64)(u32)__builtin_amdgcn_readlane((int)(u32)(e >> 32), (int)i) << 32 | (u32)__builtin_amdgcn_readlane((int)(u32)e, (int)i), pending, bitmap, home);
        };
        // most teams have one entry, and it is the first with its number: both are asked at once
        const u32 first = e != NONE64 ? few.first[(u32)e] : NONE32;
        FewFound f;
        const bool ahead = uniform(e) != NONE64;
        if (ahead) f = look_up(0);
        u64 mine = uniform((u64)__ballot(e != NONE64 && first == (u32)(k0 + (u64)lane * n_teams)));
        if (mine && !(ahead && (mine & 1ull))) f = look_up((u32)__builtin_ctzll(mine));
        while (mine) {
            mine &= mine - 1;
            const FewFound at = f;
            if (mine) f = look_up((u32)__builtin_ctzll(mine));
            take(at);
        }
        k0 += (u64)WAVE * n_teams;
        if (k0 >= few.n) break;
        e = few_entry<TEAM, NW>(few, k0, n_blocks);
    }
    // Accepted packets of this block, to its own row (an atomic nobody waits for, where += waits for what was there).  Its change of
    // the sum of squares: integers, added to one of the long accumulators, since which block a packet falls to depends on when it arrived.
    if (lane == 0) sh_accepted[wave] = accepted;
    __syncthreads();
    if (threadIdx.x < LONG_WORDS) {
        u64 t = 0;
        #pragma unroll
        for (int i = 0; i < NW; ++i) t += sh_long[i][threadIdx.x];
        if (t) atomicAdd(bitmap - LONG_ALL + blockIdx.x % LONG_COPIES * LONG_PITCH + threadIdx.x, t);
    }
    if (threadIdx.x == 0) {
        u32 total = 0;
        double odd = 0.0;
        #pragma unroll
        for (int i = 0; i < NW; ++i) { total += sh_accepted[i]; odd += sh_odd[i]; }
        if (total) atomicAdd(&accept_rows[blockIdx.x], (u64)total);
        if (!(odd == 0.0)) sumsq_rows[blockIdx.x] += odd;       // the same sum in any order
    }
}

// gather_few for batches so small that it is the better way whatever they are (few_always): nobody waits for the tallies, and
// one block more than take entries books them.
template <int NP, u32 LEAD, bool TEAM>
__global__ __launch_bounds__(GS_WAVES * WAVE) void gather_list(Geo g, const uint8_t* __restrict__ packets, u64* __restrict__ pending, u64* __restrict__ bitmap,
                                                               float* acc0, float* acc1, uint8_t* __restrict__ home, u32 pick, ArrivalList few,
                                                               const u32* __restrict__ block_tallies, u32 n_tally_rows, u64* __restrict__ counters,
                                                               u64* __restrict__ accept_rows, double* __restrict__ sumsq_rows, float inv_w, u32* __restrict__ told) {
    __shared__ u32 sh_tally[GS_WAVES * 5];
    const u32 n_blocks = gridDim.x - 1;
    if (blockIdx.x == n_blocks) {
        const BatchInfo bi = fold_index_tallies(block_tallies, n_tally_rows, counters, true, sh_tally);
        if (told && threadIdx.x == 0) *told = batch_is_sparse(bi, g.W) ? TOLD_SPARSE : TOLD_DENSE;
        return;
    }
    gather_few<NP, GS_WAVES, LEAD, TEAM>(g, packets, pending, bitmap, acc0, acc1, home, pick, few, few_entry<TEAM, GS_WAVES>(few, few_team<TEAM, GS_WAVES>(), n_blocks),
                                         n_blocks, accept_rows, sumsq_rows, inv_w);
}

// A batch of at least one arrival per two (worker, seq) pairs of the round is taken to touch all of it: its gather need not
// read the index pass's tallies, a load and two barriers, before it starts (4 x 1 M elements in 1040-byte packets 10.8,
// 8.1 us; 8 x 25.6 M in 1472-byte ones, in bursts, 156.7, 153.9).  What it may look through for nothing is 16 bytes of the index
// for each arrival at most, where the index pass has read each one's header; not even that where no arrival was valid,
// which one word says (a stale round of 8 x 124 M 62.7 us; 99.7 without the word).  Slots that a mask says were lost count as arrivals but cost
// the index pass nothing, so with a mask only rounds that the blocks walk in two turns are taken whole (8 x 124 M, a mask of 1 %
// of the range 29 against 87 us; all lost 15 and 54).
#define WHOLE_DIV 2
__device__ __forceinline__ BatchInfo whole_round(const Geo& g) {
    BatchInfo bi;
    bi.lo = 0; bi.hi = g.n_pkts; bi.cand = (u64)g.n_pkts * g.W;
    return bi;
}

// What a gather launch is told of its batch, and two kinds of words it may use:
//   flags[F_ANY + i] says whether the index pass met a valid arrival.  (Never no when it did; where launches are recorded and
//                    told again it may be yes when it did not.)  A gather clears the other one, for the next batch that uses one.
//   flags[F_TOOK]    says whether the gather_burst launch before took the batch.
enum { B_WHOLE = 1, B_ANY = 2, B_ANY_AT = 4, B_ASKED = 8 };
enum { F_ANY = 0, F_TOOK = 2, F_COUNT };
__device__ __forceinline__ bool some_arrived(u64* __restrict__ flags, u32 batch) {
    if (!(batch & B_ANY)) return true;
    const u32 at = batch & B_ANY_AT ? 1u : 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) flags[F_ANY + (at ^ 1u)] = 0;
    return flags[F_ANY + at] != 0;
}

// DENSE: the host knows that the batch is dense; otherwise the index pass's tallies decide.
template <int NP, int G, int D, int NW, u32 LEAD, bool DENSE, bool MANY>
__global__ __launch_bounds__(NW * WAVE) __attribute__((amdgpu_waves_per_eu(4))) void gather_stream(
    Geo g, const uint8_t* __restrict__ packets, u64* __restrict__ pending, u64* __restrict__ bitmap,
    float* acc0, float* acc1, uint8_t* __restrict__ home, u32 pick,
    const u32* __restrict__ block_tallies, u32 n_tally_rows, u64* __restrict__ counters,
    u64* __restrict__ accept_rows, double* __restrict__ sumsq_rows, float inv_w,
    GatherShape dense, GatherShape sparse, u32 cus, u32 heavy, u32 table_at, u32 batch, u64* __restrict__ flags, u32* __restrict__ told, ArrivalList few) {
    extern __shared__ u32 sh_dyn[];                 // per wave: slots [W rounded up][sub + 1]; then the bucket table (table_at words in, 0: not there)
    __shared__ u32 sh_tally[NW * 5];
    const u32* fs = g.first_seq;
    if (!DENSE && batch & B_ASKED && flags[F_TOOK]) {
        if (!DENSE && told && blockIdx.x == 0 && threadIdx.x == 0) *told = TOLD_BURST;
        return;
    }
    constexpr int FP = NP > 4 ? 3 : NP;             // KB of a piece, and whether the block takes them together, where the batch is few packets
    const bool teams = !DENSE && few.entries && FEW_TEAM(g, FP);
    u64 entry = NONE64;
    if (!DENSE && few.entries)                      // on its way while the tallies are
        entry = teams ? few_entry<true, NW>(few, few_team<true, NW>(), gridDim.x) : few_entry<false, NW>(few, few_team<false, NW>(), gridDim.x);
    const bool some = some_arrived(flags, batch);
    if (table_at) {
        u32* tab = sh_dyn + table_at;
        for (u32 i = threadIdx.x; i <= g.B; i += blockDim.x) tab[i] = g.first_seq[i];
        fs = tab;
    }
    // block 0 books the index pass's tallies; the barriers in there cover the table too
    BatchInfo bi;
    const bool whole = DENSE && batch & B_WHOLE;
    if (whole && blockIdx.x) {
        if (!some) return;
        bi = whole_round(g);
    } else {
        bi = fold_index_tallies(block_tallies, n_tally_rows, counters, blockIdx.x == 0 && (DENSE || !(batch & B_ASKED)), sh_tally);     // (a gather_burst launch before has booked them)
        if (whole && bi.hi) bi = whole_round(g);
    }
    if (whole) __syncthreads();
    const bool is_sparse = !DENSE && batch_is_sparse(bi, g.W);
    if (!DENSE && told && blockIdx.x == 0 && threadIdx.x == 0) *told = is_sparse ? TOLD_SPARSE : TOLD_DENSE;    // for the trace group of the launch
    if (bi.hi == 0) return;                         // no candidate in this batch (uniform over the grid)
    if (!DENSE && few.entries) {
        if (is_sparse) {
            if (teams) gather_few<FP, NW, LEAD, true>(g, packets, pending, bitmap, acc0, acc1, home, pick, few, entry, gridDim.x, accept_rows, sumsq_rows, inv_w);
            else gather_few<FP, NW, LEAD, false>(g, packets, pending, bitmap, acc0, acc1, home, pick, few, entry, gridDim.x, accept_rows, sumsq_rows, inv_w);
            return;
        }
        for (u64 i = bi.lo + (u64)blockIdx.x * blockDim.x + threadIdx.x; i < bi.hi; i += (u64)gridDim.x * blockDim.x) few.first[i] = NONE32;
    }
    if (is_sparse)
        gather_groups<2, 1, 2, NW, true, LEAD, MANY>(g, bi, sparse, fs, sh_dyn, packets, pending, bitmap, acc0, acc1, home, pick, accept_rows, sumsq_rows, inv_w);
    else {
        // a dense batch's groups are sized for the range that it covers: a step of a round that arrives in many
        // steps is a short round.  Blocks of four waves: at least a piece for each.
        u32 l = group_log2(bi.hi - bi.lo, cus, dense.n_piece > 1, heavy);
        if (NW == GS_WAVES) while (dense.n_piece << l < GS_WAVES) ++l;
        dense.sub_log2 = uniform(l);
        gather_groups<NP, G, D, NW, false, LEAD, MANY>(g, bi, dense, fs, sh_dyn, packets, pending, bitmap, acc0, acc1, home, pick, accept_rows, sumsq_rows, inv_w);
    }
}

// ------------------------------------------------------------------------------------------
// gather in bursts: large dense batches
// ------------------------------------------------------------------------------------------
// What bounds a large gather is that it writes: read alone, its payloads stream at 6.5 TB/s, and with the 3 % of
// result bytes of 32 workers stored as each packet's sum is ready, at 5.3 (a write that comes alone turns the memory
// bus round for few bytes).  One block per CU therefore sums a whole group of consecutive packets, as many as fit its
// LDS, into an image of their spans, and then stores the image at once: long, contiguous, whole 128-byte lines, while
// the block reads nothing.  In turn, a loop with this access pattern, 32 workers x 1472 B, 8.5 GB: stored at once per
// packet 1711 us, in bursts of 23 KB 1629, of 70 KB and more 1450 to 1500; read only 1290.  Three things that looked
// natural made it slower: loads of the next group in flight while the image goes out (8 workers, 9.8 GB: 1709 us
// without, 1788 with), two blocks per CU (1927), and a second step of loads in flight per wave (equal, or up to
// 2 % slower; what larger steps cost stands at burst_kernel).  What stays between two groups is kept short instead: a group's arrival index is loaded a whole group
// ahead and brought into LDS by each wave as it ends its share of the group before.
//
// Against gather_stream, us per launch (whole pass in brackets), buffers where the allocator put them:
//   8 workers x 124 M elements, 1472 B packets      895 ->  795 (1157 -> 1035)
//   8 x 124 M, 8992 B                               925 ->  790 (1033 ->  888)
//   16 x 355 M, 4112 B                             4620 -> 4080 (4843 -> 4350)
//   32 x 66 M (one of three steps), 1472 B         1632 -> 1450
//   8 x 25.6 M, 1472 B                              179 ->  158 (285 -> 265)
//   4 x 150 M, 1472 B                               596 ->  527 (777 -> 682)
//
// How the image is stored (`through`): written through to the memory-side cache (256 MB) where the written range
// stays in it, else past it: 8 x 25.6 M, 158 and 163 us; 16 x 355 M, 4376 and 4178; the passes that follow are
// faster too where the cache is left alone (index pass of 8 x 124 M 150 and 129 us).
#define BURST_WAVES 16       // one block per CU: four waves on each SIMD
#define BURST_MAX 256u       // sequence numbers of a group
#define BURST_AHEAD 4        // (worker, 64 sequence numbers) of the next group's index that a wave holds in registers
#define BURST_LDS 161792u    // dynamic: 160 KB less 2 KB for the rest
#define BUF_SC1 16           // store policy: written through

// Words of dynamic LDS: slots [W][r | 1], span starts and lengths (each for two groups), then the bucket table, then the
// image of the group's spans (32 floats more, so that it can start where its first span lies in a 128-byte line).
#define BURST_INFO_LDS(W, r) (2u * (W) * ((r) | 1u) + 6u * (r))

template <int NP, int G, u32 LEAD>
__global__ __launch_bounds__(BURST_WAVES * WAVE) void gather_burst(
    Geo g, const uint8_t* __restrict__ packets, u64* __restrict__ pending, u64* __restrict__ bitmap,
    float* acc0, float* acc1, uint8_t* __restrict__ home, u32 pick,
    const u32* __restrict__ block_tallies, u32 n_tally_rows, u64* __restrict__ counters,
    u64* __restrict__ accept_rows, double* __restrict__ sumsq_rows, float inv_w,
    u32 r_max, u32 r_step, u32 n_piece, u32 table_at, u32 image_at, u32 min_seq, u32 through_seq, u32 batch, u64* __restrict__ flags) {
    extern __shared__ __attribute__((aligned(16))) u32 sh_dyn[];
    __shared__ u32 sh_tally[BURST_WAVES * 5];
    __shared__ u32 sh_new[3][BURST_MAX / 32], sh_old[3][BURST_MAX / 32];     // by packet of the group: new copies; delivered before
    __shared__ u32 sh_accepted[BURST_WAVES];
    __shared__ double sh_sq[BURST_WAVES];
    const u32 tid = threadIdx.x, lane = lane_id();
    const u32 wave = uniform(tid / WAVE);
    const u32 W = g.W, pitch = r_max | 1u;
    u32* const sh_elem = sh_dyn + 2 * W * pitch;                    // [2][r_max][2]
    u32* const sh_len = sh_elem + 4 * r_max;                    // [2][r_max]: floats | home << 16
    float* const image = (float*)(sh_dyn + image_at);
    const u32* fs = g.first_seq;
    const bool some = some_arrived(flags, batch);
    if (table_at) {
        u32* tab = sh_dyn + table_at;
        for (u32 i = tid; i <= g.B; i += BURST_WAVES * WAVE) tab[i] = g.first_seq[i];
        fs = tab;
    }
    if (tid < 3 * (BURST_MAX / 32)) sh_new[0][tid] = sh_old[0][tid] = 0;
    BatchInfo bi = whole_round(g);
    const bool whole = batch & B_WHOLE;
    if (!whole || blockIdx.x == 0) {
        const BatchInfo found = fold_index_tallies(block_tallies, n_tally_rows, counters, blockIdx.x == 0, sh_tally);
        if (!whole || found.hi == 0) bi = found;
    } else {
        if (!some) return;
        __syncthreads();
    }
    // A batch that is none of this kernel's is left to the gather_stream launch that follows.
    const bool mine = bi.hi != 0 && (min_seq == 0 || (!batch_is_sparse(bi, g.W) && bi.hi - bi.lo >= min_seq &&
                                                      burst_pays(bi.cand, bi.hi - bi.lo, g.W, gridDim.x, r_max, NP * n_piece)));
    if (min_seq && blockIdx.x == 0 && tid == 0) flags[F_TOOK] = mine;
    if (!mine) return;
    // Groups of equal size but for one step: with all groups as long as the longest, the last turn of 4 x 61 M in 64
    // KB packets left two CUs in three idle (7.3 turns of two packets and an eighth of that; now seven of two and one of
    // one).
    const u32 lo = uniform((u32)bi.lo / r_step * r_step), n_seq = uniform((u32)bi.hi) - lo;
    const BurstTurns split(n_seq, gridDim.x, r_max, r_step);
    const u32 r_long = uniform(split.r_long);
    auto first_of = [&](u32 turn) {
        const u32 at = uniform(split.first(turn, blockIdx.x));
        return at < n_seq ? lo + at : NONE32;
    };
    auto size_of = [&](u32 turn, u32 seq0) { return uniform(split.count(turn, g.n_pkts - seq0)); };       // of the group that starts there
    const bool through = n_seq <= through_seq;
    const u32 n_chunk = (r_long + WAVE - 1) / WAVE, n_pair = W * n_chunk;        // a pair: a worker's index entries of 64 sequence numbers
    const u32* const words = (const u32*)bitmap;
    u32 accepted = 0;
    double sq = 0.0;

    struct Entry { u64 p; u32 bits; };
    auto load_entry = [&](u32 pair, u32 s0, u32 r) {
        Entry e;
        e.p = NONE64; e.bits = 0;
        const u32 w = pair / n_chunk, t = (pair - w * n_chunk) * WAVE + lane, seq = s0 + t;
        if (pair < n_pair && t < r) {
            e.p = pending[(u64)w * g.n_pkts + seq];
            e.bits = words[2 * (u64)w * g.words_pw + (seq >> 5)];
        }
        return e;
    };
    Entry ahead[BURST_AHEAD];
    u32 home_ahead = 0;
    auto load_ahead = [&](u32 s0, u32 r) {
        #pragma unroll
        for (int j = 0; j < BURST_AHEAD; ++j) ahead[j] = load_entry(wave + j * BURST_WAVES, s0, r);
        home_ahead = tid < r ? home[s0 + tid] : 0;
    };

    // A group's arrival index -> slots, bitmap, spans, in its half of the tables (par) and its flags (f).
    auto take_group = [&](u32 seq0, u32 r, u32 par, u32 f) {
        u32* const slots = sh_dyn + par * W * pitch;
        auto take_entry = [&](u32 pair, const Entry& e) {
            if (pair >= n_pair) return;
            const u32 w = pair / n_chunk, c = pair - w * n_chunk, t = c * WAVE + lane, seq = seq0 + t;
            const bool in = t < r;
            const bool had = in && (e.bits >> (seq & 31)) & 1u;             // delivered by an earlier batch
            const bool fresh = in && e.p != NONE64 && !had;
            const u64 nb = __ballot(fresh), hb = __ballot(had);
            if (in) slots[w * pitch + t] = fresh ? (u32)e.p : NONE32;
            if (in && e.p != NONE64) pending[(u64)w * g.n_pkts + seq] = NONE64;         // leave the index empty
            if (nb) {
                if (r_step == 8) {      // a group owns its bytes of the bitmap
                    const u32 mine = (u32)(nb >> (lane & ~7u)) & 0xFFu;
                    if ((lane & 7) == 0 && mine)
                        ((uint8_t*)(bitmap + (u64)w * g.words_pw))[seq >> 3] = (uint8_t)(mine | ((u32)(hb >> lane) & 0xFFu));
                } else if (fresh) atomicOr((u32*)bitmap + 2 * (u64)w * g.words_pw + (seq >> 5), 1u << (seq & 31));
            }
            if (lane < 2) {
                const u32 n = (u32)(nb >> (32 * lane)), o = (u32)(hb >> (32 * lane));
                if (n) atomicOr(&sh_new[f][2 * c + lane], n);
                if (o) atomicOr(&sh_old[f][2 * c + lane], o);
            }
            accepted += (u32)__popcll(nb);
        };
        #pragma unroll
        for (int j = 0; j < BURST_AHEAD; ++j) take_entry(wave + j * BURST_WAVES, ahead[j]);
        for (u32 pair = wave + BURST_AHEAD * BURST_WAVES; pair < n_pair; pair += BURST_WAVES) take_entry(pair, load_entry(pair, seq0, r));
        if (tid < r) {
            const u32 seq = seq0 + tid, b = find_bucket(g, fs, seq);
            const u64 start = (u64)(seq - fs[b]) * g.P, left = g.b_cnt[b] - start, elem = g.b_off[b] + start;
            u32* const elem_of = sh_elem + par * 2 * r_max;
            elem_of[2 * tid] = (u32)elem; elem_of[2 * tid + 1] = (u32)(elem >> 32);
            sh_len[par * r_max + tid] = (left < g.P ? (u32)left : g.P) | (home_ahead & 1u) << 16;
        }
    };

    u32 par = 0, f = 0;
    u32 seq0 = first_of(0);
    if (seq0 != NONE32) { load_ahead(seq0, size_of(0, seq0)); take_group(seq0, size_of(0, seq0), 0, 0); }
    __syncthreads();
    for (u32 turn = 0; seq0 != NONE32; ++turn, par ^= 1, f = f == 2 ? 0 : f + 1) {
        const u32 n_t = size_of(turn, seq0), seq_next = first_of(turn + 1);
        const u32 n_next = seq_next != NONE32 ? size_of(turn + 1, seq_next) : 0;
        const u32* const slots = sh_dyn + par * W * pitch;
        const u32* const elem_of = sh_elem + par * 2 * r_max;
        const u32* const len_of = sh_len + par * r_max;
        const u32* const is_new = sh_new[f];
        const u32* const is_old = sh_old[f];
        auto flag = [](const u32* m, u32 t) { return (m[t >> 5] >> (t & 31)) & 1u; };
        if (seq_next != NONE32) load_ahead(seq_next, n_next);
        const u64 e0 = uniform(((u64)elem_of[1] << 32) | elem_of[0]);
        const u32 pad = (u32)e0 & 31u;                  // the image starts where its first span lies in a 128-byte line

        // ---- payloads: lane i holds the wave's i-th item, a piece of NP KB of a packet; G workers' pieces make
        // one step
        const u32 item = wave + lane * BURST_WAVES;
        const u32 t_l = n_piece == 1 ? item : item / n_piece, piece_l = item - t_l * n_piece;
        u32 len_l = 0, at_l = 0, how_l = 0;             // at: first float of the span in the image; how: 1 it has contents, 3 and in the other copy
        bool need = false;
        if (t_l < n_t) {
            const u32 lw = len_of[t_l];
            len_l = lw & 0xFFFFu;
            const bool old = flag(is_old, t_l);
            need = flag(is_new, t_l) && piece_l * (NP * 256u) < len_l + LEAD;
            at_l = pad + (u32)((((u64)elem_of[2 * t_l + 1] << 32) | elem_of[2 * t_l]) - e0);
            how_l = old ? (lw >> 16 != pick ? 3u : 1u) : 0u;
        }
        u64 todo = uniform((u64)__ballot(need));
        u64 left = 0;                   // workers of item i still to be loaded
        u32 i = 0;
        u32 slot32 = NONE32;            // lane w: slot of worker w's copy of the item's packet
        f4v v[G][NP], a[NP];
        #pragma unroll
        for (int q = 0; q < NP; ++q) a[q] = f4v{0.f, 0.f, 0.f, 0.f};
        auto load = [&]() {
            if (left == 0) {
                i = (u32)__builtin_ctzll(todo);
                todo &= todo - 1;
                slot32 = lane < W ? slots[lane * pitch + (u32)__builtin_amdgcn_readlane((int)t_l, (int)i)] : NONE32;
                left = uniform((u64)__ballot(slot32 != NONE32));
            }
            const u32 len = (u32)__builtin_amdgcn_readlane((int)len_l, (int)i);
            const u32 skip = (u32)__builtin_amdgcn_readlane((int)piece_l, (int)i) * (NP * 1024u);
            const u32 have = unit_have<LEAD>(len, skip);
            int off[NP];
            #pragma unroll
            for (int q = 0; q < NP; ++q) off[q] = unit_offset<LEAD>(len, skip, q * WAVE + lane);
            #pragma unroll
            for (int j = 0; j < G; ++j) {
                const bool any = left != 0;
                const u32 w = any ? (u32)__builtin_ctzll(left) : 0u;
                left &= left - 1;
                const u32 slot = any ? (u32)__builtin_amdgcn_readlane((int)slot32, (int)w) : 0u;
                __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                    (void*)(packets + uniform((u64)slot * g.stride + unit_base<LEAD>(skip))), 0, (int)uniform(any ? have : 0u), BUF_RAW);
                #pragma unroll
                for (int q = 0; q < NP; ++q)
                    v[j][q] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r, off[q], 0, BUF_NT));
            }
        };
        auto add = [&]() {
            #pragma unroll
            for (int j = 0; j < G; ++j)
                #pragma unroll
                for (int q = 0; q < NP; ++q) a[q] += v[j][q];
            if (left) return;
            const u32 len = (u32)__builtin_amdgcn_readlane((int)len_l, (int)i), at = (u32)__builtin_amdgcn_readlane((int)at_l, (int)i);
            const u32 how = (u32)__builtin_amdgcn_readlane((int)how_l, (int)i), piece = (u32)__builtin_amdgcn_readlane((int)piece_l, (int)i);
            if (how == 0 && (LEAD || (len & 3u) == 0)) {          // a span that this batch opens
                #pragma unroll
                for (int q = 0; q < NP; ++q) {
                    const u32 row = (piece * NP + q) * (4 * WAVE);            // 256 floats of the unit grid
                    const u32 p0 = row + 4 * lane - LEAD;                     // the unit's first float in the payload (wraps before it)
                    f4v r = a[q] * inv_w;
                    a[q] = f4v{0.f, 0.f, 0.f, 0.f};
                    float* const o = image + (int)(at + p0);
                    if (row >= LEAD && row + 4 * WAVE <= len + LEAD) {
                        sq += squares(r);
                        *(f4v_a4*)o = r;
                    } else if (row < len + LEAD) {
                        const bool m0 = p0 < len, m1 = p0 + 1 < len, m2 = p0 + 2 < len, m3 = p0 + 3 < len;
                        r = f4v{m0 ? r.x : 0.f, m1 ? r.y : 0.f, m2 ? r.z : 0.f, m3 ? r.w : 0.f};
                        sq += squares(r);
                        if (m0 && m3) *(f4v_a4*)o = r;
                        else {
                            if (m0) o[0] = r.x;
                            if (m1) o[1] = r.y;
                            if (m2) o[2] = r.z;
                            if (m3) o[3] = r.w;
                        }
                    }
                }
                return;
            }
            float* const img = image + (int)(at - LEAD);
            float* const old = ((how == 3u) != (pick != 0) ? acc1 : acc0) + (e0 - pad + at) - LEAD;
            #pragma unroll
            for (int q = 0; q < NP; ++q) {
                const SpanUnit<LEAD> su((piece * NP + q) * WAVE + lane, len);
                f4v r = su.take(a[q] * inv_w, len);
                if (how) {                                        // result = old value + this batch's sum
                    const f4v ov = su.full ? *(const f4v_a4*)(old + 4 * su.u) : su.floats(old + 4 * su.u);
                    sq -= squares(ov);
                    r = ov + r;
                }
                sq += squares(r);
                if (how == 3u) su.store(old + 4 * su.u, r);       // stays in the other copy
                else su.store(img + 4 * su.u, r);
                a[q] = f4v{0.f, 0.f, 0.f, 0.f};
            }
        };
        const bool any_item = todo != 0;
        if (any_item) load();
        __syncthreads();                // every wave has read the group before out of the image
        {   // the flags of the group before are free: they are the ones of the group after the next
            const u32 z = f == 0 ? 2 : f - 1;
            if (tid < BURST_MAX / 32) sh_new[z][tid] = sh_old[z][tid] = 0;
        }
        if (tid < n_t && flag(is_new, tid) && !flag(is_old, tid)) home[seq0 + tid] = (uint8_t)pick;
        if (any_item)
            for (;;) {
                add();
                if (left == 0 && todo == 0) break;
                load();
            }
        if (seq_next != NONE32) take_group(seq_next, n_next, par ^ 1, f == 2 ? 0 : f + 1);
        __syncthreads();
        // ---- the image goes out, run by run of spans that belong to it
        float* const out = (pick ? acc1 : acc0) + (e0 - pad);
        auto in_image = [&](u32 t) { return flag(is_new, t) && !(flag(is_old, t) && len_of[t] >> 16 != pick); };
        auto at_of = [&](u32 t) { return pad + (u32)((((u64)elem_of[2 * t + 1] << 32) | elem_of[2 * t]) - e0); };
        auto store_run = [&](u32 t, u32 z) {            // spans of packets [t, z)
            const u32 from = uniform(at_of(t)), to = uniform(at_of(z - 1) + (len_of[z - 1] & 0xFFFFu));     // floats [from, to) of the image
            __amdgpu_buffer_rsrc_t o = __builtin_amdgcn_make_buffer_rsrc((void*)uniform((u64)out), 0, (int)(4 * to), BUF_RAW);
            for (u32 u = (from >> 5 << 3) + tid; 4 * u < to; u += BURST_WAVES * WAVE) {
                const f4v r = *(const f4v*)(image + 4 * u);
                if (4 * u >= from && 4 * u + 4 <= to) {
                    if (through) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4v, r), o, 16 * u, 0, BUF_SC1);
                    else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4v, r), o, 16 * u, 0, BUF_NT);
                } else {
                    #pragma unroll
                    for (u32 k = 0; k < 4; ++k)
                        if (4 * u + k >= from && 4 * u + k < to) out[4 * u + k] = r[k];
                }
            }
        };
        u32 open = NONE32;                              // first packet of the run at hand
        for (u32 c = 0; c < n_chunk; ++c) {
            const u32 t = c * WAVE + lane;
            const u64 m = uniform((u64)__ballot(t < n_t && in_image(t)));
            for (u32 pos = 0; pos < WAVE;) {
                const u64 rest = (open == NONE32 ? m : ~m) >> pos;
                if (rest == 0) break;
                pos += (u32)__builtin_ctzll(rest);
                if (open == NONE32) open = c * WAVE + pos;
                else { store_run(open, c * WAVE + pos); open = NONE32; }
            }
        }
        if (open != NONE32) store_run(open, n_t);
        seq0 = seq_next;
    }
    // accepted packets and sum-of-squares change of this block: plain adds to the block's own rows
    sq = wave_sum_f64(sq);
    if (lane == 0) { sh_accepted[wave] = accepted; sh_sq[wave] = sq; }
    __syncthreads();
    if (tid == 0) {
        u32 total = 0;
        double t = 0.0;
        #pragma unroll
        for (int i = 0; i < BURST_WAVES; ++i) { total += sh_accepted[i]; t += sh_sq[i]; }
        if (total) { accept_rows[blockIdx.x] += total; sumsq_rows[blockIdx.x] += t; }
    }
}

// ------------------------------------------------------------------------------------------
// probe: per-(worker,bucket) loss count, prefix of list lengths, ordered list
// ------------------------------------------------------------------------------------------
// Bits of word index `wd` that belong to sequence range [s0, s1).
__device__ __forceinline__ u64 range_mask(u32 wd, u32 s0, u32 s1) {
    u64 m = NONE64;
    u64 base = (u64)wd * 64;
    if (base < s0) m &= NONE64 << (s0 - base);
    if (base + 64 > s1) m &= NONE64 >> (base + 64 - s1);
    return m;
}

// BLOCK_PAIR (few pairs, buckets of more words than a wave keeps in flight): a block takes a pair, each of its waves a
// quarter of the words (148 x 8, the longest of 105 k packets: a pass of 13 us with a wave per pair, 6.5 so).  Otherwise
// a wave takes `ppw` consecutive (worker, bucket) pairs, one per lane (ppw = 1 while there are fewer pairs than waves, up
// to 64).  A pair of at most PROBE_SMALL bitmap words is its lane's own work, a larger one the whole wave's, PROBE_UNROLL
// words per lane in flight: with one wave per pair a probe over 120 k buckets x 16 workers took 250 us, and 11 so.
#define PROBE_SMALL 4
#define PROBE_UNROLL 8
struct ProbePair {
    u32 w, s0, s1;
    bool small;
    __device__ __forceinline__ ProbePair(const Geo& g, u64 pr, bool valid) : w(0), s0(0), s1(0), small(true) {
        if (!valid) return;
        w = (u32)(pr / g.B);
        const u32 b = (u32)(pr - (u64)w * g.B);
        s0 = g.first_seq[b]; s1 = g.first_seq[b + 1];
        small = ((s1 - 1) >> 6) - (s0 >> 6) < PROBE_SMALL;
    }
    // lane t's pair, in every lane
    __device__ __forceinline__ ProbePair(const ProbePair& o, u32 t)
        : w((u32)__builtin_amdgcn_readlane((int)o.w, (int)t)), s0((u32)__builtin_amdgcn_readlane((int)o.s0, (int)t)),
          s1((u32)__builtin_amdgcn_readlane((int)o.s1, (int)t)), small(o.small) {}
    // wave k's quarter of the words [*wd0, *wd1] (none: *wd0 > *wd1)
    __device__ __forceinline__ void share(u32 k, u32* wd0, u32* wd1) const {
        const u32 per = (*wd1 - *wd0 + 4) / 4, a = *wd0 + k * per, z = a + per - 1;
        *wd0 = a;
        if (z < *wd1) *wd1 = z;
    }
};

// Packets of this lane's pair that arrived (BLOCK_PAIR: in every lane of the block).  All threads call this.
template <bool BLOCK_PAIR>
__device__ __forceinline__ u32 probe_got(const Geo& g, const u64* __restrict__ bitmap, const ProbePair& p, bool valid, u32 ppw, u64* sh) {
    const u32 lane = lane_id(), wave = uniform(threadIdx.x / WAVE);
    const bool alone = ppw > 1 && p.small;
    u32 got = 0;
    if (valid && alone)
        for (u32 wd = p.s0 >> 6; wd <= (p.s1 - 1) >> 6; ++wd) got += (u32)__popcll(bitmap[(u64)p.w * g.words_pw + wd] & range_mask(wd, p.s0, p.s1));
    for (u64 m = uniform((u64)__ballot(valid && !alone)); m; m &= m - 1) {
        const u32 t = (u32)__builtin_ctzll(m);
        const ProbePair q(p, t);
        u32 wd0 = q.s0 >> 6, wd1 = (q.s1 - 1) >> 6;
        if (BLOCK_PAIR) q.share(wave, &wd0, &wd1);
        u32 cnt = 0;
        for (u32 w0 = wd0; w0 <= wd1; w0 += PROBE_UNROLL * WAVE) {
            u64 v[PROBE_UNROLL];
            #pragma unroll
            for (int k = 0; k < PROBE_UNROLL; ++k) {
                const u32 wd = w0 + k * WAVE + lane;
                v[k] = wd <= wd1 ? bitmap[(u64)q.w * g.words_pw + wd] & range_mask(wd, q.s0, q.s1) : 0ull;
            }
            #pragma unroll
            for (int k = 0; k < PROBE_UNROLL; ++k) cnt += (u32)__popcll(v[k]);
        }
        cnt = wave_reduce<OpAdd>(cnt);
        if (lane == t) got = cnt;
    }
    if (BLOCK_PAIR) {
        if (lane == 0) sh[wave] = got;
        __syncthreads();
        got = (u32)((sh[0] + sh[1]) + (sh[2] + sh[3]));
        __syncthreads();
    }
    return got;
}

// List length that a pair with `got` arrived packets asks for; *miss: packets that are missing.
__device__ __forceinline__ u32 probe_want(const ProbePair& p, u32 got, u32 bound_ppm, u32* miss) {
    const u32 n_b = p.s1 - p.s0;
    *miss = n_b - got;
    const u64 allowed = ((u64)bound_ppm * n_b) / 1000000ull;
    return (u64)*miss > allowed ? *miss : 0u;
}

// The entries of the block's pairs (`want` of this lane's, at pos0 of the list on).  sh: a word per wave (BLOCK_PAIR).
template <bool BLOCK_PAIR>
__device__ __forceinline__ void probe_emit(const Geo& g, const u64* __restrict__ bitmap, const ProbePair& p, u32 want, u64 pos0, u32 ppw,
                                           u64* __restrict__ list, u64 capacity, u64* sh) {
    const u32 lane = lane_id(), wave = uniform(threadIdx.x / WAVE);
    const bool alone = ppw > 1 && p.small;
    if (want && alone) {
        u64 pos = pos0;
        for (u32 wd = p.s0 >> 6; wd <= (p.s1 - 1) >> 6; ++wd)
            for (u64 m = ~bitmap[(u64)p.w * g.words_pw + wd] & range_mask(wd, p.s0, p.s1); m; m &= m - 1, ++pos)
                if (pos < capacity) list[pos] = ((u64)p.w << 32) | ((u64)wd * 64 + (u32)__builtin_ctzll(m));
    }
    for (u64 todo = uniform((u64)__ballot(want && !alone)); todo; todo &= todo - 1) {
        const u32 t = (u32)__builtin_ctzll(todo);
        const ProbePair q(p, t);
        u64 at = ((u64)(u32)__builtin_amdgcn_readlane((int)(u32)(pos0 >> 32), (int)t) << 32) | (u32)__builtin_amdgcn_readlane((int)(u32)pos0, (int)t);
        u32 wd0 = q.s0 >> 6, wd1 = (q.s1 - 1) >> 6;
        if (BLOCK_PAIR) {           // (want is the same in all waves: all come here) what the quarters before this one hold
            q.share(wave, &wd0, &wd1);
            u32 c = 0;
            #pragma unroll PROBE_UNROLL
            for (u32 wd = wd0 + lane; wd <= wd1; wd += WAVE) c += (u32)__popcll(~bitmap[(u64)q.w * g.words_pw + wd] & range_mask(wd, q.s0, q.s1));
            c = wave_reduce<OpAdd>(c);
            if (lane == 0) sh[wave] = c;
            __syncthreads();
            for (u32 i = 0; i < wave; ++i) at += sh[i];
        }
        for (u32 w0 = wd0; w0 <= wd1; w0 += PROBE_UNROLL * WAVE) {
            u64 v[PROBE_UNROLL];
            #pragma unroll
            for (int k = 0; k < PROBE_UNROLL; ++k) {
                const u32 wd = w0 + k * WAVE + lane;
                v[k] = wd <= wd1 ? ~bitmap[(u64)q.w * g.words_pw + wd] & range_mask(wd, q.s0, q.s1) : 0ull;
            }
            #pragma unroll
            for (int k = 0; k < PROBE_UNROLL; ++k) {
                if (w0 + k * WAVE > wd1) break;
                const u32 c = (u32)__popcll(v[k]), inc = wave_scan_incl<OpAdd>(c);
                u64 pos = at + (inc - c);
                for (u64 m = v[k]; m; m &= m - 1, ++pos)
                    if (pos < capacity) list[pos] = ((u64)q.w << 32) | ((u64)(w0 + k * WAVE + lane) * 64 + (u32)__builtin_ctzll(m));
                at += (u32)__builtin_amdgcn_readlane((int)inc, 63);
            }
        }
    }
}

// Sums over the 64 lanes: of u32 whose sum may not fit 32 bits, and of values below 2^46.
__device__ __forceinline__ u64 wave_sum_wide(u32 v) { return ((u64)wave_reduce<OpAdd>(v >> 16) << 16) + wave_reduce<OpAdd>(v & 0xFFFFu); }
__device__ __forceinline__ u64 wave_sum_u46(u64 v) {
    const u32 lo = (u32)v & 0xFFFFFu, mid = (u32)(v >> 20) & 0xFFFFFu, hi = (u32)(v >> 40);     // 64 x 2^20 fits 32 bits
    return ((u64)wave_reduce<OpAdd>(hi) << 40) + ((u64)wave_reduce<OpAdd>(mid) << 20) + wave_reduce<OpAdd>(lo);
}

// The probe in one launch, for up to seven blocks per four CUs: each block counts its pairs and tells the others the
// length of its part of the list; a block whose part is not empty, and the last one, which tells the host the whole
// length, then add up what the blocks before it told.  totals[j] = tag | length, in one 64-bit word that is stored
// and loaded as a relaxed atomic at device scope, so no fence is needed (one would write back the L2 that the gather has
// just dirtied); the tag differs from probe to probe, so nothing is cleared in between.
//
// A block tells its length before it waits for anything, and waits only for blocks of lower index.  As a rule these
// are running: a launch takes a quarter of what the chip holds at a time.  But nothing promises it: launches of other
// contexts that wait too, on streams with few CUs, on many hardware queues or from other processes, can hold every place
// that a block waited for could start in.  So a block looks `polls` times at most, then says so (mailbox[M_PROBE_GAVE_UP]) and
// ends; the host, which waits for the launch anyway, then has the list made in the launches below, whose blocks wait
// for nothing.
// Latency bounds the probe: a second launch for the list, which it was, costs its own start and a second walk to the same
// words.  us of the two launches, and of this one, first probe of a round: 64 x 4 pairs of 64 packets 6.7, 4.2; 161 x 8
// of 435 packets on average 8.9, 5.6.  (Where blocks are many the two launches cost little more: 148 x 8 pairs of 2300
// packets 11.7, 9.8; 292 x 16 of 1190 15.7, 13.9.)
#define PROBE_TAG_SHIFT 40
#define PROBE_POLL 2
#define PROBE_RESIDENT 7         // blocks (a wave on each SIMD) that a CU holds, or one fewer with more than 72 registers
#define PROBE_LOOKS 16384u       // polls, unless the caller says otherwise: 10 ms or more
template <bool BLOCK_PAIR>
__global__ __launch_bounds__(256) void probe_once(Geo g, const u64* __restrict__ bitmap, u32 bound_ppm, u32 ppw, u64 pairs, u32* __restrict__ missing_out,
                                                  u64* totals, u64 tag, u32 polls, u64* __restrict__ list, u64 capacity, u64* __restrict__ mailbox) {
    __shared__ u64 sh[4], sh_sum[4];
    const u32 lane = lane_id(), wave = uniform(threadIdx.x / WAVE);
    const u64 pr = BLOCK_PAIR ? blockIdx.x : ((u64)blockIdx.x * 4 + wave) * ppw + lane;
    const bool valid = lane < ppw && pr < pairs;
    const ProbePair p(g, pr, valid);
    const u32 got = probe_got<BLOCK_PAIR>(g, bitmap, p, valid, ppw, sh);
    u32 want = 0;
    if (valid) {
        u32 miss;
        want = probe_want(p, got, bound_ppm, &miss);
        if (missing_out && (!BLOCK_PAIR || wave == 0)) missing_out[pr] = miss;
    }
    const u32 inc_hi = wave_scan_incl<OpAdd>(want >> 16), inc_lo = wave_scan_incl<OpAdd>(want & 0xFFFFu);
    const u64 incl = ((u64)inc_hi << 16) + inc_lo;
    const u64 sum = ((u64)(u32)__builtin_amdgcn_readlane((int)inc_hi, 63) << 16) + (u32)__builtin_amdgcn_readlane((int)inc_lo, 63);
    if (lane == 0) sh_sum[wave] = sum;
    __syncthreads();
    const u64 mine = BLOCK_PAIR ? sh_sum[0] : (sh_sum[0] + sh_sum[1]) + (sh_sum[2] + sh_sum[3]);
    if (threadIdx.x == 0) __hip_atomic_store(&totals[blockIdx.x], tag | mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool last = blockIdx.x == gridDim.x - 1;
    if (!last && (mine == 0 || capacity == 0)) return;          // the same in all threads of the block
    u64 before = 0;
    u32 looks = 0;
    bool all = true;
    for (u32 i0 = threadIdx.x; all && i0 < blockIdx.x; i0 += PROBE_POLL * 256) {
        u64 v[PROBE_POLL] = {};
        do {
            all = looks++ < polls;
            if (!all) break;
            #pragma unroll
            for (u32 k = 0; k < PROBE_POLL; ++k) {
                const u32 i = i0 + k * 256;
                v[k] = i < blockIdx.x ? __hip_atomic_load(&totals[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : tag;
            }
            #pragma unroll
            for (u32 k = 0; k < PROBE_POLL; ++k) all = all && v[k] >> PROBE_TAG_SHIFT == tag >> PROBE_TAG_SHIFT;
        } while (!all);
        #pragma unroll
        for (u32 k = 0; k < PROBE_POLL; ++k) before += all ? v[k] ^ tag : 0ull;
    }
    before = wave_sum_u46(before);
    if (__ballot(!all)) before = NONE64;
    if (lane == 0) sh[wave] = before;
    __syncthreads();
    if (sh[0] == NONE64 || sh[1] == NONE64 || sh[2] == NONE64 || sh[3] == NONE64) {
        if (threadIdx.x == 0) mailbox[M_PROBE_GAVE_UP] = 1;
        return;
    }
    u64 base = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    if (last && threadIdx.x == 0) mailbox[0] = base + mine;
    if (!BLOCK_PAIR)
        for (u32 i = 0; i < wave; ++i) base += sh_sum[i];
    if (capacity == 0) return;
    __syncthreads();                // sh and sh_sum have been read
    probe_emit<BLOCK_PAIR>(g, bitmap, p, want, base + incl - want, ppw, list, capacity, sh);
}

// The probe of a short round: every block reads the whole bitmap into LDS and counts all pairs for itself, so nobody waits for
// anybody; the blocks share out the bitmap's words when it comes to the list.  A pair's count is the difference of two entries of a prefix
// sum over the words' bits, whatever the buckets' sizes, and a missing packet's place in the list its pair's plus
// its number less those that arrived.  Latency bounds it: one trip to memory, LDS and three scans, where probe_once tells lengths from block
// to block and takes a pair's list bit by bit.  us until the host has the answer, probe_once and this, by the words of the bitmap:
//                                          2 % lost, all in the list    half lost        nothing arrived
//   256, 4 workers x 64 buckets             17.5, 17.0                   21.6, 16.5       24.8, 16.5
//   678, 3 x 1                              18.0, 16.1                   30.0, 16.0       39.0, 16.1
//   1093, 1 x 161                           17.3, 17.7                   20.4, 17.0       22.6, 17.0
//   2015, 13 x 16                           17.7, 17.0                   23.2, 17.0       27.0, 17.1
//   3992, 8 x 161 (not taken)               18.3, 19.3                   21.8, 19.1       24.9, 19.2
// Above PROBE_ALL_WORDS the usual probe with few losses takes longer, as every block reads all of it.  Below, with 161 buckets and
// few losses, it takes 0.1 to 0.4 us longer too (1093 words 17.7, 18.0; 4 x 161, 1060 words 17.9, 18.2; 8 x 161, 1872 words 18.3, 18.6;
// 499 words 17.6, 17.8; 1952 words 18.1, 17.9; with 16 x 300, 32 x 64 or 13 x 16 buckets 0.2 to 0.7 less): a search of eight steps for the
// bucket of what is missing.  It is taken there all the same, for the 3 to 8 us that it saves where much is lost.
#define PROBE_ALL_THREADS 1024u
#define PROBE_ALL_WORDS 2048u
#define PROBE_ALL_PAIRS 8192u
#define PROBE_ALL_SHARE 16u          // words of the bitmap per block: one a wave
#define PROBE_ALL_LDS(words, B, pairs) (8u * (words) + 4u * ((words) + 1u + (B) + 1u + (pairs)))
__global__ __launch_bounds__(PROBE_ALL_THREADS) void probe_all(Geo g, const u64* __restrict__ bitmap, u32 bound_ppm, u32 n_words, u32 pairs,
                                                               u32* __restrict__ missing_out, u64* __restrict__ list, u64 capacity, u64* __restrict__ mailbox) {
    extern __shared__ __attribute__((aligned(16))) u64 sh_words[];
    u32* const before = (u32*)(sh_words + n_words);         // [n_words + 1]: packets that arrived in the words before
    u32* const fs = before + n_words + 1;                   // [B + 1]
    u32* const place = fs + g.B + 1;                        // [pairs]: where the pair's entries begin; all-ones: it has none
    __shared__ u32 part[PROBE_ALL_THREADS / WAVE];
    const u32 t = threadIdx.x, lane = lane_id(), wave = uniform(t / WAVE), wpw = (u32)g.words_pw;
    #pragma unroll 4
    for (u32 i = t; i < n_words; i += PROBE_ALL_THREADS) sh_words[i] = bitmap[i];
    for (u32 i = t; i <= g.B; i += PROBE_ALL_THREADS) fs[i] = g.first_seq[i];
    __syncthreads();
    // Sum over the threads before this one, and over all.
    auto scan = [&](u32 v, u32* all) {
        const u32 incl = wave_scan_incl<OpAdd>(v);
        if (lane == WAVE - 1) part[wave] = incl;
        __syncthreads();
        u32 own = incl - v, sum = 0;
        for (u32 k = 0; k < PROBE_ALL_THREADS / WAVE; ++k) {
            if (k < wave) own += part[k];
            sum += part[k];
        }
        __syncthreads();
        *all = sum;
        return own;
    };
    u32 total;
    {
        const u32 per = (n_words + PROBE_ALL_THREADS - 1) / PROBE_ALL_THREADS, i0 = t * per;
        u32 n = 0;
        for (u32 i = i0; i < i0 + per && i < n_words; ++i) n += (u32)__popcll(sh_words[i]);
        u32 at = scan(n, &total);
        for (u32 i = i0; i < i0 + per && i < n_words; ++i) { before[i] = at; at += (u32)__popcll(sh_words[i]); }
        if (t == 0) before[n_words] = total;
    }
    __syncthreads();
    // Packets of the workers before w, and of w below number s, that arrived (s may be n_pkts).
    auto arrived = [&](u32 w, u32 s) {
        const u32 i = w * wpw + (s >> 6);
        return before[i] + (s & 63 ? (u32)__popcll(sh_words[i] & ((1ull << (s & 63)) - 1)) : 0u);
    };
    {
        const u32 per = (pairs + PROBE_ALL_THREADS - 1) / PROBE_ALL_THREADS, p0 = t * per;
        u32 n = 0;
        for (u32 pr = p0; pr < p0 + per && pr < pairs; ++pr) {
            const u32 w = pr / g.B, b = pr - w * g.B, n_b = fs[b + 1] - fs[b], miss = n_b - (arrived(w, fs[b + 1]) - arrived(w, fs[b]));
            const u32 want = (u64)miss > ((u64)bound_ppm * n_b) / 1000000ull ? miss : 0u;
            if (missing_out && blockIdx.x == 0) missing_out[pr] = miss;
            place[pr] = want;
            n += want;
        }
        u32 at = scan(n, &total);
        for (u32 pr = p0; pr < p0 + per && pr < pairs; ++pr) {
            const u32 want = place[pr];
            place[pr] = want ? at : NONE32;
            at += want;
        }
    }
    if (blockIdx.x == 0 && t == 0) mailbox[0] = total;
    if (capacity == 0 || total == 0) return;
    __syncthreads();
    // A wave takes a word, a lane a packet: what is missing goes out in order, whatever the number of buckets and losses.
    for (u32 i = blockIdx.x * (PROBE_ALL_THREADS / WAVE) + wave; i < n_words; i += gridDim.x * (PROBE_ALL_THREADS / WAVE)) {
        const u32 w = i / wpw, s = (i - w * wpw) * 64 + lane;
        if (s >= g.n_pkts || (sh_words[i] >> lane) & 1ull) continue;
        u32 b = 0, hi = g.B;
        while (hi - b > 1) { const u32 mid = (b + hi) >> 1; if (fs[mid] <= s) b = mid; else hi = mid; }
        const u32 from = place[w * g.B + b];
        if (from == NONE32) continue;
        const u64 pos = (u64)from + (s - fs[b]) - (arrived(w, s) - arrived(w, fs[b]));
        if (pos < capacity) list[pos] = ((u64)w << 32) | s;
    }
}

// More blocks than probe_once takes, in two launches or three.  Missing packets per pair, list length it asks for (need), and the
// block's total of those.
template <bool BLOCK_PAIR>
__global__ __launch_bounds__(256) void loss_count(Geo g, const u64* __restrict__ bitmap, u32 bound_ppm, u32 ppw, u64 pairs,
                                                  u32* __restrict__ missing_out, u32* __restrict__ need, u64* __restrict__ totals) {
    __shared__ u64 sh[4];
    const u32 lane = lane_id(), wave = uniform(threadIdx.x / WAVE);
    const u64 pr = BLOCK_PAIR ? blockIdx.x : ((u64)blockIdx.x * 4 + wave) * ppw + lane;
    const bool valid = lane < ppw && pr < pairs;
    const ProbePair p(g, pr, valid);
    const u32 got = probe_got<BLOCK_PAIR>(g, bitmap, p, valid, ppw, sh);
    u32 want = 0;
    if (valid && (!BLOCK_PAIR || wave == 0)) {
        u32 miss;
        want = probe_want(p, got, bound_ppm, &miss);
        if (missing_out) missing_out[pr] = miss;
        need[pr] = want;
    }
    const u64 sum = wave_sum_wide(want);
    if (lane == 0) sh[wave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) totals[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// Where blocks are many: exclusive prefix of totals[0..n) in place, by one block of 1024 threads.
#define PROBE_SCAN_BLOCKS 4096u
__global__ __launch_bounds__(1024) void scan_totals(u64* __restrict__ totals, u32 n) {
    __shared__ u64 part[1024];
    const u32 t = threadIdx.x;
    u64 base = 0;
    for (u32 i0 = 0; i0 < n; i0 += 1024) {
        const u64 v = i0 + t < n ? totals[i0 + t] : 0;
        part[t] = v;
        __syncthreads();
        for (u32 d = 1; d < 1024; d <<= 1) {
            const u64 u = t >= d ? part[t - d] : 0;
            __syncthreads();
            part[t] += u;
            __syncthreads();
        }
        if (i0 + t < n) totals[i0 + t] = base + part[t] - v;
        base += part[1023];
        __syncthreads();
    }
}

// The list: block j writes the entries of the pairs that block j of loss_count counted, from the sum of the
// totals before its own on (scanned: totals holds those sums).  The last block tells the host the length.
template <bool BLOCK_PAIR>
__global__ __launch_bounds__(256) void emit_retx(Geo g, const u64* __restrict__ bitmap, u32 ppw, u64 pairs, const u32* __restrict__ need,
                                                 const u64* __restrict__ totals, int scanned, u64* __restrict__ list, u64 capacity,
                                                 u64* __restrict__ mailbox) {
    __shared__ u64 sh[4], sh_sum[4];
    const u32 lane = lane_id(), wave = uniform(threadIdx.x / WAVE);
    const u64 pr = BLOCK_PAIR ? blockIdx.x : ((u64)blockIdx.x * 4 + wave) * ppw + lane;
    const bool valid = lane < ppw && pr < pairs;
    const u32 want = valid ? need[pr] : 0;
    u64 before = 0;
    if (scanned) before = threadIdx.x == 0 ? totals[blockIdx.x] : 0;
    else
        for (u32 i = threadIdx.x; i < blockIdx.x; i += 256) before += totals[i];
    before = wave_sum_u46(before);
    const u32 inc_hi = wave_scan_incl<OpAdd>(want >> 16), inc_lo = wave_scan_incl<OpAdd>(want & 0xFFFFu);
    const u64 incl = ((u64)inc_hi << 16) + inc_lo;
    const u64 sum = ((u64)(u32)__builtin_amdgcn_readlane((int)inc_hi, 63) << 16) + (u32)__builtin_amdgcn_readlane((int)inc_lo, 63);
    if (lane == 0) { sh[wave] = before; sh_sum[wave] = sum; }
    __syncthreads();
    u64 base = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) mailbox[0] = base + (BLOCK_PAIR ? sh_sum[0] : (sh_sum[0] + sh_sum[1]) + (sh_sum[2] + sh_sum[3]));
    if (!BLOCK_PAIR)
        for (u32 i = 0; i < wave; ++i) base += sh_sum[i];
    if (capacity == 0 || sum == 0) return;      // (a block that takes a pair: the same in all its waves)
    if (BLOCK_PAIR) __syncthreads();            // sh has been read
    probe_emit<BLOCK_PAIR>(g, bitmap, ProbePair(g, pr, valid), want, base + incl - want, ppw, list, capacity, sh);
}

// ------------------------------------------------------------------------------------------
// finalize (zero-fill + mean over all W) with fused partial sums of squares; norm reduction
// ------------------------------------------------------------------------------------------
// Per-block partial sums that the last block of the same launch adds up.  words[0] numbers the launches that have used
// the array; block i's sum is two words, tag << 32 | half of the double, stored and loaded as relaxed atomics at device scope.
// The tag comes from device memory, not from the host, so that a launch recorded into a graph can be replayed.
// The wait ends: no block waits before it tells its sum, and one block of a launch, the last, waits.  To keep a block from
// starting, waiting ones of other launches would have to fill its XCD's CUs, eight to a CU, and those another XCD's in
// turn: 16 such launches at once on streams of one CU per XCD, 512 on the whole chip, which runs fewer at a time.
// A second launch for the sum cost 2 to 4 us of the stream (3 workers x 5.3 M, copied out: 103.6 us a pass with it, 102.7 without).
#define PARTIALS_WORDS(blocks) (1u + 2u * (blocks))
__device__ __forceinline__ u32 partials_tag(const u64* words) { return (u32)words[0] + 1u; }
__device__ __forceinline__ void tell_partial(u64* words, u32 i, u32 tag, double v) {
    const u64 bits = (u64)__double_as_longlong(v), t = (u64)tag << 32;
    __hip_atomic_store(&words[1 + 2 * i], t | (u32)bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&words[2 + 2 * i], t | (u32)(bits >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Sum of the n blocks' partials in a fixed order, in every thread.  All 256 threads of the launch's last block; n_max: of any launch.
__device__ __forceinline__ double fold_partials(u64* words, u32 n, u32 tag, u32 n_max, double* wsum) {
    double s = 0.0;
    for (u32 i0 = threadIdx.x; i0 < n; i0 += 4 * 256) {
        u64 lo[4], hi[4];
        bool all;
        do {
            all = true;
            #pragma unroll
            for (u32 k = 0; k < 4; ++k) {
                const u32 i = i0 + k * 256;
                lo[k] = i < n ? __hip_atomic_load(&words[1 + 2 * i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : (u64)tag << 32;
                hi[k] = i < n ? __hip_atomic_load(&words[2 + 2 * i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : (u64)tag << 32;
            }
            #pragma unroll
            for (u32 k = 0; k < 4; ++k) all = all && (u32)(lo[k] >> 32) == tag && (u32)(hi[k] >> 32) == tag;
        } while (!all);
        #pragma unroll
        for (u32 k = 0; k < 4; ++k) s += __longlong_as_double((long long)((hi[k] << 32) | (u32)lo[k]));
    }
    s = wave_sum_f64(s);
    if (lane_id() == 0) wsum[threadIdx.x / WAVE] = s;
    __syncthreads();
    // every block has read words[0] by now.  Before the tags start again from 1, what longer launches left goes.
    if (tag == 0xFFFFFFFFu)
        for (u32 i = threadIdx.x; i < 2 * n_max; i += 256) words[1 + i] = 0;
    if (threadIdx.x == 0) words[0] = tag == 0xFFFFFFFFu ? 0 : tag;
    return (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

// Compensation pass (Alg. "DBLP_RECV" last statements, Alg. "Server" mean).  Per packet span:
//   some worker delivered it   out = src            (scale_mode 0: the gather already divided by W)
//                              out = src / W        (scale_mode 1: W is not a power of two)
//                              where src is the accumulator copy that home[seq] names;
//                              nothing at all when src and out are the same memory and there is
//                              no scaling (in-place form: only moved and missing spans are touched)
//   nobody delivered it        out = 0 exactly
// A wave takes a group of 2^grp_log2 consecutive packets (at most 64: one bitmap word), or one of the
// n_piece pieces of per_piece elements of its range.  Consecutive packets are consecutive elements,
// across bucket boundaries too, so a group that arrived whole and lives in one copy is a plain copy of its
// range in aligned 16-byte units, four in flight per lane (PAST: eight, and past the caches); other groups go run by run.  Memory bounds
// it; a wave's share is bounded in elements because with 8 packets per wave, whatever their length, a round
// of long packets had a few hundred waves, and groups that cross a bucket went element by element:
//   3 workers x 15.5 M in 64 KB packets    568 -> 27 us
//   3 x 5.3 M, 1472 B (2 x 21 MB moved)     23 -> 13 us
//   8 x 215 M, 1472 B (2 x 862 MB moved)   443 -> 387 us
// move_home (in-place form, n_piece = 1): the homes of spans that were moved are reset to copy 0.
// With scale_mode 1 the per-block sums of out^2 go to `partials`.  Otherwise the sum of squares is already known: the
// gather kernels kept it per block in sumsq_rows, and that of batches gathered by a list (`listed`) in the long accumulators before the
// bitmap.  The one extra block of this launch (blockIdx.x == n_work_blocks) adds
// up the one or the other in an order that the sizes of the round's batches fix, not that of the arrivals, and
// writes the total to the host mailbox.
template <bool TABLE_IN_LDS, bool PAST>
__global__ __launch_bounds__(256) void finalize_pass(Geo g, const u64* __restrict__ bitmap, const float* acc0,
                                                     const float* acc1, uint8_t* __restrict__ home,
                                                     float* out, int scale_mode, float wf, int move_home,
                                                     u32 grp_log2, u32 n_piece, u32 per_piece, u64* partials, u32 n_max, u32 n_work_blocks,
                                                     const double* __restrict__ sumsq_rows, const u64* __restrict__ accept_rows,
                                                     u32 n_rows, u32 listed,
                                                     u64* __restrict__ counters, u64* __restrict__ mailbox, RoundState other) {
    __shared__ double wsum[4];
    __shared__ u64 asum[4];
    __shared__ u64 lsum[4][LONG_PITCH];
    extern __shared__ u32 fs_lds[];             // bucket boundaries (B + 1 words) when TABLE_IN_LDS
    const u32 lane = lane_id();
    const u32 wave_in_block = threadIdx.x / WAVE;
    if (blockIdx.x >= n_work_blocks) {
        // the extra block: fixed-order sum of the gather's rows (sum of squares for Eq. 1, accepted
        // packets), and the round's counters mirrored into the host mailbox:
        // mailbox[1] = sum of squares, mailbox[8..11] = accepted,
        // candidates, stale, invalid
        // Only the n_rows rows that a launch of this round can have written are read; the rest are zero.
        double s = 0.0;
        u64 a = 0, l = 0;                                   // l: word lane % LONG_PITCH of the thread's accumulators
        #pragma unroll
        for (u32 i = 0; i < LONG_ALL; i += 256) l += listed ? bitmap[(int)(i + threadIdx.x) - (int)LONG_ALL] : 0ull;
        for (u32 i0 = 0; i0 < n_rows; i0 += 4 * 256) {      // four independent loads of each kind in flight
            double sv[4]; u64 av[4];
            #pragma unroll
            for (u32 j = 0; j < 4; ++j) {
                const u32 i = i0 + j * 256 + threadIdx.x;
                sv[j] = i < n_rows ? sumsq_rows[i] : 0.0;
                av[j] = i < n_rows ? accept_rows[i] : 0ull;
            }
            #pragma unroll
            for (u32 j = 0; j < 4; ++j) { s += sv[j]; a += av[j]; }
        }
        s = wave_sum_f64(s);
        const u32 a_lo = wave_reduce<OpAdd>((u32)(a & 0xFFFFFu)), a_hi = wave_reduce<OpAdd>((u32)(a >> 20));   // 64 x 2^20 fits 32 bits
        if (lane == 0) { wsum[wave_in_block] = s; asum[wave_in_block] = ((u64)a_hi << 20) + a_lo; }
        l += lane_value(l, lane ^ LONG_PITCH);
        if (lane < LONG_PITCH) lsum[wave_in_block][lane] = l;
        __syncthreads();
        double total = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
        if (listed && wave_in_block == 0) {
            // The words as doubles, as exact as their size allows (below 2^53 they are), added up.
            const long long word = lane < LONG_WORDS ? (long long)((lsum[0][lane] + lsum[1][lane]) + (lsum[2][lane] + lsum[3][lane])) : 0;
            total += wave_sum_f64(ldexp((double)word, (int)(32 * lane) - LONG_SHIFT));
        }
        if (scale_mode) {
            __syncthreads();
            total = fold_partials(partials, n_work_blocks, partials_tag(partials), n_max, wsum);
        }
        if (threadIdx.x == 0) {
            const u64 accepted = (asum[0] + asum[1]) + (asum[2] + asum[3]);
            counters[C_ACCEPTED] = accepted;
            ((double*)mailbox)[1] = total;
            mailbox[8] = accepted; mailbox[9] = counters[C_CANDIDATES];
            mailbox[10] = counters[C_STALE]; mailbox[11] = counters[C_INVALID];
        }
        return;
    }
    if (other.bitmap) {         // the state of the next round
        const u64 n_words = LONG_ALL + (u64)g.W * g.words_pw, n = n_words + 2 * other.rows_used, first = (u64)blockIdx.x * blockDim.x + threadIdx.x;
        u64* const words = other.bitmap - LONG_ALL;
        for (u64 i = first; i < n; i += (u64)n_work_blocks * blockDim.x) {
            const u64 r = i - n_words;
            if (i < n_words) words[i] = 0;
            else other.rows[r < other.rows_used ? r : r - other.rows_used + ACCEPT_ROWS] = 0;
        }
        if (first < C_COUNT) other.counters[first] = 0;
    }
    const u32 wave = blockIdx.x * (blockDim.x / WAVE) + wave_in_block;
    const u32 n_waves = n_work_blocks * (blockDim.x / WAVE);
    const u32 grp = 1u << grp_log2;
    const u64 n_items = (((u64)g.n_pkts + grp - 1) >> grp_log2) * n_piece;
    // An item's workers' bitmap words (lane w loads worker w's: one load instruction for the wave, W <= 64) and
    // the copies of its packets (meaningful where they arrived).  The first item's are on their way while the table is.
    u32 gi = 0, piece = 0, seq0 = 0, n_t = 0, hm = 0;
    u64 mine = 0;
    auto fetch = [&](u64 item) {
        if (item >= n_items) return;
        gi = n_piece == 1 ? (u32)item : (u32)(item / n_piece);
        piece = (u32)(item - (u64)gi * n_piece);
        seq0 = gi << grp_log2;
        n_t = g.n_pkts - seq0 < grp ? g.n_pkts - seq0 : grp;
        mine = lane < g.W ? bitmap[(u64)lane * g.words_pw + (seq0 >> 6)] : 0ull;
        hm = lane < n_t ? home[seq0 + lane] : 0;
    };
    fetch(wave);
    const u32* fs = g.first_seq;
    if (TABLE_IN_LDS) {
        for (u32 i = threadIdx.x; i <= g.B; i += blockDim.x) fs_lds[i] = g.first_seq[i];
        __syncthreads();
        fs = fs_lds;
    }
    const bool skip_same = scale_mode == 0;     // a span that already sits in `out` needs no copy
    double dsum = 0.0;

    // Elements [e0, e1) of the result by the whole wave: src / W, src, or zeros where src is null.
    auto write_range = [&](const float* src, u64 e0, u64 e1) {
        auto scaled = [&](f4v v) {
            if (scale_mode) {
                v.x = v.x / wf; v.y = v.y / wf; v.z = v.z / wf; v.w = v.w / wf;
                dsum += (double)((v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w));
            }
            return v;
        };
        const u64 up = (e0 + 3) & ~3ull, a0 = up < e1 ? up : e1, a1 = (e1 & ~3ull) > a0 ? e1 & ~3ull : a0;
        if (lane < (u32)(a0 - e0) || (lane >= 32 && lane - 32 < (u32)(e1 - a1))) {      // what lies outside whole 16-byte units
            const u64 e = lane < 32 ? e0 + lane : a1 + (lane - 32);
            f4v v = {src ? src[e] : 0.f, 0.f, 0.f, 0.f};
            if (src) v = scaled(v);
            out[e] = v.x;
        }
        u64 c = (a0 >> 2) + lane;
        const u64 c1 = a1 >> 2;
        f4v* o = (f4v*)out;
        const f4v zero = {0.f, 0.f, 0.f, 0.f};
        if (!src) {
            for (; c < c1; c += WAVE) o[c] = zero;
            return;
        }
        const f4v* s = (const f4v*)src;
        constexpr int R = PAST ? 8 : 4;             // units in flight per lane
        for (; c < c1; c += R * WAVE) {
            f4v v[R];
            #pragma unroll
            for (int k = 0; k < R; ++k) {
                v[k] = zero;
                if (c + k * WAVE < c1) v[k] = PAST ? __builtin_nontemporal_load(s + c + k * WAVE) : s[c + k * WAVE];
            }
            #pragma unroll
            for (int k = 0; k < R; ++k) {
                if (c + k * WAVE >= c1) break;
                const f4v r = scaled(v[k]);
                if (PAST) __builtin_nontemporal_store(r, o + c + k * WAVE);
                else o[c + k * WAVE] = r;
            }
        }
    };

    for (u64 item = wave; item < n_items; item += n_waves, fetch(item)) {
        const u64 full = NONE64 >> (64 - n_t);
        const u64 any = uniform(((((u64)wave_reduce<OpOr>((u32)(mine >> 32)) << 32) | wave_reduce<OpOr>((u32)mine)) >> (seq0 & 63)) & full);
        const u64 second = (u64)__ballot(hm & 1u);
        // the packets that need work at all
        const u64 same = skip_same ? (acc0 == out ? ~second : 0ull) | (acc1 == out ? second : 0ull) : 0ull;
        const u64 todo = uniform(full & ~(any & same));
        if (!todo) continue;
        u64 elem_l = 0;
        u32 len_l = 0;
        if (lane < n_t) {
            const u32 b = find_bucket(g, fs, seq0 + lane);
            const u64 start = (u64)(seq0 + lane - fs[b]) * g.P, left = g.b_cnt[b] - start;
            elem_l = g.b_off[b] + start;
            len_l = left < g.P ? (u32)left : g.P;
        }
        auto elem_of = [&](u32 t) {
            return ((u64)(u32)__builtin_amdgcn_readlane((int)(u32)(elem_l >> 32), (int)t) << 32) | (u32)__builtin_amdgcn_readlane((int)(u32)elem_l, (int)t);
        };
        const u64 g0 = elem_of(0), g1 = elem_of(n_t - 1) + (u32)__builtin_amdgcn_readlane((int)len_l, (int)(n_t - 1));
        const u64 p0 = g0 + (u64)piece * per_piece, p1 = n_piece == 1 || p0 + per_piece > g1 ? g1 : p0 + per_piece;
        if (p0 >= p1) continue;
        if (todo == full && any == full && ((second & full) == 0 || (second & full) == full)) {
            write_range((second & 1ull) ? acc1 : acc0, p0, p1);
            if (move_home && (second & 1ull) && lane < n_t) home[seq0 + lane] = 0;
            continue;
        }
        for (u64 m = todo; m;) {                                // runs of packets of one kind
            const u32 t = (u32)__builtin_ctzll(m);
            const u64 kind = uniform(m & (!((any >> t) & 1ull) ? ~any : ((second >> t) & 1ull) ? any & second : any & ~second));
            const u64 after = ~(kind >> t);                     // bit k: packet t + k is of another kind
            const u32 n = after ? (u32)__builtin_ctzll(after) : 64 - t, z = t + n - 1;
            m &= z == 63 ? 0ull : NONE64 << (z + 1);
            const u64 e0 = elem_of(t), e1 = elem_of(z) + (u32)__builtin_amdgcn_readlane((int)len_l, (int)z);
            const u64 lo = e0 > p0 ? e0 : p0, hi = e1 < p1 ? e1 : p1;
            if (lo >= hi) continue;
            write_range(!((any >> t) & 1ull) ? nullptr : ((second >> t) & 1ull) ? acc1 : acc0, lo, hi);
        }
        // in-place form: the spans that were moved now live in copy 0
        if (move_home && lane < n_t && ((any >> lane) & 1ull) && (hm & 1u)) home[seq0 + lane] = 0;
    }
    if (scale_mode) {
        dsum = wave_sum_f64(dsum);
        if (lane == 0) wsum[wave_in_block] = dsum;
        __syncthreads();
        if (threadIdx.x == 0) tell_partial(partials, blockIdx.x, partials_tag(partials), (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]));
    }
}

// Sum of squares of a plain vector (16-byte aligned).  Memory bounds it.  A block reads runs of SQ_RUN x 4 KB, all
// loads of a run in flight, with the non-temporal hint, and two blocks per CU are enough: fewer DRAM rows are open at a time
// than with eight blocks that read 4 KB here and there.  us (TB/s), before and now: 25.6 M floats 19.9, 18.4 (5.1, 5.6);
// 124 M 79.6, 72.8 (6.3, 6.8); 1000 M 642, 554 (6.2, 7.2); runs of 8 and 16 with as many blocks 75.4 and 77.5 at 124 M, four
// blocks per CU 74.6, eight 75.7.
#define SQ_RUN 4
#define SQ_BLOCKS_PER_CU 2
__device__ __forceinline__ double vec_sumsq(const float* __restrict__ v, u64 n) {
    const u64 n4 = n / 4;
    const f4v* v4 = (const f4v*)v;
    double dsum = 0.0;
    auto add = [&](f4v x) { dsum += (double)((x.x * x.x + x.y * x.y) + (x.z * x.z + x.w * x.w)); };
    for (u64 u0 = (u64)blockIdx.x * (SQ_RUN * 256); u0 < n4; u0 += (u64)gridDim.x * (SQ_RUN * 256)) {
        const u64 u = u0 + threadIdx.x;
        if (u0 + SQ_RUN * 256 <= n4) {
            f4v x[SQ_RUN];
            #pragma unroll
            for (int k = 0; k < SQ_RUN; ++k) x[k] = __builtin_nontemporal_load(v4 + u + k * 256);
            #pragma unroll
            for (int k = 0; k < SQ_RUN; ++k) add(x[k]);
        } else
            for (int k = 0; k < SQ_RUN; ++k)
                if (u + k * 256 < n4) add(v4[u + k * 256]);
    }
    if (blockIdx.x == 0 && threadIdx.x < (u32)(n - 4 * n4)) {
        const float x = v[4 * n4 + threadIdx.x];
        dsum += (double)(x * x);
    }
    return wave_sum_f64(dsum);
}

// The sum of squares to the host mailbox: the launch's last block adds the blocks' sums up.
__global__ __launch_bounds__(256) void sumsq_vec(const float* __restrict__ v, u64 n, u64* partials, u32 n_max, double* __restrict__ mailbox) {
    __shared__ double wsum[4];
    const u32 tag = partials_tag(partials);
    const double w = vec_sumsq(v, n);
    if (lane_id() == 0) wsum[threadIdx.x / WAVE] = w;
    __syncthreads();
    if (threadIdx.x == 0) tell_partial(partials, blockIdx.x, tag, (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]));
    if (blockIdx.x != gridDim.x - 1) return;
    __syncthreads();
    const double total = fold_partials(partials, gridDim.x, tag, n_max, wsum);
    if (threadIdx.x == 0) mailbox[0] = total;
}

// The same in two launches, for calls without a context, whose words no call owns: sums per block, and their sum in the order of
// fold_partials.  (Calls on one GPU share the array of sums, and the caller orders them.)
__global__ __launch_bounds__(256) void sumsq_blocks(const float* __restrict__ v, u64 n, double* __restrict__ partials) {
    __shared__ double wsum[4];
    const double w = vec_sumsq(v, n);
    if (lane_id() == 0) wsum[threadIdx.x / WAVE] = w;
    __syncthreads();
    if (threadIdx.x == 0) partials[blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}
__global__ __launch_bounds__(256) void reduce_partials(const double* __restrict__ partials, u32 n, double* __restrict__ out) {
    __shared__ double wsum[4];
    double s = 0.0;
    for (u32 i = threadIdx.x; i < n; i += 256) s += partials[i];
    s = wave_sum_f64(s);
    if (lane_id() == 0) wsum[threadIdx.x / WAVE] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

// Blocks of a sum of squares over n floats: a rule of the size alone, so that all entry points add in the same order.
static u32 sumsq_grid(u32 cus, u64 n) {
    const u64 runs = (n / 4 + SQ_RUN * 256 - 1) / (SQ_RUN * 256), most = (u64)cus * SQ_BLOCKS_PER_CU;
    return (u32)(runs == 0 ? 1 : runs < most ? runs : most);
}

// ------------------------------------------------------------------------------------------
// where to write: measuring a buffer against the accumulator copies
// ------------------------------------------------------------------------------------------
// On this chip a stream of payload reads with a few percent of result writes mixed in runs about
// 15 % slower when the reads and the writes fall into the same third of the HBM address space
// than when they fall into different thirds (measured with this very loop: 1.60 vs 1.39 ms per
// 8.5 GB; which third a buffer lies in cannot be asked for, only measured).  The library
// therefore keeps two copies of the accumulator in different thirds when it can, and sends the
// spans a batch writes for the first time to the copy that is faster for that batch's buffer.
//
// The loop below has the access pattern of the gather (CLS_STREAMS streams of 1472-byte pieces,
// each wave sums one piece per stream and stores the 1472-byte result): a plain linear copy does
// not show the effect.  It reads CLS_SAMPLE_BYTES from src and writes CLS_SCRATCH_BYTES.
#define CLS_STREAMS 32u
#define CLS_PIECE 1472u
#define CLS_SEQS 22795u
#define CLS_SAMPLE_BYTES ((u64)CLS_STREAMS * CLS_SEQS * CLS_PIECE)      /* 1.07 GB */
#define CLS_SCRATCH_BYTES ((u64)CLS_SEQS * CLS_PIECE)                    /* 33.6 MB */
__global__ __launch_bounds__(256) void classify_rw(const uint8_t* __restrict__ src, float* __restrict__ scratch) {
    const u32 lane = lane_id();
    const u32 wave = (blockIdx.x * 256 + threadIdx.x) / WAVE, n_waves = gridDim.x * 4;
    const bool second = lane < CLS_PIECE / 16 - WAVE;            // 92 units per piece: lanes 0..27 take two
    for (u32 seq = wave; seq < CLS_SEQS; seq += n_waves) {
        f4v a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
        for (u32 w0 = 0; w0 < CLS_STREAMS; w0 += 4) {
            f4v v0[4], v1[4];
            #pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint8_t* b = src + ((u64)(w0 + j) * CLS_SEQS + seq) * CLS_PIECE + 16ull * lane;
                v0[j] = __builtin_nontemporal_load((const f4v*)b);
                v1[j] = f4v{0.f, 0.f, 0.f, 0.f};
                if (second) v1[j] = __builtin_nontemporal_load((const f4v*)(b + 1024));
            }
            #pragma unroll
            for (int j = 0; j < 4; ++j) { a0 += v0[j]; a1 += v1[j]; }
        }
        f4v* d = (f4v*)(scratch + (u64)seq * (CLS_PIECE / 4)) + lane;
        *d = a0;
        if (second) d[WAVE] = a1;
    }
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
// What the context's gather_burst launches are given (burst_plan); fn null: none are made.
typedef void (*burst_fn)(Geo, const uint8_t*, u64*, u64*, float*, float*, uint8_t*, u32, const u32*, u32, u64*, u64*, double*, float,
                         u32, u32, u32, u32, u32, u32, u32, u32, u64*);
struct BurstPlan { burst_fn fn; u32 kb, r_max, r_step, n_piece, table_at, image_at, min_seq, through_seq; size_t lds; };

struct dblp_ctx {
    Geo g;
    BurstPlan burst;
    u64 N;
    double eta;
    int device;
    hipStream_t stream;
    int n_cus;
    // device state
    u64* slab;              // what follows, but for the hints and the accumulator
    u32* d_hint;
    RoundState state[2];    // the open round's (cur) and the other one
    int cur;
    int other_clean;        // the state that is not in use is all zero, once what has been launched has ended
    int recorded;           // calls were recorded into a graph, which holds the addresses of one state: it stays in use
    u64* d_pending; u64* d_flags;   // F_COUNT words
    ArrivalList few; u64 max_few;   // arrivals of a batch that gather_few takes, at most
    u32 any_no;             // batches that used one of the first two
    // accumulator: one or two copies (d_acc[1] == d_acc[0] when there is one); each copy's
    // allocation ends with CLS_SCRATCH_BYTES that classify_rw may overwrite
    void* acc_alloc[2]; float* d_acc[2]; float* d_scratch[2];
    int n_acc;              // 1 or 2
    int acc_caller;         // the copies are the caller's buffers: never measured, never freed
    int acc_distinct;       // the two copies were measured to lie in different thirds of HBM
    float place_ms[2];      // that measurement: probe time writing to copy 0 / copy 1 (0 = not taken)
    int place_steps;        // candidates tried by the placement search
    double place_seconds;   // time the search took
    double search_fraction; // share of the free memory the search may hold
    double search_seconds;  // its time limit
    int fold;               // W is a power of two: the gather stores sum / W
    int counters_in_mailbox; // the last finalize left the round's counters in the host mailbox (until the next batch or round)
    int mailbox_seen;       // the stream has been synchronised since that finalize
    int acc_policy;         // DBLP_ACC_*
    int last_pick;          // copy the last batch wrote new spans to
    u32 batch_no;
    uint8_t* d_home;        // [n_pkts rounded up to 8] copy that holds each packet's span
    struct Picked { const void* p; u64 bytes; int pick; } picked[32];   // measured buffers
    u32 n_picked;
    hipEvent_t cls_ev[2];
    int probe_all;          // probe: by probe_all
    int probe_block_pair;   // else: a block per (worker, bucket) pair
    u32 probe_no;           // probes made: what their words in d_totals are told apart by
    u32 probe_polls;        // looks that a block of probe_once takes at the totals before its own
    u32* d_need; u64* d_totals;   // list length per pair, and per block of pairs
    u64* d_partials; u32 max_partials;    // sums of squares per block, told to the launch's last block
    u32* d_block_tallies;   // [IDX_BLOCKS_PER_CU * n_cus][5], written by index_arrivals
    int result_in_place;    // the form of the last dblp_finalize (in place until one says otherwise): prices the second copy
    u64* h_mailbox;         // pinned host memory, 16 x u64, also mapped into the device
    u64* d_mailbox;         // device address of h_mailbox
    // host copies of the geometry
    u32* h_first_seq; u64* h_b_off; u64* h_b_cnt;
    u64* h_tables;          // the three as they lie on the device, while dblp_create copies them there
    // protocol state
    int round_open; int finalized; uint16_t round;
    double prev_norm; int have_prev;
    // optional per-kernel timing (HIP events on the context's stream)
    int profiling;          // bit k set: launches of kernel group k are bracketed by events
    struct Timed { hipEvent_t a, b; int kernel; u32 told; bool burst; };     // kernel < 0: minus the wanted groups; h_told[told] says which
    std::vector<Timed>* timed;        // recorded, not yet read
    u32* h_told; u32* d_told;         // mapped host memory: a gather launch that decides on the device tells here what it was (TOLD_*)
    u32 n_told;                       // entries in use, by records not yet read
    u64 n_burst;                      // of the dense gathers last read: those in bursts
    std::vector<hipEvent_t>* ev_pool; // free events
    char err[256];
};

static hipEvent_t prof_event(dblp_ctx* c) {
    hipEvent_t e = nullptr;
    if (!c->ev_pool->empty()) { e = c->ev_pool->back(); c->ev_pool->pop_back(); }
    else if (hipEventCreate(&e) != hipSuccess) { (void)hipGetLastError(); e = nullptr; }
    return e;
}

#define PROF_MAX_RECORDS 16384   // brackets kept between two dblp_profile_read calls; more are dropped

// Brackets one kernel launch with events when profiling is on.  `told`: the launch decides on the device whether it
// is a dense or a sparse gather, so the bracket's group is known when it is read.
struct ProfScope {
    dblp_ctx* c; hipEvent_t a; int kernel; u32 at; bool burst;
    ProfScope(dblp_ctx* c_, int kernel_, bool told = false, bool burst_ = false) : c(c_), a(nullptr), kernel(kernel_), at(0), burst(burst_) {
        const int want = c->profiling & (told ? 1 << DBLP_K_GATHER | 1 << DBLP_K_GATHER_DIRECT : 1 << kernel);
        if (!want || (told && c->n_told >= PROF_MAX_RECORDS)) return;
        if (!(a = prof_event(c))) return;
        if (told) { kernel = -want; at = c->n_told++; }
        (void)hipEventRecord(a, c->stream);
    }
    u32* d_told() const { return a && kernel < 0 ? c->d_told + at : nullptr; }
    ~ProfScope() { end(); }
    void end() {                // before a wait that is no part of the launches
        if (!a) return;
        hipEvent_t b = prof_event(c);
        if (!b) { c->ev_pool->push_back(a); a = nullptr; return; }
        (void)hipEventRecord(b, c->stream);
        if (c->timed->size() < c->timed->capacity()) c->timed->push_back({a, b, kernel, at, burst});   // never reallocates
        else { c->ev_pool->push_back(a); c->ev_pool->push_back(b); }                            // buffer full: drop the sample
        a = nullptr;
    }
};

static int fail(dblp_ctx* c, int code, const char* what) {
    if (c) snprintf(c->err, sizeof c->err, "%s", what);
    return code;
}

static int fail_hip(dblp_ctx* c, hipError_t e, const char* what) {
    if (c) snprintf(c->err, sizeof c->err, "%s: %s", what, hipGetErrorString(e));
    return DBLP_EHIP;
}

#define HIP_TRY(c, call)                                            \
    do {                                                            \
        hipError_t e__ = (call);                                    \
        if (e__ != hipSuccess) return fail_hip((c), e__, #call);    \
    } while (0)

#define LAUNCH_CHECK(c, name)                                       \
    do {                                                            \
        hipError_t e__ = hipGetLastError();                         \
        if (e__ != hipSuccess) return fail_hip((c), e__, name);     \
    } while (0)

static u32 grid_for(const dblp_ctx* c, u64 blocks_wanted, u32 blocks_per_cu) {
    u64 cap = (u64)c->n_cus * blocks_per_cu;
    u64 g = blocks_wanted < cap ? blocks_wanted : cap;
    return (u32)(g ? g : 1);
}

extern "C" const char* dblp_last_error(const dblp_ctx* ctx) { return ctx ? ctx->err : "null context"; }

extern "C" int dblp_destroy(dblp_ctx* c) {
    if (!c) return DBLP_OK;
    (void)hipSetDevice(c->device);
    (void)hipStreamSynchronize(c->stream);
    void* dev[] = {c->slab, c->d_hint, c->acc_caller ? nullptr : c->acc_alloc[0], c->acc_caller ? nullptr : c->acc_alloc[1]};
    for (void* p : dev) if (p) (void)hipFree(p);
    for (hipEvent_t e : c->cls_ev) if (e) (void)hipEventDestroy(e);
    if (c->h_mailbox) (void)hipHostFree(c->h_mailbox);
    if (c->h_told) (void)hipHostFree(c->h_told);
    if (c->timed) { for (auto& t : *c->timed) { (void)hipEventDestroy(t.a); (void)hipEventDestroy(t.b); } delete c->timed; }
    if (c->ev_pool) { for (auto e : *c->ev_pool) (void)hipEventDestroy(e); delete c->ev_pool; }
    free(c->h_first_seq); free(c->h_b_off); free(c->h_b_cnt); free(c->h_tables);
    free(c);
    return DBLP_OK;
}

// Milliseconds of classify_rw reading src and writing scratch (best of two after one untimed run), < 0 on error.
static float time_rw(dblp_ctx* c, const void* src, float* scratch) {
    for (hipEvent_t& e : c->cls_ev)
        if (!e && hipEventCreate(&e) != hipSuccess) { (void)hipGetLastError(); e = nullptr; return -1.f; }
    float best = -1.f;
    for (int r = 0; r < 3; ++r) {
        if (hipEventRecord(c->cls_ev[0], c->stream) != hipSuccess) return -1.f;
        hipLaunchKernelGGL(classify_rw, dim3(4 * c->n_cus), dim3(256), 0, c->stream, (const uint8_t*)src, scratch);
        if (hipEventRecord(c->cls_ev[1], c->stream) != hipSuccess) return -1.f;
        if (hipEventSynchronize(c->cls_ev[1]) != hipSuccess) return -1.f;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, c->cls_ev[0], c->cls_ev[1]) != hipSuccess) return -1.f;
        if (r > 0 && (best < 0.f || ms < best)) best = ms;
    }
    return best;
}

// (Re)allocates the library-owned accumulator as `copies` copies.  place != 0: search for a second
// copy in another third of the HBM address space than the first, within the context's limits
// (share of the free memory held at once, seconds), and have no second copy if none is found.
// The contents of the round in progress are lost.
#define PLACE_MAX_STEPS 40
#define PLACE_STRIDE_BYTES (6ull << 30)
static double wall_seconds() {
    struct timespec ts;
    clock_gettime(CLOCK_MONOTONIC, &ts);
    return (double)ts.tv_sec + 1e-9 * (double)ts.tv_nsec;
}

static int set_accumulator_copies(dblp_ctx* c, int copies, int place) {
    if (hipStreamSynchronize(c->stream) != hipSuccess) return fail(c, DBLP_EHIP, "accumulator_copies: synchronize");
    for (int i = 0; i < 2; ++i) { if (c->acc_alloc[i]) (void)hipFree(c->acc_alloc[i]); c->acc_alloc[i] = nullptr; }
    c->n_acc = 1; c->acc_distinct = 0; c->place_ms[0] = c->place_ms[1] = 0.f; c->place_steps = 0; c->place_seconds = 0.0;
    c->n_picked = 0; c->last_pick = 0; c->round_open = 0; c->finalized = 0; c->counters_in_mailbox = 0;
    const size_t bytes = (c->N * sizeof(float) + 255) / 256 * 256;     // the scratch area starts aligned
    const size_t scratch = copies == 2 ? CLS_SCRATCH_BYTES : 0;
    if (hipMalloc(&c->acc_alloc[0], bytes + scratch) != hipSuccess) { (void)hipGetLastError(); return fail(c, DBLP_ENOMEM, "accumulator"); }
    c->d_acc[0] = c->d_acc[1] = (float*)c->acc_alloc[0];
    c->d_scratch[0] = c->d_scratch[1] = (float*)((uint8_t*)c->acc_alloc[0] + bytes);
    if (copies != 2) return DBLP_OK;
    auto adopt = [&](void* p) {
        c->acc_alloc[1] = p; c->n_acc = 2;
        c->d_acc[1] = (float*)p; c->d_scratch[1] = (float*)((uint8_t*)p + bytes);
    };
    if (!place) {
        void* p = nullptr;
        if (hipMalloc(&p, bytes + scratch) == hipSuccess) adopt(p); else (void)hipGetLastError();
        return DBLP_OK;
    }
    // Walk through the free memory: candidate, then a holder allocation that pushes the next
    // candidate further on, until a candidate measures differently from the first copy against
    // the same read buffer, or the share of the free memory that may be held is reached, or time
    // is up.  What the probe reads: a buffer allocated right after the first copy (next to its
    // end, where the scratch area that the reference measurement writes lies).
    const double t_start = wall_seconds();
    void* near0 = nullptr;
    if (hipMalloc(&near0, CLS_SAMPLE_BYTES) != hipSuccess) { (void)hipGetLastError(); return DBLP_OK; }
    const void* rd = near0;
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) { (void)hipGetLastError(); free_b = 0; }
    const size_t may_hold = (size_t)((double)free_b * c->search_fraction);
    const float t_ref = time_rw(c, rd, c->d_scratch[0]);
    c->place_ms[0] = t_ref > 0.f ? t_ref : 0.f;
    void* held[2 * PLACE_MAX_STEPS];
    int n_held = 0;
    size_t held_bytes = 0;
    for (int step = 0; step < PLACE_MAX_STEPS && t_ref > 0.f; ++step) {
        if (held_bytes + bytes + scratch > may_hold) break;
        if (wall_seconds() - t_start > c->search_seconds) break;
        void* cand = nullptr;
        if (hipMalloc(&cand, bytes + scratch) != hipSuccess) { (void)hipGetLastError(); break; }
        // both ends of the candidate must differ from the first copy, and in the same direction
        // (a candidate that straddles two thirds is passed over); its contents are scratch here
        const float t_end = time_rw(c, rd, (float*)((uint8_t*)cand + bytes));
        const float t_beg = bytes >= CLS_SCRATCH_BYTES ? time_rw(c, rd, (float*)cand) : t_end;
        auto differs = [&](float t) { const float hi = t > t_ref ? t : t_ref; return t > 0.f && fabsf(t - t_ref) > 0.07f * hi; };
        c->place_ms[1] = t_end > 0.f ? t_end : 0.f;
        c->place_steps = step + 1;
        if (differs(t_end) && differs(t_beg) && (t_end < t_ref) == (t_beg < t_ref)) { adopt(cand); c->acc_distinct = 1; break; }
        held[n_held++] = cand; held_bytes += bytes + scratch;
        if (held_bytes + PLACE_STRIDE_BYTES > may_hold) break;
        void* holder = nullptr;
        if (hipMalloc(&holder, PLACE_STRIDE_BYTES) != hipSuccess) { (void)hipGetLastError(); break; }
        held[n_held++] = holder; held_bytes += PLACE_STRIDE_BYTES;
    }
    for (int i = 0; i < n_held; ++i) (void)hipFree(held[i]);
    (void)hipFree(near0);
    (void)hipGetLastError();
    c->place_seconds = wall_seconds() - t_start;
    return DBLP_OK;
}

// Which copy the spans that this batch writes first should go to.  Never allocates.  Measures
// (and then waits for its probe kernel) only under the automatic policy on a context with two
// library-owned copies, once per large packet buffer.
static int pick_copy(dblp_ctx* c, const void* d_packets, u64 bytes, u64 n_slots, u64 n_arrivals) {
    if (c->n_acc < 2) return 0;
    switch (c->acc_policy) {
    case DBLP_ACC_FIRST: return 0;
    case DBLP_ACC_SECOND: return 1;
    case DBLP_ACC_ALTERNATE: return (int)(c->batch_no & 1u);
    default: break;
    }
    // automatic: measure the buffer once; small or thinly used buffers are not worth it, and
    // caller-owned copies have no scratch area to write to
    if (c->acc_caller || bytes < CLS_SAMPLE_BYTES || n_arrivals < n_slots / 8) return 0;
    for (u32 i = 0; i < c->n_picked; ++i)
        if (c->picked[i].p == d_packets && c->picked[i].bytes == bytes) return c->picked[i].pick;
    const u64 last = (bytes - CLS_SAMPLE_BYTES) & ~15ull;
    const u64 offs[3] = {0, (last / 2) & ~15ull, last};
    const int n_offs = bytes >= 3 * CLS_SAMPLE_BYTES ? 3 : 1;
    auto measure = [&](float* scratch) {           // summed over the sample positions, < 0 on error
        float sum = 0.f;
        for (int i = 0; i < n_offs; ++i) {
            const float ms = time_rw(c, (const uint8_t*)d_packets + offs[i], scratch);
            if (ms < 0.f) { (void)hipGetLastError(); return -1.f; }
            sum += ms;
        }
        return sum;
    };
    const float t0 = measure(c->d_scratch[0]);
    if (t0 < 0.f) return 0;
    const float t1 = measure(c->d_scratch[1]);
    // The second copy has to be that much faster: 3 % when the result is copied out of the
    // accumulator anyway; when it is left in place, spans written to the second copy are moved to
    // the first by finalize (8 bytes per element, at about two thirds of the gather's rate, against
    // the 4 W (1 + 2/P) + 4 bytes per element that the gather moves).
    float margin = 0.03f;
    if (c->result_in_place) {
        const float gather_bytes = 4.f * (float)c->g.W * (1.f + 2.f / (float)c->g.P) + 4.f;
        margin += 1.5f * 8.f / gather_bytes;
    }
    const int pick = t1 > 0.f && t1 < (1.f - margin) * t0 ? 1 : 0;
    dblp_ctx::Picked& slot = c->picked[c->n_picked < 32 ? c->n_picked++ : c->batch_no % 32];
    slot.p = d_packets; slot.bytes = bytes; slot.pick = pick;
    return pick;
}

#define FIN_BLOCKS_PER_CU 8
// Elements from which a copy goes past the caches, eight units in flight per lane: what a large gradient's lines would displace is
// worth more than they are, and the mean is read again only once it has all been written.  us of a pass that copies out, and in
// brackets with a kernel that reads the mean behind it, before and now: 3 x 22 M elements 187, 177 (222, 214); 13 x 22 M 336, 332 (372, 365); 1 x 60 M
// 242, 215 (316, 303); 1 x 137 M 583, 526 (778, 714); 3 x 200 M 1000, 983 (1266, 1253).  Below, the caches hold it: 4 x 16 M 122.5,
// 122.5 (143, 146), 1 x 12 M 73, 75 (88, 91), 3 x 8 M 106, 108 (122, 126).  The launch alone: 3 x 22 M 56, 41; 4 x 60 M 117, 91; 1 x 137 M
// 249, 221; 3 x 200 M 343, 310.
#define FIN_PAST 20000000ull
#ifndef IDX_BLOCKS_PER_CU
#define IDX_BLOCKS_PER_CU 4   // 2-4 blocks per CU index 3 % faster than 8: its bound is requests to memory, not latency
#endif
// Largest bucket-boundary table (bytes) a kernel copies into LDS; with up to 8 blocks per CU
// (finalize) this keeps all of them resident in the CU's 160 KB.  Larger tables are searched in global memory.
#define IDX_TABLE_LDS_MAX 16384u

// Probe: pairs per wave, blocks.
static u32 probe_ppw(const dblp_ctx* c, u64 pairs) {
    const u64 waves = (u64)c->n_cus * 32, ppw = (pairs + waves - 1) / waves;
    return ppw > WAVE ? WAVE : ppw ? (u32)ppw : 1;
}
static u64 probe_blocks(const dblp_ctx* c, u64 pairs) {
    if (c->probe_block_pair) return pairs;
    const u64 per = 4ull * probe_ppw(c, pairs);
    return (pairs + per - 1) / per;
}

// The instance for `np` KB of a packet per step.  4 KB of loads in flight per wave, 64 KB per CU, are enough; twice as
// many only spread the DRAM accesses over more open rows.  us of a pass with 8 KB, 4 KB: 32 workers x 60 M in packets of 1000
// floats 1530, 1461; 8 x 60 M of 4097 490, 465; 32 x 30 M of 16374 795, 746; 2 x 150 M of 366 464, 446; 8 x 124 M of 366
// 989, 992; 16 x 355 M of 1024 4455, 4458.  For packets of one KB, which end with every step, more workers in a step are
// worth more (8 x 60 M of 128: G 4 693, G 2 772).
template <u32 LEAD>
static burst_fn burst_kernel(u32 np) {
    return np == 1 ? gather_burst<1, 4, LEAD> : np == 2 ? gather_burst<2, 2, LEAD> : np == 3 ? gather_burst<3, 1, LEAD> : gather_burst<4, 1, LEAD>;
}

// Units of 16 bytes from the packet's start (LEAD 2), or from the payload's (LEAD 0) where that takes one
// pass of 64 less: payloads of 256, 512, 768 and 1024 floats (or one float fewer) would need one more
// for the two floats that the 8-byte header pushes out (16 x 256 floats, 60 M: 860 -> 818 us; 1 x 256,
// 25.6 M: 55 -> 48; 1024-float retransmissions: 162 -> 144).  Other lengths are better off from the
// start, where fewer passes begin inside a 128-byte line (32 x 1472 B: 1.64 against 1.65 ms).
static bool units_from_packet(const Geo& g) { return !(g.P <= 1024 && (g.P + 255) / 256 < (g.P + 2 + 255) / 256); }
static u32 unit_passes(const Geo& g, bool lead) { return lead ? (g.units + WAVE - 1) / WAVE : (g.P + 4 * WAVE - 1) / (4 * WAVE); }

// The line between gather_burst and gather_stream, by the bytes that a batch reads (measured on 256 CUs and not scaled
// with their number: what a smaller part of the chip would ask for is not known; us of a whole pass with gather_stream,
// with bursts; P = 366 unless said):
//   8 workers and more   150 MB (8 x 5 M elements, 160 MB: 116, 113; 16 x 2 M, 128 MB: 106, 106; 32 x 1 M: 114, 116)
//   5 to 7               300 MB (6 x 10 M: 156, 155; 5 x 10 M: 149, 149; 6 x 25 M: 281, 269; 5 x 25 M: 261, 252)
//   by the bytes that it writes, where these weigh more and a group's turn is short:
//   3 and 4              144 MB (4 x 25 M: 184, 186; 3 x 25 M: 205, 206; 4 x 40 M: 265, 249; 3 x 40 M: 302, 291)
//   2                    256 MB (2 x 38 M: 180, 180; 2 x 75 M: 290, 276; 2 x 150 M: 505, 467)
//   1                    never (200 M: 473, 505)
// Packets of up to 128 floats cost gather_stream, which finishes each in registers, more than they cost bursts: from
// 48 MB read on (2 x 10 M of 128 floats: 130, 127; 4 x 10 M of 64: 220, 185; 4 x 40 M of 64: 608, 462).
// The groups have to fill the chip: of 8 or a multiple of 8 packets (a group owns whole bytes of the bitmap) eleven
// packets a CU, which leaves a CU in three idle at most (64 x 2 M of 1024 floats, 8 a CU: 183, 201; 32 x 3 M, 12 a
// CU: 165, 156), of fewer and larger ones two (32 x 5 M of 16374, one a CU: 238, 251; 32 x 5 M of 8191: 238, 233).

static BurstPlan burst_plan(const Geo& g, u32 cus) {
    BurstPlan b = {};
    if (g.W == 1) return b;
    const bool lead = units_from_packet(g);
    const u32 n_pass = unit_passes(g, lead);
    const u64 span = 4ull * g.P, packets = (u64)g.W * g.stride;         // bytes written and read per sequence number
    const u64 least = g.P <= 128 ? 48000000ull / packets : g.W >= 8 ? 150000000ull / packets : g.W >= 5 ? 300000000ull / packets
                    : g.W >= 3 ? 144000000ull / span : 256000000ull / span;
    const size_t table = ((size_t)g.B + 1) * sizeof(u32);
    const u32 table_words = table <= IDX_TABLE_LDS_MAX ? g.B + 1 : 0u;
    auto image_at = [&](u32 r) { return (BURST_INFO_LDS(g.W, r) + table_words + 31u) / 32u * 32u; };
    auto lds = [&](u32 r) { return 4ull * (image_at(r) + (u64)r * g.P + 40u); };
    u32 r = BURST_MAX, step = 8;
    while (r > 8 && lds(r) > BURST_LDS) r -= 8;
    if (lds(r) > BURST_LDS) { step = 1; while (r > 0 && lds(r) > BURST_LDS) --r; }
    if (r == 0) return b;
    const u32 turn = (u32)(((u64)g.n_pkts + cus - 1) / cus), most = (turn + step - 1) / step * step;
    if (r > most) r = most;                             // short rounds: what gives every CU a group
    const u64 fill = (u64)(step == 8 ? 11u : 2u) * cus;
    b.min_seq = (u32)(least > fill ? (least < NONE32 ? least : NONE32) : fill);
    if (b.min_seq > g.n_pkts) return b;
    b.n_piece = (n_pass + 3) / 4;                       // five passes are two pieces (16 x 100 M of 1200 floats: 1342 us as one, 1317 as two)
    const u32 np = (n_pass + b.n_piece - 1) / b.n_piece;
    b.n_piece = (n_pass + np - 1) / np;
    b.kb = np * b.n_piece;
    b.r_max = r; b.r_step = step;
    b.table_at = table_words ? BURST_INFO_LDS(g.W, r) : 0u;
    b.image_at = image_at(r);
    b.lds = lds(r);
    // written through up to 16 MB per worker, 272 MB at most (us of a pass, through and past: 8 x 25 M 260, 263; 8 x 40 M
    // 377, 373; 16 x 40 M 606, 622; 24 x 60 M 1392, 1417; 32 x 66 M 1896, 1903; 16 x 120 M 1806, 1782)
    b.through_seq = (u32)((g.W < 17 ? 16000000ull * g.W : 272000000ull) / span);
    b.fn = lead ? burst_kernel<2>(np) : burst_kernel<0>(np);
    return b;
}

static void reset_state(dblp_ctx* c, int i) {
    RoundState& st = c->state[i];
    const u64 n = LONG_ALL + c->g.W * c->g.words_pw;
    hipLaunchKernelGGL(reset_round, dim3(grid_for(c, (n + 2 * ACCEPT_ROWS + 255) / 256, 16)), dim3(256), 0, c->stream,
                       st.bitmap - LONG_ALL, n, st.rows, (u64)(2 * ACCEPT_ROWS), st.counters);
    st.rows_used = 0; st.listed = 0;
}

// A call that is recorded now will be told again with the state's addresses as they are, and a begin_round among the
// recorded ones has to clear it each time: from the first such call on, one state stays in use and each begin_round launches.
static void note_recording(dblp_ctx* c) {
    if (c->recorded || !c->stream) return;      // (the null stream cannot be recorded)
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &st) != hipSuccess) { (void)hipGetLastError(); c->recorded = 1; }
    else if (st != hipStreamCaptureStatusNone) c->recorded = 1;
}

extern "C" int dblp_create(dblp_ctx** out, const dblp_config* cfg) {
    if (!out || !cfg || !cfg->buckets) return DBLP_EINVAL;
    if (cfg->n_workers == 0 || cfg->n_workers > DBLP_MAX_WORKERS) return DBLP_EINVAL;
    if (cfg->payload_floats == 0 || cfg->payload_floats > 65535) return DBLP_EINVAL;
    if (cfg->n_buckets == 0 || cfg->n_elems == 0) return DBLP_EINVAL;
    if (!(cfg->eta >= 0.0)) return DBLP_EINVAL;
    if (cfg->accumulator_mode < DBLP_ACCMODE_SINGLE || cfg->accumulator_mode > DBLP_ACCMODE_SEARCH) return DBLP_EINVAL;
    if (cfg->search_free_fraction < 0.0 || cfg->search_free_fraction > 0.9 || !(cfg->search_seconds >= 0.0)) return DBLP_EINVAL;
    for (int i = 0; i < 2; ++i)
        if (cfg->d_accumulator[i] && ((uintptr_t)cfg->d_accumulator[i] & 255) != 0) return DBLP_EINVAL;
    if (cfg->d_accumulator[1] && (!cfg->d_accumulator[0] || cfg->accumulator_mode != DBLP_ACCMODE_PAIR ||
                                  cfg->d_accumulator[1] == cfg->d_accumulator[0])) return DBLP_EINVAL;
    if (cfg->d_accumulator[0] && cfg->accumulator_mode == DBLP_ACCMODE_SEARCH) return DBLP_EINVAL;   // the search owns both copies
    if (cfg->d_accumulator[0] && cfg->accumulator_mode == DBLP_ACCMODE_PAIR && !cfg->d_accumulator[1]) return DBLP_EINVAL;
    const u32 B = cfg->n_buckets, P = cfg->payload_floats;
    u64 expect = 0, n_pkts = 0;
    for (u32 b = 0; b < B; ++b) {
        if (cfg->buckets[b].elem_offset != expect) return DBLP_EINVAL;
        if (cfg->buckets[b].elem_count == 0 || cfg->buckets[b].elem_count >= (1ull << 32)) return DBLP_EINVAL;
        expect += cfg->buckets[b].elem_count;
        n_pkts += (cfg->buckets[b].elem_count + P - 1) / P;
    }
    if (expect != cfg->n_elems) return DBLP_EINVAL;
    if (n_pkts >= 0xFFFFFFFFull) return DBLP_EINVAL;

    dblp_ctx* c = (dblp_ctx*)calloc(1, sizeof *c);
    if (!c) return DBLP_ENOMEM;
    c->N = cfg->n_elems; c->eta = cfg->eta; c->device = cfg->device; c->stream = (hipStream_t)cfg->stream;
    c->search_fraction = cfg->search_free_fraction > 0.0 ? cfg->search_free_fraction : 0.5;
    c->search_seconds = cfg->search_seconds > 0.0 ? cfg->search_seconds : 2.0;
    c->probe_polls = PROBE_LOOKS;
    c->fold = (cfg->n_workers & (cfg->n_workers - 1)) == 0;
    c->result_in_place = c->fold ? 1 : 0;     // the in-place finalize exists for power-of-two worker counts
    c->timed = new (std::nothrow) std::vector<dblp_ctx::Timed>();
    c->ev_pool = new (std::nothrow) std::vector<hipEvent_t>();
    if (!c->timed || !c->ev_pool) { dblp_destroy(c); return DBLP_ENOMEM; }
    c->h_first_seq = (u32*)malloc((B + 1) * sizeof(u32));
    c->h_b_off = (u64*)malloc(B * sizeof(u64));
    c->h_b_cnt = (u64*)malloc(B * sizeof(u64));
    if (!c->h_first_seq || !c->h_b_off || !c->h_b_cnt) { dblp_destroy(c); return DBLP_ENOMEM; }
    u64 seq = 0;
    for (u32 b = 0; b < B; ++b) {
        c->h_first_seq[b] = (u32)seq;
        c->h_b_off[b] = cfg->buckets[b].elem_offset;
        c->h_b_cnt[b] = cfg->buckets[b].elem_count;
        seq += (c->h_b_cnt[b] + P - 1) / P;
    }
    c->h_first_seq[B] = (u32)seq;

    Geo& g = c->g;
    g.B = B; g.P = P; g.W = cfg->n_workers; g.n_pkts = (u32)n_pkts;
    g.stride = (8 + 4 * P + 15) / 16 * 16;
    g.units = g.stride / 16;
    g.words_pw = (n_pkts + 63) / 64;

    hipError_t e = hipSetDevice(c->device);
    if (e != hipSuccess) { dblp_destroy(c); return DBLP_EHIP; }
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, c->device);
    if (e != hipSuccess) { dblp_destroy(c); return DBLP_EHIP; }
    c->n_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    if ((u64)c->n_cus * 16 > ACCEPT_ROWS) c->n_cus = ACCEPT_ROWS / 16;   // grids are sized n_cus x (<= 16) blocks

    const u64 pairs = (u64)g.W * B;
    c->max_partials = (u32)c->n_cus * FIN_BLOCKS_PER_CU;
    u32 longest = 0;        // packets of the longest bucket
    for (u32 b = 0; b < B; ++b) longest = c->h_first_seq[b + 1] - c->h_first_seq[b] > longest ? c->h_first_seq[b + 1] - c->h_first_seq[b] : longest;
    c->probe_block_pair = pairs <= 8u * (u32)c->n_cus && longest > WAVE * WAVE * PROBE_UNROLL;
    c->max_few = g.n_pkts / FEW_DIV < FEW_MAX ? g.n_pkts / FEW_DIV : FEW_MAX;
    // One allocation for all of it, and two launches to fill it: a context of 1 M elements and 4 workers is made in 130 us (with an
    // allocation each 184).
    const u64 n_totals = probe_blocks(c, pairs), n_pending = (u64)g.W * n_pkts, n_first = (n_pkts + 1) / 2, n_home = (n_pkts + 7) / 8 + 1;
    u64 size = 0;
    auto part = [&](u64 words) { const u64 at = size; size += (words + 31) / 32 * 32; return at; };      // of 8 bytes, 256-byte aligned
    const u64 at_first = part(B / 2 + 1), at_off = part(B), at_cnt = part(B), tables = size;               // as on the host
    const u64 at_tallies = part((u64)c->n_cus * IDX_BLOCKS_PER_CU * 5 / 2 + 1), at_need = part((pairs + 1) / 2), at_list = part(c->max_few + 1);
    const u64 zeros = size;
    const u64 at_flags = part(F_COUNT), at_partials = part(PARTIALS_WORDS(c->max_partials)), at_totals = part(n_totals);
    u64 at_state[2][3];
    for (auto& at : at_state) { at[0] = part(C_COUNT); at[1] = part(2 * ACCEPT_ROWS); at[2] = part(LONG_ALL + g.W * g.words_pw) + LONG_ALL; }
    const u64 at_home = part(n_home), n_zeros = size - zeros;
    const u64 ones = size, at_list_first = part(n_first), at_pending = part(n_pending), n_ones = size - ones;
    bool ok = hipMalloc(&c->slab, size * sizeof(u64)) == hipSuccess;
    c->h_tables = (u64*)calloc(tables, sizeof(u64));
    if (!c->h_tables) ok = false;
    if (ok) {
        u64* const base = c->slab;
        c->d_block_tallies = (u32*)(base + at_tallies); c->d_need = (u32*)(base + at_need);
        c->d_flags = base + at_flags; c->d_partials = base + at_partials; c->d_totals = base + at_totals;
        for (int k = 0; k < 2; ++k) c->state[k] = {base + at_state[k][2], base + at_state[k][1], base + at_state[k][0], 0, 0};
        c->d_home = (uint8_t*)(base + at_home);
        c->few.entries = base + at_list; c->few.first = (u32*)(base + at_list_first); c->d_pending = base + at_pending;
        g.first_seq = (const u32*)(base + at_first); g.b_off = base + at_off; g.b_cnt = base + at_cnt;
        memcpy(c->h_tables + at_first, c->h_first_seq, (B + 1) * sizeof(u32));
        memcpy(c->h_tables + at_off, c->h_b_off, B * sizeof(u64));
        memcpy(c->h_tables + at_cnt, c->h_b_cnt, B * sizeof(u64));
    }
    ok = ok && hipHostMalloc((void**)&c->h_mailbox, 16 * sizeof(u64), hipHostMallocMapped) == hipSuccess;
    if (!ok) { (void)hipGetLastError(); dblp_destroy(c); return DBLP_ENOMEM; }
    ok = ok && hipHostGetDevicePointer((void**)&c->d_mailbox, c->h_mailbox, 0) == hipSuccess;
    ok = ok && hipMemcpyAsync(c->slab + at_first, c->h_tables, tables * sizeof(u64), hipMemcpyHostToDevice, c->stream) == hipSuccess;
    if (!ok) { (void)hipGetLastError(); dblp_destroy(c); return DBLP_EHIP; }
    if (((size_t)B + 1) * sizeof(u32) > IDX_TABLE_LDS_MAX) {
        const size_t n = (size_t)g.words_pw + 1;
        u32* h = (u32*)malloc(n * sizeof(u32));
        if (!h || hipMalloc(&c->d_hint, n * sizeof(u32)) != hipSuccess) { free(h); (void)hipGetLastError(); dblp_destroy(c); return DBLP_ENOMEM; }
        u32 b = 0;
        for (size_t i = 0; i < n; ++i) {
            while (b + 1 < B && (u64)c->h_first_seq[b + 1] <= 64ull * i) ++b;
            h[i] = b;                               // the entry behind the last one: the last bucket
        }
        const hipError_t ce = hipMemcpy(c->d_hint, h, n * sizeof(u32), hipMemcpyHostToDevice);
        free(h);
        if (ce != hipSuccess) { (void)hipGetLastError(); dblp_destroy(c); return DBLP_EHIP; }
        g.hint = c->d_hint;
    }
    const u64 all_words = (u64)g.W * g.words_pw;
    c->probe_all = all_words <= PROBE_ALL_WORDS && pairs <= PROBE_ALL_PAIRS &&
                   hipFuncSetAttribute((const void*)probe_all, hipFuncAttributeMaxDynamicSharedMemorySize, (int)PROBE_ALL_LDS(PROBE_ALL_WORDS, PROBE_ALL_PAIRS, PROBE_ALL_PAIRS)) == hipSuccess;
    (void)hipGetLastError();
    c->burst = burst_plan(g, (u32)c->n_cus);
    // The limit is the kernel's, not the context's: the same whatever the plan, so that contexts which share an instance
    // do not lower it for each other.
    if (c->burst.fn && hipFuncSetAttribute((const void*)c->burst.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)BURST_LDS) != hipSuccess) {
        (void)hipGetLastError();
        c->burst.fn = nullptr;
    }

    hipLaunchKernelGGL(fill_u64, dim3(grid_for(c, (n_ones + 255) / 256, 16)), dim3(256), 0, c->stream, c->slab + ones, n_ones, NONE64);
    hipLaunchKernelGGL(fill_u64, dim3(grid_for(c, (n_zeros + 255) / 256, 16)), dim3(256), 0, c->stream, c->slab + zeros, n_zeros, 0ull);
    c->other_clean = 1;
    e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess || hipGetLastError() != hipSuccess) { dblp_destroy(c); return DBLP_EHIP; }
    free(c->h_tables);
    c->h_tables = nullptr;
    // accumulator last
    if (cfg->d_accumulator[0]) {
        c->acc_caller = 1;
        c->acc_alloc[0] = cfg->d_accumulator[0]; c->acc_alloc[1] = cfg->d_accumulator[1];
        c->d_acc[0] = cfg->d_accumulator[0];
        c->d_acc[1] = cfg->d_accumulator[1] ? cfg->d_accumulator[1] : cfg->d_accumulator[0];
        c->n_acc = cfg->d_accumulator[1] ? 2 : 1;
        c->d_scratch[0] = c->d_scratch[1] = nullptr;
    } else {
        const int rc = set_accumulator_copies(c, cfg->accumulator_mode == DBLP_ACCMODE_SINGLE ? 1 : 2,
                                              cfg->accumulator_mode == DBLP_ACCMODE_SEARCH ? 1 : 0);
        if (rc != DBLP_OK) { dblp_destroy(c); return rc; }
    }
    c->err[0] = 0;
    *out = c;
    return DBLP_OK;
}

extern "C" int dblp_layout(const dblp_ctx* c, uint64_t* n_pkts, uint32_t* stride, uint64_t* words_pw) {
    if (!c) return DBLP_EINVAL;
    if (n_pkts) *n_pkts = c->g.n_pkts;
    if (stride) *stride = c->g.stride;
    if (words_pw) *words_pw = c->g.words_pw;
    return DBLP_OK;
}

extern "C" int dblp_accumulator_copies(dblp_ctx* c, int copies, int place) {
    if (!c) return DBLP_EINVAL;
    if (copies != 1 && copies != 2) return fail(c, DBLP_EINVAL, "accumulator_copies: 1 or 2");
    if (place < 0 || place > 1) return fail(c, DBLP_EINVAL, "accumulator_copies: place is 0 or 1");
    if (c->acc_caller) return fail(c, DBLP_EINVAL, "accumulator_copies: the accumulator is the caller's");
    HIP_TRY(c, hipSetDevice(c->device));
    return set_accumulator_copies(c, copies, place);
}

extern "C" int dblp_accumulator_policy(dblp_ctx* c, int policy) {
    if (!c) return DBLP_EINVAL;
    if (policy < DBLP_ACC_AUTO || policy > DBLP_ACC_ALTERNATE) return fail(c, DBLP_EINVAL, "accumulator_policy: unknown policy");
    c->acc_policy = policy;
    return DBLP_OK;
}

extern "C" int dblp_accumulator_info(const dblp_ctx* c, int* copies, int* distinct, int* last_pick, double* placement_ms) {
    if (!c) return DBLP_EINVAL;
    if (placement_ms) { placement_ms[0] = c->place_ms[0]; placement_ms[1] = c->place_ms[1]; placement_ms[2] = c->place_steps; placement_ms[3] = c->place_seconds; }
    if (copies) *copies = c->n_acc;
    if (distinct) *distinct = c->acc_distinct;
    if (last_pick) *last_pick = c->last_pick;
    return DBLP_OK;
}

extern "C" int dblp_accumulator_ptr(const dblp_ctx* c, int which, float** d_copy) {
    if (!c || !d_copy) return DBLP_EINVAL;
    if (which < 0 || which >= c->n_acc || !c->acc_alloc[0]) return DBLP_EINVAL;
    *d_copy = c->d_acc[which];
    return DBLP_OK;
}

extern "C" int dblp_begin_round(dblp_ctx* c, uint16_t round) {
    if (!c) return DBLP_EINVAL;
    if (!c->acc_alloc[0]) return fail(c, DBLP_ESTATE, "begin_round: no accumulator (dblp_accumulator_copies ran out of memory)");
    HIP_TRY(c, hipSetDevice(c->device));
    note_recording(c);
    if (c->other_clean && !c->recorded) {
        c->cur ^= 1;
        c->other_clean = 0;
    } else {
        reset_state(c, c->cur);
        LAUNCH_CHECK(c, "begin_round");
    }
    c->round = round; c->round_open = 1; c->finalized = 0; c->counters_in_mailbox = 0;
    return DBLP_OK;
}

// Element window [lo, hi) covered by packets first_seq .. first_seq + n - 1 (host geometry).
static void seq_window(const dblp_ctx* c, u64 first_seq, u64 n, u64* lo, u64* hi) {
    const Geo& g = c->g;
    auto span = [&](u64 seq, u64* elem, u64* len) {
        u32 a = 0, b = g.B;
        while (b - a > 1) { u32 m = (a + b) / 2; if (c->h_first_seq[m] <= seq) a = m; else b = m; }
        u64 start = (seq - c->h_first_seq[a]) * g.P;
        u64 left = c->h_b_cnt[a] - start;
        *elem = c->h_b_off[a] + start;
        *len = left < g.P ? left : g.P;
    };
    u64 e0, l0, e1, l1;
    span(first_seq, &e0, &l0);
    span(first_seq + n - 1, &e1, &l1);
    *lo = e0; *hi = e1 + l1;
}

// Packets that a wave of the sender takes at once: as many as fill the lanes of its passes best, of a short list fewer, so that
// every CU has 16 waves' worth (300 k elements in packets of 64, 4.7 k of them: 6 us either way).  0: one, by write_packet.
static SenderSplit sender_split(const dblp_ctx* c, u64 n) {
    const u32 units = c->g.units;
    SenderSplit best = {0, (65536 + units - 1) / units};
    u32 fill = 0;
    for (u32 k = 2; k <= WAVE && k * units <= SENDER_PASSES * WAVE && (u64)k * c->n_cus * 16 <= n; ++k) {
        const u32 passes = (k * units + WAVE - 1) / WAVE, here = k * units * 1000 / (passes * WAVE);
        if (here >= fill) { fill = here; best.k = k; }
    }
    return best;
}
static u32 sender_grid(const dblp_ctx* c, const SenderSplit& split, u64 n) {
    const u64 waves = split.k ? (n + split.k - 1) / split.k : n;
    return grid_for(c, (waves + 3) / 4, 8);
}

extern "C" int dblp_packetize(dblp_ctx* c, uint32_t w, uint16_t round, const float* d_grad, uint64_t elem_base,
                              uint64_t n_grad, uint64_t first_seq, uint64_t n_pkts, const uint32_t* d_slot_map,
                              uint64_t slot_base, uint64_t n_slots, void* d_packets, uint16_t* d_src_worker) {
    if (!c) return DBLP_EINVAL;
    if (n_pkts == 0) return DBLP_OK;
    if (!d_grad || !d_packets || !d_src_worker) return fail(c, DBLP_EINVAL, "packetize: null pointer");
    if (w >= c->g.W) return fail(c, DBLP_EINVAL, "packetize: worker out of range");
    if (first_seq >= c->g.n_pkts || n_pkts > c->g.n_pkts - first_seq) return fail(c, DBLP_EINVAL, "packetize: seq range");
    if (((uintptr_t)d_packets & 15) != 0) return fail(c, DBLP_EINVAL, "packetize: d_packets must be 16-byte aligned");
    if (!d_slot_map && (slot_base > n_slots || n_pkts > n_slots - slot_base)) return fail(c, DBLP_EINVAL, "packetize: slots exceed buffer");
    u64 lo, hi;
    seq_window(c, first_seq, n_pkts, &lo, &hi);
    if (lo < elem_base || hi > elem_base + n_grad) return fail(c, DBLP_EINVAL, "packetize: packets outside the gradient window");
    HIP_TRY(c, hipSetDevice(c->device));
    *(volatile u64*)(c->h_mailbox + 4) = 0;
    const size_t table = ((size_t)c->g.B + 1) * sizeof(u32);
    const SenderSplit split = sender_split(c, n_pkts);
    const bool lds = table <= IDX_TABLE_LDS_MAX;
    void (*const kern)(Geo, SenderSplit, u32, u32, const float*, u64, u32, u32, const u32*, u64, u64, uint8_t*, uint16_t*, u64*) =
        split.k ? (lds ? packetize_kernel<true, true> : packetize_kernel<false, true>) : (lds ? packetize_kernel<true, false> : packetize_kernel<false, false>);
    hipLaunchKernelGGL(kern, dim3(sender_grid(c, split, n_pkts)), dim3(256), lds ? table : 0, c->stream, c->g, split, w, (u32)round, d_grad, (u64)elem_base,
                       (u32)first_seq, (u32)n_pkts, d_slot_map, (u64)slot_base, (u64)n_slots, (uint8_t*)d_packets, d_src_worker, c->d_mailbox + 4);
    LAUNCH_CHECK(c, "packetize");
    if (d_slot_map) {   // slots come from device memory: the kernel checks them, report here
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        if (*(volatile u64*)(c->h_mailbox + 4)) return fail(c, DBLP_EINVAL, "packetize: slot map entry outside the packet buffer");
    }
    return DBLP_OK;
}

extern "C" int dblp_packetize_list(dblp_ctx* c, uint16_t round, const float* const* h_grads, const uint64_t* d_list,
                                   uint64_t n, uint64_t slot_base, uint64_t n_slots, void* d_packets,
                                   uint16_t* d_src_worker) {
    if (!c) return DBLP_EINVAL;
    if (n == 0) return DBLP_OK;
    if (!h_grads || !d_list || !d_packets || !d_src_worker) return fail(c, DBLP_EINVAL, "packetize_list: null pointer");
    if (((uintptr_t)d_packets & 15) != 0) return fail(c, DBLP_EINVAL, "packetize_list: d_packets must be 16-byte aligned");
    if (slot_base > n_slots || n > n_slots - slot_base) return fail(c, DBLP_EINVAL, "packetize_list: slots exceed buffer");
    GradPtrs gp;
    for (u32 w = 0; w < DBLP_MAX_WORKERS; ++w) gp.p[w] = nullptr;
    for (u32 w = 0; w < c->g.W; ++w) {
        if (!h_grads[w]) return fail(c, DBLP_EINVAL, "packetize_list: null gradient pointer");
        gp.p[w] = h_grads[w];
    }
    HIP_TRY(c, hipSetDevice(c->device));
    *(volatile u64*)(c->h_mailbox + 4) = 0;
    const size_t table = ((size_t)c->g.B + 1) * sizeof(u32);
    const SenderSplit split = sender_split(c, n);
    const bool lds = table <= IDX_TABLE_LDS_MAX;
    void (*const kern)(Geo, SenderSplit, GradPtrs, u32, const u64*, u64, u64, uint8_t*, uint16_t*, u64*) =
        split.k ? (lds ? packetize_list_kernel<true, true> : packetize_list_kernel<false, true>) : (lds ? packetize_list_kernel<true, false> : packetize_list_kernel<false, false>);
    hipLaunchKernelGGL(kern, dim3(sender_grid(c, split, n)), dim3(256), lds ? table : 0, c->stream, c->g, split, gp, (u32)round, (const u64*)d_list, (u64)n,
                       (u64)slot_base, (uint8_t*)d_packets, d_src_worker, c->d_mailbox + 4);
    LAUNCH_CHECK(c, "packetize_list");
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    if (*(volatile u64*)(c->h_mailbox + 4)) return fail(c, DBLP_EINVAL, "packetize_list: list entry with worker or seq out of range");
    return DBLP_OK;
}

typedef void (*gather_fn)(Geo, const uint8_t*, u64*, u64*, float*, float*, uint8_t*, u32, const u32*, u32, u64*, u64*, double*, float,
                          GatherShape, GatherShape, u32, u32, u32, u32, u64*, u32*, ArrivalList);

// The instance for `np` KB of a packet per step and w workers.
template <bool DENSE, u32 LEAD, bool MANY>
static gather_fn short_kernel(u32 np) {
    return np == 1 ? gather_stream<1, 4, 2, 4, LEAD, DENSE, MANY> : np == 2 ? gather_stream<2, 4, 2, 4, LEAD, DENSE, MANY>
         : np == 3 ? gather_stream<3, 2, 2, 4, LEAD, DENSE, MANY> : np == 4 || !LEAD ? gather_stream<4, 2, 2, 4, LEAD, DENSE, MANY>
                                                                                    : gather_stream<5, 1, 3, 4, 2, DENSE, MANY>;
}
template <bool DENSE, u32 LEAD>
static gather_fn short_kernel(u32 w, u32 np) {
    if (w < 4) return np == 1 ? gather_stream<1, 1, 4, 4, LEAD, DENSE, false> : np == 2 ? gather_stream<2, 1, 4, 4, LEAD, DENSE, false>
                    : np == 3 ? gather_stream<3, 1, 3, 4, LEAD, DENSE, false> : np == 4 || !LEAD ? gather_stream<4, 1, 3, 4, LEAD, DENSE, false>
                                                                                                : gather_stream<5, 1, 3, 4, 2, DENSE, false>;
    return w > 16 ? short_kernel<DENSE, LEAD, true>(np) : short_kernel<DENSE, LEAD, false>(np);
}
template <bool DENSE, bool MANY>
static gather_fn long_kernel(u32 np) {
    return np == 1 ? gather_stream<1, 4, 2, 16, 2, DENSE, MANY> : np == 2 ? gather_stream<2, 2, 2, 16, 2, DENSE, MANY> : gather_stream<4, 2, 2, 16, 2, DENSE, MANY>;
}
template <bool DENSE>
static gather_fn gather_kernel(u32 nw, bool lead, u32 w, u32 np) {
    if (nw == 16) return w > 16 ? long_kernel<DENSE, true>(np) : long_kernel<DENSE, false>(np);
    return lead ? short_kernel<DENSE, 2>(w, np) : short_kernel<DENSE, 0>(w, np);
}

typedef void (*list_fn)(Geo, const uint8_t*, u64*, u64*, float*, float*, uint8_t*, u32, ArrivalList, const u32*, u32, u64*, u64*, double*, float, u32*);
// The instance for pieces of `np` KB; units are counted from the payload in packets of up to four passes only.
static list_fn list_kernel(bool lead, u32 np, bool team) {
    if (team) return np == 3 ? gather_list<3, 2, true> : gather_list<4, 2, true>;
    if (lead) return np == 1 ? gather_list<1, 2, false> : np == 2 ? gather_list<2, 2, false> : np == 3 ? gather_list<3, 2, false> : gather_list<4, 2, false>;
    return np == 1 ? gather_list<1, 0, false> : np == 2 ? gather_list<2, 0, false> : np == 3 ? gather_list<3, 0, false> : gather_list<4, 0, false>;
}
// Batches that a gather_list launch takes whatever they are: as few as that it is the shorter way for dense ones too (us of
// a batch that is dense, and of one that is not, by a launch that decides and by the list: 1 x 512 packets of 1472 B 14.6, 13.0 and 13.1, 11.5, of
// 1024 14.7, 16.0 and 13.4, 11.6; 3 x 512 15.5, 14.8 and 13.6, 11.8; 8 x 192 15.8, 13.2 and 14.0, 12.4, 8 x 512 16.0, 19.6 and 15.6, 14.1), and
// no packet is summed in many steps one after the other (eight: 32 workers of 1472 B 17.0 to 22.2, 17.6; 16: 64 workers 20.6 to 22.8, 22.0 to 25.0;
// 24: 48 x 2816 B 22.4, 25.2; 32: 32 x 4816 B 25.7, 33.8).
static bool few_always(const Geo& g, u64 n, u32 kb, bool team) {
    const u32 pieces = (g.units + kb * WAVE - 1) / (kb * WAVE), steps = (g.W + FEW_DEPTH(kb) - 1) / FEW_DEPTH(kb) * (team ? (pieces + GS_WAVES - 1) / GS_WAVES : pieces);
    return n <= 1536 && n <= 384ull * g.W && steps <= 8;
}

#define HEAVY_BYTES 131072u  // from all workers for one sequence number
// Waves of a gather block: 4; 16 in rounds of heavy packets with fewer sequence numbers than CUs (64 workers x 4016 B,
// 60 packets: 19 against 28 us; with 260 packets 35 against 31, with 1000 61 against 51: groups of one or two
// packets spread four waves over the chip as well).
static u32 block_waves(const dblp_ctx* c) {
    return c->g.n_pkts < (u32)c->n_cus && (u64)c->g.W * c->g.stride >= HEAVY_BYTES ? 16 : GS_WAVES;
}

// Index pass + gather pass over one batch.  Exactly one of (d_src_worker [+ d_mask, d_order]) and
// d_queue describes the arrivals.
static int apply_batch(dblp_ctx* c, const void* d_packets, const uint16_t* d_src_worker, uint64_t n_slots,
                       const uint64_t* d_mask, const uint32_t* d_order, const uint64_t* d_queue, uint64_t n_arrivals) {
    HIP_TRY(c, hipSetDevice(c->device));
    note_recording(c);
    const Geo& g = c->g;
    const int pick = pick_copy(c, d_packets, n_slots * g.stride, n_slots, n_arrivals);
    c->last_pick = pick;
    ++c->batch_no;
    const bool lead = units_from_packet(g) || block_waves(c) == 16;
    // Dense or sparse.  At least one arrival per SPARSE_DIV (worker, seq) pairs of the whole round is dense
    // whatever range it touches, and the launch is told so.  Fewer are a retransmission or a step of a round
    // that arrives in many steps; the number does not say which, so the blocks decide, from the sequence
    // range that the index pass found (a launch that took fewer than one per 64 pairs for sparse saved it 0 to
    // 0.4 us, and cost a round of 32 x 60 M elements in 129 steps 11.7 against 4.7 ms).
    const u64 pairs = (u64)g.W * g.n_pkts;
    const bool is_dense = n_arrivals * SPARSE_DIV >= pairs, small = n_arrivals * SPARSE_DIV * 8 < pairs;
    const u32 nw = small && g.stride < 8192 ? GS_WAVES      // 16 waves for a handful of 4 KB packets: 29 against 22 us
                                            : block_waves(c);
    // Dense.  Packets of up to 5 KB are one piece, longer ones are cut evenly into pieces of 3 or 4 KB; in
    // a short round finer, so that a group gives each of the block's waves a piece.
    GatherShape dense, sparse;
    const u32 n_pass = unit_passes(g, lead);
    dense.n_piece = n_pass <= 5 ? 1 : (n_pass + 3) / 4;
    const u32 heavy = (u64)g.W * g.stride >= HEAVY_BYTES ? 2 : (u64)g.W * g.stride >= HEAVY_BYTES / 2 ? 1 : 0;
    dense.sub_log2 = group_log2(g.n_pkts, (u32)c->n_cus, dense.n_piece > 1, heavy);      // (the whole round's)
    if (nw == 16) {
        const u32 want = nw >> dense.sub_log2 < n_pass ? nw >> dense.sub_log2 : n_pass;
        if (dense.n_piece < want) dense.n_piece = want;
    }
    const u32 np = (n_pass + dense.n_piece - 1) / dense.n_piece;
    dense.n_piece = (n_pass + np - 1) / np;
    // One to three workers: a step is one worker's piece, four of them in flight, and six blocks per
    // CU (1 worker: 45 us, against 54 with three blocks, 68 with steps of four workers; 25.6 M elements of 366
    // floats, 2 workers 61 against 73 with steps of four, 3 workers 78 and 82, 4 workers 98 and 97, 8 workers 176
    // and 174).  More: 4 to 8 KB per step, two steps in flight, three blocks per CU for short packets, two for
    // long ones (8992 B: 930 against 940 us; more blocks only spread the DRAM accesses over more open rows).
    const bool few = g.W < 4;
    const u32 per_cu = nw == 16 ? 1 : few ? (np <= 2 && is_dense ? 6 : 4) : np <= 2 ? 3 : 2;
    const u64 groups = ((u64)g.n_pkts + (1u << dense.sub_log2) - 1) >> dense.sub_log2;
    dense.blocks = grid_for(c, groups, per_cu);

    // Sparse.  One worker's 2 KB per step.  Groups of 32 packets of up to 2 KB in long rounds, longer rows of the
    // index and fewer empty groups to pass: 1 x 1.9 M packets of 136 bytes, 562 lost 26 us against 37 with 16; 8 x
    // 340 k of 1472 B, 14 k lost 46 against 48 (with more of them, or in bursts, 16 would do better: 6.9 k lost
    // there 50 against 43).  Otherwise as for dense batches.
    sparse.n_piece = lead ? (g.units + 2 * WAVE - 1) / (2 * WAVE) : (g.P + 8 * WAVE - 1) / (8 * WAVE);
    sparse.sub_log2 = sparse.n_piece == 1 && g.n_pkts >= (g.W <= 4 ? 32u : 64u) * (u32)c->n_cus ? 5 : group_log2(g.n_pkts, (u32)c->n_cus, sparse.n_piece > 1, heavy == 2 ? 2 : 0);
    // Packets of 16 KB and more fill a block's waves four at a time: fewer to one block where lost packets
    // follow each other (1 worker x 66 M in 64 KB packets, 12 lost 18 against 23 us, 247 lost 32 against 48; 4 x
    // 61 M, 80 lost 29 against 42), until the groups get many.
    if (sparse.n_piece >= 8 && sparse.sub_log2 > 2 && g.n_pkts <= 64u * (u32)c->n_cus) sparse.sub_log2 = 2;
    sparse.blocks = grid_for(c, ((u64)g.n_pkts + (1u << sparse.sub_log2) - 1) >> sparse.sub_log2, nw == 16 ? 1 : 4);

    // Bursts.  A batch of at least burst.min_seq packets per worker covers that many sequence numbers or more.  Where the number
    // of arrivals alone says that it is dense enough, it is one gather_burst launch.  Where the blocks have to find out (or
    // with a mask, whose lost slots count as arrivals), that launch leaves a batch that is not to a gather_stream launch
    // after it, which ends at once if it was.  The second launch costs 2 to 4 us, so it is made for batches of 256 MB and more only,
    // which take 60 us and more as a dense step and 130 as a retransmission; and not for many arrivals of two or three
    // workers, whose gather_stream of both kinds has fewer waves in flight (half of 2 x 150 M 297 us, 325 asked).
    const BurstPlan& burst = c->burst;
    const bool enough = burst.fn && n_arrivals >= (u64)burst.min_seq * g.W;
    const bool known = enough && is_dense && !d_mask && burst_pays(n_arrivals, g.n_pkts, g.W, (u32)c->n_cus, burst.r_max, burst.kb);
    const bool asked = enough && !known && n_arrivals * g.stride >= 256000000ull && !(few && is_dense && !d_mask);
    const bool in_bursts = known || asked, dense_only = is_dense && !asked;
    ArrivalList list = {nullptr, nullptr, 0};
    if (!in_bursts && !is_dense && n_arrivals <= c->max_few) { list = c->few; list.n = (u32)n_arrivals; }
    const u64 turns = in_bursts ? 8 : (groups + dense.blocks - 1) / dense.blocks;
    const bool whole = n_arrivals * WHOLE_DIV >= pairs && !asked && (!d_mask || turns <= 2);
    const bool any = whole && turns > 4;                // (two turns for nothing take 1 us; the word costs 0.4 to 1.5)
    const u32 any_at = any ? c->any_no++ & 1u : 0u;
    RoundState& now = c->state[c->cur];
    if (list.entries) now.listed = 1;
    const u32 batch = (whole ? B_WHOLE : 0) | (any ? B_ANY : 0) | (any_at ? B_ANY_AT : 0) | (asked ? B_ASKED : 0);

    u32 n_tally_rows = 0;
    {
        ProfScope ps(c, DBLP_K_INDEX);
        const u32 grid = grid_for(c, (n_arrivals + 255) / 256, IDX_BLOCKS_PER_CU);
        const size_t table = ((size_t)g.B + 1) * sizeof(u32);
        const bool lds = table <= IDX_TABLE_LDS_MAX;
        void (*idx)(Geo, const uint8_t*, const uint16_t*, u64, const u64*, const u32*, const u64*, u64, u32, u64*, u32*, u64*, ArrivalList) =
            lds ? (d_queue ? index_arrivals<true, true> : index_arrivals<true, false>)
                : (d_queue ? index_arrivals<false, true> : index_arrivals<false, false>);
        hipLaunchKernelGGL(idx, dim3(grid), dim3(256), lds ? table : 0, c->stream, g,
                           (const uint8_t*)d_packets, d_src_worker, (u64)n_slots, (const u64*)d_mask, d_order,
                           (const u64*)d_queue, (u64)n_arrivals, (u32)c->round, c->d_pending, c->d_block_tallies, any ? c->d_flags + F_ANY + any_at : nullptr,
                           list);
        n_tally_rows = grid;
    }
    const float inv_w = c->fold ? 1.0f / (float)g.W : 1.0f;   // exact for the powers of two it is used with
    const u32 passes = unit_passes(g, units_from_packet(g)), list_kb = (passes + (passes + 3) / 4 - 1) / ((passes + 3) / 4);
    const bool team = FEW_TEAM(g, list_kb);
    if (list.entries && few_always(g, n_arrivals, list_kb, team)) {
        const u32 blocks = grid_for(c, team ? n_arrivals : (n_arrivals + GS_WAVES - 1) / GS_WAVES, 4);
        ProfScope ps(c, DBLP_K_GATHER_DIRECT, !small);
        if (blocks > now.rows_used) now.rows_used = blocks;
        hipLaunchKernelGGL(list_kernel(units_from_packet(g), list_kb, team), dim3(blocks + 1), dim3(GS_WAVES * WAVE), 0, c->stream, g, (const uint8_t*)d_packets,
                           c->d_pending, now.bitmap, c->d_acc[0], c->d_acc[1], c->d_home, (u32)pick, list, (const u32*)c->d_block_tallies, n_tally_rows,
                           now.counters, now.rows, (double*)(now.rows + ACCEPT_ROWS), inv_w, ps.d_told());
    } else {
        u32 slots = 0, grid = dense.blocks;
        for (u32 l = 0; l <= (dense.sub_log2 > 2 ? dense.sub_log2 : 2); ++l)        // whatever the launch may choose
            if (GS_TEAM_LDS(g.W, l) > slots) slots = GS_TEAM_LDS(g.W, l);
        if (!dense_only) {
            if (GS_TEAM_LDS(g.W, sparse.sub_log2) > slots) slots = GS_TEAM_LDS(g.W, sparse.sub_log2);
            if (sparse.blocks > grid) grid = sparse.blocks;
            // Few arrivals: a team for each, and, should they be dense, a group for each sequence number that they can touch.
            const u64 teams = FEW_TEAM(g, np > 4 ? 3 : np) ? n_arrivals : (n_arrivals + nw - 1) / nw, groups_touched = ((n_arrivals * SPARSE_DIV + g.W - 1) / g.W >> (heavy ? 0 : 3)) + 2;
            if (list.entries) {
                const u64 most = teams > groups_touched ? teams : groups_touched;
                if (grid > most) grid = (u32)most;
                if (dense.blocks > grid) dense.blocks = grid;
                if (sparse.blocks > grid) sparse.blocks = grid;
            }
        }
        size_t lds = (size_t)nw * slots * sizeof(u32);
        const size_t table = ((size_t)g.B + 1) * sizeof(u32);
        const u32 table_at = table <= IDX_TABLE_LDS_MAX ? nw * slots : 0u;
        if (table_at) lds += table;
        const gather_fn kern = dense_only ? gather_kernel<true>(nw, lead, g.W, np) : gather_kernel<false>(nw, lead, g.W, np);
        ProfScope ps(c, small ? DBLP_K_GATHER_DIRECT : DBLP_K_GATHER, !dense_only && !small && !known, known);
        if (in_bursts) {
            if ((u32)c->n_cus > now.rows_used) now.rows_used = (u32)c->n_cus;
            hipLaunchKernelGGL(burst.fn, dim3(c->n_cus), dim3(BURST_WAVES * WAVE), burst.lds, c->stream, g, (const uint8_t*)d_packets, c->d_pending, now.bitmap,
                               c->d_acc[0], c->d_acc[1], c->d_home, (u32)pick, (const u32*)c->d_block_tallies, n_tally_rows, now.counters,
                               now.rows, (double*)(now.rows + ACCEPT_ROWS), inv_w, burst.r_max, burst.r_step, burst.n_piece, burst.table_at, burst.image_at,
                               known ? 0u : burst.min_seq, burst.through_seq, batch, c->d_flags);
        }
        if (!known) {
            if (grid > now.rows_used) now.rows_used = grid;
            hipLaunchKernelGGL(kern, dim3(grid), dim3(nw * WAVE), lds, c->stream, g, (const uint8_t*)d_packets, c->d_pending, now.bitmap,
                               c->d_acc[0], c->d_acc[1], c->d_home, (u32)pick, (const u32*)c->d_block_tallies, n_tally_rows, now.counters,
                               now.rows, (double*)(now.rows + ACCEPT_ROWS), inv_w, dense, sparse, (u32)c->n_cus, heavy, table_at, batch, c->d_flags, ps.d_told(), list);
        }
    }
    LAUNCH_CHECK(c, "apply_arrivals");
    c->finalized = 0; c->counters_in_mailbox = 0;
    return DBLP_OK;
}

extern "C" int dblp_apply_arrivals(dblp_ctx* c, const void* d_packets, const uint16_t* d_src_worker, uint64_t n_slots,
                                   const uint64_t* d_mask, const uint32_t* d_order, uint64_t n_arrivals) {
    if (!c) return DBLP_EINVAL;
    if (!c->round_open) return fail(c, DBLP_ESTATE, "apply_arrivals before begin_round");
    if (n_arrivals == 0) return DBLP_OK;
    if (!d_packets || !d_src_worker) return fail(c, DBLP_EINVAL, "apply_arrivals: null pointer");
    if (((uintptr_t)d_packets & 15) != 0) return fail(c, DBLP_EINVAL, "apply_arrivals: d_packets must be 16-byte aligned");
    if (n_slots >= 0xFFFFFFFFull || n_arrivals >= 0xFFFFFFFFull) return fail(c, DBLP_EINVAL, "apply_arrivals: too many slots");
    if (!d_order && n_arrivals > n_slots) return fail(c, DBLP_EINVAL, "apply_arrivals: identity order longer than the buffer");
    return apply_batch(c, d_packets, d_src_worker, n_slots, d_mask, d_order, nullptr, n_arrivals);
}

extern "C" int dblp_apply_arrivals_queue(dblp_ctx* c, const void* d_packets, uint64_t n_slots, const uint64_t* d_queue,
                                         uint64_t n_arrivals) {
    if (!c) return DBLP_EINVAL;
    if (!c->round_open) return fail(c, DBLP_ESTATE, "apply_arrivals_queue before begin_round");
    if (n_arrivals == 0) return DBLP_OK;
    if (!d_packets || !d_queue) return fail(c, DBLP_EINVAL, "apply_arrivals_queue: null pointer");
    if (((uintptr_t)d_packets & 15) != 0) return fail(c, DBLP_EINVAL, "apply_arrivals_queue: d_packets must be 16-byte aligned");
    if (((uintptr_t)d_queue & 7) != 0) return fail(c, DBLP_EINVAL, "apply_arrivals_queue: d_queue must be 8-byte aligned");
    if (n_slots >= 0xFFFFFFFFull || n_arrivals >= 0xFFFFFFFFull) return fail(c, DBLP_EINVAL, "apply_arrivals_queue: too many slots");
    return apply_batch(c, d_packets, nullptr, n_slots, nullptr, nullptr, d_queue, n_arrivals);
}

extern "C" int dblp_loss_account(dblp_ctx* c, uint32_t bound_ppm, uint32_t* d_missing, uint64_t* d_retx_list,
                                 uint64_t retx_capacity, uint64_t* h_retx_count, int* h_all_met) {
    if (!c) return DBLP_EINVAL;
    if (!c->round_open) return fail(c, DBLP_ESTATE, "loss_account before begin_round");
    if (!h_retx_count || !h_all_met) return fail(c, DBLP_EINVAL, "loss_account: null host pointer");
    if (!d_retx_list && retx_capacity) return fail(c, DBLP_EINVAL, "loss_account: null list with capacity");
    if (bound_ppm > 1000000u) return fail(c, DBLP_EINVAL, "loss_account: bound above 100%");
    HIP_TRY(c, hipSetDevice(c->device));
    const Geo& g = c->g;
    const u64* const bitmap = c->state[c->cur].bitmap;
    const u64 pairs = (u64)g.W * g.B, blocks = probe_blocks(c, pairs);
    const u32 ppw = probe_ppw(c, pairs);
    if (blocks > 0x7FFFFFFFull) return fail(c, DBLP_EINVAL, "loss_account: too many (worker, bucket) pairs");
    if (c->probe_all) {
        const u64 words = (u64)g.W * g.words_pw;
        ProfScope ps(c, DBLP_K_PROBE);
        hipLaunchKernelGGL(probe_all, dim3((u32)(words + PROBE_ALL_SHARE - 1) / PROBE_ALL_SHARE), dim3(PROBE_ALL_THREADS), PROBE_ALL_LDS((u32)words, g.B, (u32)pairs), c->stream, g,
                           bitmap, bound_ppm, (u32)words, (u32)pairs, d_missing, (u64*)d_retx_list, (u64)retx_capacity, c->d_mailbox);
        LAUNCH_CHECK(c, "loss_account");
        ps.end();
        HIP_TRY(c, hipStreamSynchronize(c->stream));
    } else {
        ProfScope ps(c, DBLP_K_PROBE);
        bool done = blocks * 4 <= (u64)PROBE_RESIDENT * c->n_cus;
        if (done) {
            if ((++c->probe_no & 0xFFFFFFu) == 0) ++c->probe_no;        // 0 is no tag: the launches below leave totals without one
            const u64 tag = (u64)(c->probe_no & 0xFFFFFFu) << PROBE_TAG_SHIFT;
            volatile u64* const gave_up = c->h_mailbox + M_PROBE_GAVE_UP;
            *gave_up = 0;
            hipLaunchKernelGGL(c->probe_block_pair ? probe_once<true> : probe_once<false>, dim3((u32)blocks), dim3(256), 0, c->stream, g,
                               bitmap, bound_ppm, ppw, pairs, d_missing, c->d_totals, tag, c->probe_polls, (u64*)d_retx_list, (u64)retx_capacity, c->d_mailbox);
            LAUNCH_CHECK(c, "loss_account");
            ps.end();
            HIP_TRY(c, hipStreamSynchronize(c->stream));
            done = *gave_up == 0;
        }
        if (!done) {
            // Each block of emit_retx adds up the totals of the blocks before it (2048 of them: about a
            // microsecond) unless they are so many that a pass in between is shorter.
            const int scanned = blocks > PROBE_SCAN_BLOCKS ? 1 : 0;
            hipLaunchKernelGGL(c->probe_block_pair ? loss_count<true> : loss_count<false>, dim3((u32)blocks), dim3(256), 0, c->stream, g,
                               bitmap, bound_ppm, ppw, pairs, d_missing, c->d_need, c->d_totals);
            if (scanned) hipLaunchKernelGGL(scan_totals, dim3(1), dim3(1024), 0, c->stream, c->d_totals, (u32)blocks);
            hipLaunchKernelGGL(c->probe_block_pair ? emit_retx<true> : emit_retx<false>, dim3((u32)blocks), dim3(256), 0, c->stream, g, bitmap, ppw, pairs,
                               (const u32*)c->d_need, (const u64*)c->d_totals, scanned, (u64*)d_retx_list, (u64)retx_capacity, c->d_mailbox);
            LAUNCH_CHECK(c, "loss_account");
            ps.end();
            HIP_TRY(c, hipStreamSynchronize(c->stream));
        }
    }
    c->mailbox_seen = 1;
    const u64 total = c->h_mailbox[0];
    *h_retx_count = total;
    *h_all_met = total == 0;
    if (total > retx_capacity) return fail(c, DBLP_ECAPACITY, "retransmit list truncated");
    return DBLP_OK;
}

extern "C" int dblp_probe_polls(dblp_ctx* c, uint32_t polls) {
    if (!c) return DBLP_EINVAL;
    c->probe_polls = polls;
    return DBLP_OK;
}

extern "C" int dblp_finalize(dblp_ctx* c, int compensation, float* d_out) {
    if (!c) return DBLP_EINVAL;
    if (!c->round_open) return fail(c, DBLP_ESTATE, "finalize before begin_round");
    if (compensation != DBLP_COMP_ZEROFILL_MEAN) return fail(c, DBLP_EINVAL, "finalize: unknown compensation mode");
    const bool in_place = !d_out || d_out == c->d_acc[0];
    if (in_place && !c->fold) return fail(c, DBLP_EINVAL, "finalize: the in-place form needs a power-of-two worker count");
    if (!in_place && c->n_acc == 2 && d_out == c->d_acc[1]) return fail(c, DBLP_EINVAL, "finalize: d_out is the second accumulator copy");
    if (((uintptr_t)d_out & 15) != 0) return fail(c, DBLP_EINVAL, "finalize: d_out must be 16-byte aligned");
    HIP_TRY(c, hipSetDevice(c->device));
    const Geo& g = c->g;
    // Packets per wave: where the result is left in place most waves have nothing to write, so they look
    // at a whole bitmap word (fewer packets when they are long: what is written is written by one wave);
    // into another buffer as many as make up to 8192 elements, in pieces of up to 4096 and of equal size (past the caches
    // whole groups of 4096; of a short gradient 2048, so that all CUs have some).  us of the launch, each alone: pieces of equal size
    // against 4096 and what is left, 3 x 5.3 M in 366-float packets 20.1, 19.5, 13 x 5.7 M 21.0, 20.3; pieces of 4096 and of 2048, 6 x 0.9 M 12.4, 10.9, 1 x 1.9 M
    // in 16374-float ones 12.4, 10.7, 3 x 2.8 M 14.9, 14.7 (and above 4 M elements a pass of 13 x 5.7 M 161, 164).
    u32 grp_log2 = 6;
    const bool past = !in_place && c->N >= FIN_PAST, brief = c->N < 4000000ull;
    const u64 most = in_place ? 32768 : brief ? 2048 : past ? 4096 : 8192;
    while (grp_log2 > 0 && ((u64)g.P << grp_log2) > most) --grp_log2;
    const u64 elems = (u64)g.P << grp_log2, cap = brief ? 2048 : 4096;
    const u32 n_piece = in_place ? 1 : (u32)((elems + cap - 1) / cap), per_piece = (u32)(((elems + n_piece - 1) / n_piece + 255) / 256 * 256);
    const u64 items = (((u64)g.n_pkts + (1u << grp_log2) - 1) >> grp_log2) * n_piece;
    const u32 work = grid_for(c, (items + 3) / 4, FIN_BLOCKS_PER_CU);
    note_recording(c);
    const RoundState& now = c->state[c->cur];
    RoundState other = c->state[c->cur ^ 1];
    if (c->other_clean || c->recorded) other.bitmap = nullptr;
    const u32 grid = work + 1;      // one more block sums the gather's rows: accepted packets, and the sum of squares for Eq. 1
    float* out = in_place ? c->d_acc[0] : d_out;
    {
        ProfScope ps(c, DBLP_K_FINALIZE);
        const size_t table = ((size_t)g.B + 1) * sizeof(u32);
        void (*kern)(Geo, const u64*, const float*, const float*, uint8_t*, float*, int, float, int, u32, u32, u32, u64*, u32, u32,
                     const double*, const u64*, u32, u32, u64*, u64*, RoundState) =
            table <= IDX_TABLE_LDS_MAX ? (past ? finalize_pass<true, true> : finalize_pass<true, false>) : (past ? finalize_pass<false, true> : finalize_pass<false, false>);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(256), table <= IDX_TABLE_LDS_MAX ? table : 0, c->stream, g, (const u64*)now.bitmap,
                           (const float*)c->d_acc[0], (const float*)c->d_acc[1], c->d_home, out, c->fold ? 0 : 1, (float)g.W,
                           in_place ? 1 : 0, grp_log2, n_piece, per_piece, c->d_partials, c->max_partials, work, (const double*)(now.rows + ACCEPT_ROWS), (const u64*)now.rows,
                           now.rows_used, c->fold ? now.listed : 0u, now.counters, c->d_mailbox, other);
    }
    LAUNCH_CHECK(c, "finalize");
    if (other.bitmap) {
        c->other_clean = 1;
        c->state[c->cur ^ 1].rows_used = 0; c->state[c->cur ^ 1].listed = 0;
    }
    c->result_in_place = in_place ? 1 : 0;
    c->finalized = 1;
    c->counters_in_mailbox = 1;     // valid on the host once the stream has been synchronised (mailbox_seen)
    c->mailbox_seen = 0;
    return DBLP_OK;
}

extern "C" int dblp_phase_signal(dblp_ctx* c, const float* d_vec, double* h_norm, double* h_rel_delta, int* h_critical) {
    if (!c) return DBLP_EINVAL;
    if (!h_norm || !h_rel_delta || !h_critical) return fail(c, DBLP_EINVAL, "phase_signal: null host pointer");
    HIP_TRY(c, hipSetDevice(c->device));
    if (d_vec) {
        if (((uintptr_t)d_vec & 15) != 0) return fail(c, DBLP_EINVAL, "phase_signal: d_vec must be 16-byte aligned");
        hipLaunchKernelGGL(sumsq_vec, dim3(sumsq_grid((u32)c->n_cus, c->N)), dim3(256), 0, c->stream, d_vec, (u64)c->N, c->d_partials, c->max_partials,
                           (double*)(c->d_mailbox + 1));
        c->finalized = 0;   // the mailbox does not belong to a finalize any more
    } else {
        if (!c->finalized) return fail(c, DBLP_ESTATE, "phase_signal without a finalize in this round");
    }
    LAUNCH_CHECK(c, "phase_signal");
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    c->mailbox_seen = 1;
    double ss;
    memcpy(&ss, c->h_mailbox + 1, sizeof ss);
    if (ss < 0.0) ss = 0.0;     // the running sum of squares can end a rounding error below zero
    const double norm = sqrt(ss);
    if (!c->have_prev || c->prev_norm == 0.0) {
        *h_rel_delta = INFINITY;
        *h_critical = 1;
    } else {
        *h_rel_delta = fabs(c->prev_norm - norm) / c->prev_norm;
        *h_critical = *h_rel_delta >= c->eta;
    }
    *h_norm = norm;
    c->prev_norm = norm;
    c->have_prev = 1;
    return DBLP_OK;
}

// ------------------------------------------------------------------------------------------
// sum of squares without any allocation: per-block partial sums in a static device array
// ------------------------------------------------------------------------------------------
#define STATIC_PARTIALS 4096                    // blocks of one launch at most; 32 KB per GPU
#define STATIC_MAX_ELEMS (1ull << 36)           // 64 Gi floats: more than any one GPU holds
#define STATIC_MAX_DEVICES 16
static __device__ __align__(256) double static_partials[STATIC_PARTIALS];
static double* static_partials_ptr[STATIC_MAX_DEVICES];     // device address of the array on each GPU
static int static_cus[STATIC_MAX_DEVICES];
static thread_local char static_err[160] = "";

extern "C" const char* dblp_sumsq_static_error(void) { return static_err; }

extern "C" int dblp_sumsq_static(int device, void* stream, const float* d_vec, uint64_t n_elems, double* d_sumsq) {
    if (device < 0 || device >= STATIC_MAX_DEVICES) { snprintf(static_err, sizeof static_err, "sumsq_static: device ordinal outside 0..%d", STATIC_MAX_DEVICES - 1); return DBLP_EINVAL; }
    if (!d_vec || !d_sumsq) { snprintf(static_err, sizeof static_err, "sumsq_static: null pointer"); return DBLP_EINVAL; }
    if (((uintptr_t)d_vec & 15) != 0 || ((uintptr_t)d_sumsq & 7) != 0) { snprintf(static_err, sizeof static_err, "sumsq_static: d_vec must be 16-byte and d_sumsq 8-byte aligned"); return DBLP_EINVAL; }
    if (n_elems == 0 || n_elems > STATIC_MAX_ELEMS) { snprintf(static_err, sizeof static_err, "sumsq_static: n_elems must be 1..2^36"); return DBLP_EINVAL; }
    hipError_t e = hipSetDevice(device);
    if (e != hipSuccess) { snprintf(static_err, sizeof static_err, "sumsq_static: hipSetDevice: %s", hipGetErrorString(e)); return DBLP_EHIP; }
    if (!static_partials_ptr[device]) {         // once per device: where this GPU keeps its copy of the array
        double* p = nullptr;
        e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(static_partials));
        if (e != hipSuccess || !p) { snprintf(static_err, sizeof static_err, "sumsq_static: hipGetSymbolAddress: %s", hipGetErrorString(e)); (void)hipGetLastError(); return DBLP_EHIP; }
        int cus = 0;
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
        if (e != hipSuccess || cus <= 0) { (void)hipGetLastError(); cus = 256; }
        static_cus[device] = cus;
        static_partials_ptr[device] = p;
    }
    double* partials = static_partials_ptr[device];
    u32 blocks = sumsq_grid((u32)static_cus[device], n_elems);      // the grid rule of dblp_phase_signal, so the two agree to the bit
    if (blocks > STATIC_PARTIALS) blocks = STATIC_PARTIALS;
    hipLaunchKernelGGL(sumsq_blocks, dim3(blocks), dim3(256), 0, (hipStream_t)stream, d_vec, (u64)n_elems, partials);
    hipLaunchKernelGGL(reduce_partials, dim3(1), dim3(256), 0, (hipStream_t)stream, (const double*)partials, blocks, d_sumsq);
    e = hipGetLastError();
    if (e != hipSuccess) { snprintf(static_err, sizeof static_err, "sumsq_static: launch: %s", hipGetErrorString(e)); return DBLP_EHIP; }
    static_err[0] = 0;
    return DBLP_OK;
}

extern "C" int dblp_get_bitmap(dblp_ctx* c, uint64_t* d_out) {
    if (!c || !d_out) return DBLP_EINVAL;
    HIP_TRY(c, hipSetDevice(c->device));
    note_recording(c);
    HIP_TRY(c, hipMemcpyAsync(d_out, c->state[c->cur].bitmap, c->g.W * c->g.words_pw * sizeof(u64), hipMemcpyDeviceToDevice, c->stream));
    return DBLP_OK;
}

extern "C" int dblp_get_counters(dblp_ctx* c, uint64_t h[4]) {
    if (!c || !h) return DBLP_EINVAL;
    if (c->counters_in_mailbox && c->mailbox_seen) {
        // the last finalize mirrored the counters into the host mailbox and the stream has been
        // synchronised since: nothing to launch, nothing to wait for
        h[0] = c->h_mailbox[8];
        h[1] = c->h_mailbox[9] - c->h_mailbox[8];
        h[2] = c->h_mailbox[10];
        h[3] = c->h_mailbox[11];
        return DBLP_OK;
    }
    HIP_TRY(c, hipSetDevice(c->device));
    u64 tmp[C_COUNT];
    hipLaunchKernelGGL(fold_accept_rows, dim3(1), dim3(256), 0, c->stream, c->state[c->cur].rows, (u32)ACCEPT_ROWS,
                       c->state[c->cur].counters);
    LAUNCH_CHECK(c, "get_counters");
    HIP_TRY(c, hipMemcpyAsync(tmp, c->state[c->cur].counters, sizeof tmp, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    h[0] = tmp[C_ACCEPTED];
    h[1] = tmp[C_CANDIDATES] - tmp[C_ACCEPTED];   // valid arrivals that were not the first copy of their packet
    h[2] = tmp[C_STALE];
    h[3] = tmp[C_INVALID];
    return DBLP_OK;
}

extern "C" int dblp_profile_enable(dblp_ctx* c, int on) {
    if (!c) return DBLP_EINVAL;
    if (on) {
        try {
            c->timed->reserve(PROF_MAX_RECORDS);
            c->ev_pool->reserve(2 * PROF_MAX_RECORDS + 64);
        } catch (...) {
            return fail(c, DBLP_ENOMEM, "profile_enable: out of host memory");
        }
        HIP_TRY(c, hipSetDevice(c->device));
        if (!c->h_told && hipHostMalloc((void**)&c->h_told, PROF_MAX_RECORDS * sizeof(u32), hipHostMallocMapped) != hipSuccess) {
            (void)hipGetLastError();
            c->h_told = nullptr;
            return fail(c, DBLP_ENOMEM, "profile_enable: out of pinned host memory");
        }
        HIP_TRY(c, hipHostGetDevicePointer((void**)&c->d_told, c->h_told, 0));
    }
    c->profiling = on & ((1 << DBLP_K_COUNT) - 1);
    return DBLP_OK;
}

extern "C" int dblp_profile_read(dblp_ctx* c, int kernel, double* h_total_ms, uint64_t* h_launches) {
    if (!c || !h_total_ms || !h_launches || kernel < 0 || kernel >= DBLP_K_COUNT) return DBLP_EINVAL;
    HIP_TRY(c, hipSetDevice(c->device));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    double total = 0.0; u64 n = 0, n_burst = 0;
    size_t kept = 0;                      // compact in place: no allocation on this path
    for (size_t i = 0; i < c->timed->size(); ++i) {
        dblp_ctx::Timed t = (*c->timed)[i];
        if (t.kernel < 0) {               // the launch has ended and told its group
            const int wanted = -t.kernel;
            const u32 told = *(volatile u32*)(c->h_told + t.told);
            t.kernel = told == TOLD_SPARSE ? DBLP_K_GATHER_DIRECT : DBLP_K_GATHER;
            t.burst = told == TOLD_BURST;
            if (!((wanted >> t.kernel) & 1)) { c->ev_pool->push_back(t.a); c->ev_pool->push_back(t.b); continue; }
        }
        if (t.kernel != kernel) { (*c->timed)[kept++] = t; continue; }
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, t.a, t.b) == hipSuccess) { total += ms; ++n; n_burst += t.burst; } else (void)hipGetLastError();
        c->ev_pool->push_back(t.a); c->ev_pool->push_back(t.b);   // within the reserved capacity
    }
    c->timed->resize(kept);
    c->n_told = 0;                        // no record waits for an entry any more
    *h_total_ms = total; *h_launches = n;
    if (kernel == DBLP_K_GATHER) c->n_burst = n_burst;
    return DBLP_OK;
}

extern "C" int dblp_profile_bursts(const dblp_ctx* c, uint64_t* h_bursts) {
    if (!c || !h_bursts) return DBLP_EINVAL;
    *h_bursts = c->n_burst;
    return DBLP_OK;
}

extern "C" int dblp_set_prev_norm(dblp_ctx* c, double norm, int have) {
    if (!c || !(norm >= 0.0)) return DBLP_EINVAL;
    c->prev_norm = norm; c->have_prev = have != 0;
    return DBLP_OK;
}

extern "C" int dblp_get_prev_norm(const dblp_ctx* c, double* h_norm, int* h_have) {
    if (!c || !h_norm || !h_have) return DBLP_EINVAL;
    *h_norm = c->prev_norm; *h_have = c->have_prev;
    return DBLP_OK;
}

extern "C" uint32_t dblp_policy_two_level(int critical, uint32_t p_low_ppm, uint32_t p_high_ppm) {
    return critical ? p_low_ppm : p_high_ppm;
}

extern "C" uint32_t dblp_policy_three_level(double rel_delta, double eta, uint32_t tight_ppm, uint32_t mid_ppm,
                                            uint32_t loose_ppm) {
    if (rel_delta >= eta) return tight_ppm;
    return rel_delta >= 0.5 * eta ? mid_ppm : loose_ppm;
}

extern "C" uint32_t dblp_policy_linear(double rel_delta, double eta, uint32_t lo_ppm, uint32_t hi_ppm) {
    double x = rel_delta / eta;
    if (!(x < 1.0)) x = 1.0;
    const double ppm = (double)hi_ppm - ((double)hi_ppm - (double)lo_ppm) * x;
    return (uint32_t)(floor(ppm / 1000.0 + 0.5)) * 1000u;
}

extern "C" int dblp_clr_init(dblp_clr_state* st, uint32_t p_low_ppm, uint32_t p_high_ppm, uint32_t iters_per_epoch) {
    if (!st || iters_per_epoch == 0 || p_low_ppm > 1000000u || p_high_ppm > 1000000u) return DBLP_EINVAL;
    st->p_low_ppm = p_low_ppm; st->p_high_ppm = p_high_ppm; st->iters_per_epoch = iters_per_epoch;
    st->bound_ppm = p_low_ppm;      // training starts in the critical regime
    st->step = 0;
    return DBLP_OK;
}

extern "C" uint32_t dblp_clr_step(dblp_clr_state* st, int critical) {
    if (st->step % st->iters_per_epoch == 0)      // first iteration of an epoch: re-decide
        st->bound_ppm = critical ? st->p_low_ppm : st->p_high_ppm;
    st->step += 1;
    return st->bound_ppm;
}
