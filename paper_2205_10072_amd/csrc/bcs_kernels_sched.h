// Schedule construction kernels: the tables of the low levels and low rounds, receive and send rows of one p in closed
// form, and the batch of unrelated (p, r, root) triples.
#ifndef BCS_KERNELS_SCHED_H
#define BCS_KERNELS_SCHED_H

#include "bcs_kernels_common.h"
#include "bcs_rows.h"

namespace {

// ----------------------------------------------------------------------------------------------
// The low-level table of bcs_core.h lives in the code object; k_build_lowtab fills it once per device
// and process (one thread per entry, by the level walk).
// ----------------------------------------------------------------------------------------------
__device__ __align__(16) uint8_t g_lowtab[kLowTableBytes];   // read a dword at a time by stage_lowtab

__global__ __launch_bounds__(kBlock) void k_build_lowtab() {
    const int e = blockIdx.x * kBlock + threadIdx.x;
    if (e >= kLowTableBytes) return;
    const int shape = e / kLowShapeBytes;
    const int rest = e - shape * kLowShapeBytes;
    g_lowtab[e] = (uint8_t)low_table_entry(shape, rest >> 7, rest & 127);
}

// copies one shape of the table (kLowShapeBytes, a multiple of 4) into LDS; callers synchronise
__device__ __forceinline__ void stage_lowtab(uint32_t *dst, int shape) {
    const uint32_t *src = reinterpret_cast<const uint32_t *>(g_lowtab + (size_t)shape * kLowShapeBytes);
    for (int i = threadIdx.x; i < kLowShapeBytes / 4; i += kBlock) dst[i] = src[i];
}

// ----------------------------------------------------------------------------------------------
// The table of the low rounds (bcs_rows.h), 6.6 MB in the code object, filled once per device and process after the
// low-level table.  A launch reads one shape of it (103 KB, which stays in the caches), one entry a rank.
// ----------------------------------------------------------------------------------------------
__device__ __align__(16) LowRow g_lowrows[kRowsAll];

__global__ __launch_bounds__(kBlock) void k_build_lowrows() {
    const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
    if (e < kRowsAll) g_lowrows[e] = low_row_entry(e, g_lowtab);
}

// Rows of a workgroup's LDS tile of bytes (rank-major, Q bytes a rank, so the tile is the table's piece with one byte
// an entry) to their place in the rank-major int32 table: a lane reads four bytes, widens them and writes 16 bytes.
template <int Q, int LANES>
__device__ __forceinline__ void byte_tile_to_rows(const int8_t *tile, uint32_t rows, int32_t *__restrict__ dst) {
    const uint32_t n = rows * Q;
    if ((reinterpret_cast<uintptr_t>(dst) & 15u) == 0) {
        const uint32_t n4 = n >> 2;
        for (uint32_t g = threadIdx.x; g < n4; g += LANES) {
            const int32_t w = reinterpret_cast<const int32_t *>(tile)[g];
            const v4i pack = {(int32_t)(int8_t)w, (int32_t)(int8_t)(w >> 8), (int32_t)(int8_t)(w >> 16), w >> 24};
            __builtin_nontemporal_store(pack, reinterpret_cast<v4i *>(dst) + g);
        }
        const uint32_t e = (n4 << 2) + threadIdx.x;
        if (e < n) dst[e] = tile[e];
        return;
    }
    for (uint32_t e = threadIdx.x; e < n; e += LANES) dst[e] = tile[e];
}

// The same rows as bytes for an expansion that follows: T[k] = entry[k] - k, the first three once more, padding.
template <int Q, int LANES>
__device__ __forceinline__ void byte_tile_to_byte_rows(const int8_t *tile, uint32_t rows, int8_t *__restrict__ dst) {
    constexpr uint32_t kW4 = byte_row_stride(Q) / 4;
    uint32_t *out4 = reinterpret_cast<uint32_t *>(dst);
    for (uint32_t w = threadIdx.x; w < rows * kW4; w += LANES) {
        const uint32_t row = w / kW4, pos0 = 4u * (w - row * kW4);
        uint32_t packed = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t pos = pos0 + c;
            const uint32_t slot = pos < (uint32_t)Q ? pos : pos - Q;
            const bool slot_ok = pos < (uint32_t)(Q + 3) && slot < (uint32_t)Q;
            const int32_t t = slot_ok ? (int32_t)tile[row * Q + slot] - (int32_t)slot : 0;
            packed |= ((uint32_t)t & 0xffu) << (8 * c);
        }
        out4[w] = packed;
    }
}

// ----------------------------------------------------------------------------------------------
// K1: receive and send rows of ranks [r0, r1), one p per launch, from the closed form in bcs_rows.h.  Lane = rank.
// A workgroup takes kTileRanks ranks.  The entries of rounds 7 and up, of both tables, follow from a lane's own digits
// (about eight vector ops a level); those of the receive rounds below 7 are one 8-byte table entry; those of the send
// rounds below 7 are entries of the next skips[6] <= 64 ranks, so kTileAhead more lanes compute the low rounds alone and
// the send entries are read across the lanes in LDS.  Both tables' rows are staged in LDS as bytes, laid out like the
// table, and leave widened to int32 in 16-byte streaming stores.  Nothing else is read or written: no table of
// all ranks in memory, no second pass, and a range of ranks costs the same a rank as all of them.
// Bound by the stores.  Measured: all ranks of 2^27-1, 29 GB, 7.31 ms before (digit table, receive rows by windows, send
// rows by look-up in a slot-major table), 5.22 ms now; all of 2^20+1 59 -> 34 us; 2^24 ranks of 2^27-1 1.10 -> 0.62 ms.
// ----------------------------------------------------------------------------------------------
constexpr int kTileRanks = 256;
constexpr int kTileAhead = 64;
constexpr int kTileLanes = kTileRanks + kTileAhead;
constexpr int kWantRecv = 1, kWantSend = 2;

template <int Q>
struct RowTiles {
    __align__(16) int8_t recv[kTileRanks * Q + 16];
    __align__(16) int8_t send[kTileRanks * Q + 16];
    LowRow low[kTileLanes];                                       // entries of the rounds below 7, as bytes
};

template <int Q, int WANT>
__device__ __forceinline__ void fill_row_tiles(const SkipTab &tab, uint32_t root, uint32_t first_rank, RowTiles<Q> &tiles) {
    Uniform<Q> pol;
#pragma unroll
    for (int k = 0; k <= Q; ++k) pol.S[k] = tab.s[k];
    pol.tab = &tab;
    pol.low = nullptr;
    const uint32_t p = pol.p();
    uint32_t r = first_rank + threadIdx.x;                        // lanes past the end wrap around like the look-ahead
    if constexpr (Q < 10) r %= p;                                 // p < 513 may be below the tile's lanes
    else r = r >= p ? r - p : r;
    const uint32_t v = r >= root ? r - root : r + p - root;
    const uint32_t base = row_base(pol);
    const RankPlace pl = rank_place(pol, v);
    const LowRow w = g_lowrows[base + pl.ctx * 128u + pl.low];
    const LowRow b = row_bytes(w, pl.ctx, pl.J, (uint32_t)Q);
    if constexpr ((WANT & kWantSend) != 0) tiles.low[threadIdx.x] = b;
    const bool own_rank = threadIdx.x < (uint32_t)kTileRanks;     // wave-uniform
    int8_t *my_recv = tiles.recv + threadIdx.x * Q;
    int8_t *my_send = tiles.send + threadIdx.x * Q;
    constexpr int kLow = Q < kLowLevels ? Q : kLowLevels;
    if (own_rank) {
        if constexpr ((WANT & kWantRecv) != 0) {
#pragma unroll
            for (int k = 0; k < kLow; ++k) my_recv[k] = (int8_t)(k < 4 ? b.lo >> (8 * k) : b.hi >> (8 * (k - 4)));
        }
        high_entries(pol, pl, place_own(pl, w),
                     [&](int k, int32_t e) { if constexpr ((WANT & kWantRecv) != 0) my_recv[k] = (int8_t)e; },
                     [&](int k, int32_t e) { if constexpr ((WANT & kWantSend) != 0) my_send[k] = (int8_t)e; });
        if constexpr ((WANT & kWantRecv) != 0) recv_fix(pol, pl, w, [&](int k, int32_t e) { my_recv[k] = (int8_t)e; });
        if constexpr ((WANT & kWantSend) != 0)
            send_fix(pol, v, pl, base, [](uint32_t e) { return g_lowrows[e]; }, [&](int k, int32_t e) { my_send[k] = (int8_t)e; });
    }
    __syncthreads();
    if constexpr ((WANT & kWantSend) != 0) {
        if (own_rank) {
            const int8_t *low = reinterpret_cast<const int8_t *>(tiles.low);
#pragma unroll
            for (int k = 0; k < kLow; ++k) my_send[k] = low[(threadIdx.x + pol.S[k]) * 8u + k];
        }
        __syncthreads();
    }
}

template <int Q, int WANT>
__global__ __launch_bounds__(kTileLanes) void k_sched(const SkipTab tab, uint32_t root, uint32_t r0, uint32_t r1,
                                                      int32_t *__restrict__ recv_out, int32_t *__restrict__ send_out,
                                                      slot_t *__restrict__ recvT, uint64_t ldT,
                                                      int8_t *__restrict__ recvB, int8_t *__restrict__ sendB) {
    __shared__ RowTiles<Q> tiles;
    const uint64_t first = (uint64_t)blockIdx.x * kTileRanks;     // offset of this tile inside [r0, r1)
    fill_row_tiles<Q, WANT>(tab, root, r0 + (uint32_t)first, tiles);
    const uint64_t left = (uint64_t)r1 - r0 - first;
    const uint32_t rows = left < (uint64_t)kTileRanks ? (uint32_t)left : (uint32_t)kTileRanks;
    if constexpr ((WANT & kWantRecv) != 0) {
        if (recv_out) byte_tile_to_rows<Q, kTileLanes>(tiles.recv, rows, recv_out + first * Q);
        if (recvB) byte_tile_to_byte_rows<Q, kTileLanes>(tiles.recv, rows, recvB + first * byte_row_stride(Q));
        if (recvT) {
            // slot-major: each slot's kTileRanks bytes are one aligned piece of the table, whose rows are padded to a
            // multiple of them (the last tile writes its idle lanes' bytes into the padding)
            for (uint32_t g = threadIdx.x; g < (uint32_t)Q * (kTileRanks / 4); g += kTileLanes) {
                const uint32_t k = g / (kTileRanks / 4), four = g % (kTileRanks / 4);
                uint32_t packed = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) packed |= (uint32_t)(uint8_t)tiles.recv[(four * 4u + c) * Q + k] << (8 * c);
                *reinterpret_cast<uint32_t *>(recvT + (uint64_t)k * ldT + first + four * 4u) = packed;
            }
        }
    }
    if constexpr ((WANT & kWantSend) != 0) {
        if (send_out) byte_tile_to_rows<Q, kTileLanes>(tiles.send, rows, send_out + first * Q);
        if (sendB) byte_tile_to_byte_rows<Q, kTileLanes>(tiles.send, rows, sendB + first * byte_row_stride(Q));
    }
}

// Work lists for send entries left to Alg. 5 (k_batch).  Each lane working down its own entries
// makes a wave run as many turns as its unluckiest lane has entries, each turn as far as the largest k any lane asked
// for; so the entries named by the lanes' masks (bit k of lane L: entry (L, k)) are made one list of the workgroup,
// ranked by k and then by lane, and handed out one entry a lane: neighbouring places hold entries of the same k (and,
// in the batch kernel, whose lanes are in the order of q, of neighbouring q), and a wave's loops run about as far as
// each of its lanes needs.  Entry (L, k) goes to place
// kstart[k] + (entries for k in earlier waves) + (earlier lanes of L's wave with bit k), found with ballots.  The
// list is filled and handed out QUEUE entries at a time (QUEUE a multiple of BLOCK, the workgroup's lanes), one entry a lane: fn(has, who, k) runs in every lane of
// every wave that has an entry.  All lanes of the workgroup must call this (it synchronises them).
template <int BLOCK, int QUEUE, class Fn>
__device__ __forceinline__ void work_list(uint32_t mask, uint32_t (*wcnt)[32], uint32_t *kstart, uint16_t *queue, Fn fn) {
    static_assert(QUEUE % BLOCK == 0 && BLOCK % 64 == 0 && BLOCK <= 2048, "whole waves; a lane index and k share 16 bits");
    const int wave = threadIdx.x >> 6;
    // the k for which any lane of this wave has an entry (wave-uniform): the loops below visit only these
    uint32_t any_k = mask;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) any_k |= (uint32_t)__shfl_xor((int)any_k, off, 64);
    any_k = __builtin_amdgcn_readfirstlane(any_k);
    __syncthreads();                                        // earlier users of wcnt / kstart / queue are done
    {
        uint32_t mine = 0;                                  // lane k of a wave: the wave's entries for k
        for (uint32_t m = any_k; m != 0u; m &= m - 1u) {
            const int k = __builtin_ctz(m);
            const uint32_t c = (uint32_t)__popcll(__ballot((mask >> k) & 1u));
            mine = (threadIdx.x & 63u) == (uint32_t)k ? c : mine;
        }
        if ((threadIdx.x & 63u) < 32u) wcnt[wave][threadIdx.x & 63u] = mine;
    }
    __syncthreads();
    if (threadIdx.x < 32) {                                 // entries for k = threadIdx.x: running count over the waves
        uint32_t acc = 0;
        for (int w = 0; w < BLOCK / 64; ++w) {
            const uint32_t c = wcnt[w][threadIdx.x];
            wcnt[w][threadIdx.x] = acc;
            acc += c;
        }
        kstart[threadIdx.x] = acc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t acc = 0;
        for (int k = 0; k < 32; ++k) {
            const uint32_t c = kstart[k];
            kstart[k] = acc;
            acc += c;
        }
        kstart[32] = acc;
    }
    __syncthreads();
    const uint32_t total = kstart[32];
    for (uint32_t base = 0; base < total; base += QUEUE) {
        for (uint32_t m = any_k; m != 0u; m &= m - 1u) {
            const int k = __builtin_ctz(m);
            const uint64_t bal = __ballot((mask >> k) & 1u);
            const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            const uint32_t place = kstart[k] + wcnt[wave][k] + before - base;
            if (((mask >> k) & 1u) && place < (uint32_t)QUEUE) queue[place] = (uint16_t)((threadIdx.x << 5) | (uint32_t)k);
        }
        __syncthreads();
        const uint32_t n = total - base < (uint32_t)QUEUE ? total - base : (uint32_t)QUEUE;
        for (uint32_t e0 = 0; e0 < n; e0 += BLOCK) {   // workgroup-uniform
            if (e0 + (threadIdx.x & ~63u) >= n) continue;    // a wave with no entry left (wave-uniform)
            const uint32_t e = e0 + threadIdx.x;
            const bool has = e < n;
            const uint32_t entry = has ? queue[e] : 0u;
            fn(has, entry >> 5, has ? (int)(entry & 31u) : -1);
        }
        __syncthreads();                                    // the next part of the list overwrites the queue
    }
}

// K3: unrelated (p, r, root) triples; rows of BCS_BATCH_STRIDE ints (one 128-byte line each), padded.
// A workgroup takes kBatchBlock triples and first orders them by q in LDS (counting sort), because a
// wave runs its level loops to the largest q among its lanes and the work grows like q^3: after the
// sort a wave holds neighbouring q only.  Each lane then builds the rows of its triple into an LDS tile of
// bytes (entries lie in [-31, 30]; a byte of -128 stands for the padding), at the triple's place in the
// input order; the workgroup then writes the tile out as whole 128-byte lines, eight lanes a row and 16 bytes
// a lane.  (Storing each entry straight into its row, 4 bytes at a time into a line of the lane's own, made the
// memory system write five times the table's bytes as partial lines, and a call for receive rows alone was
// bound by those stores: measured 0.254 ms with the vector ALU busy 28 % of the time.)
constexpr int kBatchBlock = 1024;
constexpr int kBatchRowBytes = BCS_BATCH_STRIDE + 4;       // LDS row stride: nine words, so lanes' rows spread over the banks
constexpr int8_t kBatchPadByte = -128;
constexpr int kQueue = 4 * kBatchBlock;                    // entries of the Alg. 5 work list held at a time

// the workgroup's byte tile -> rows of the table (after a barrier); `rows` = triples of this workgroup that exist
__device__ __forceinline__ void batch_rows_out(const int8_t *tileB, uint32_t rows, int32_t *__restrict__ dst) {
    const bool vec = (reinterpret_cast<uintptr_t>(dst) & 15u) == 0;
#pragma unroll
    for (int it = 0; it < BCS_BATCH_STRIDE / 4; ++it) {
        const uint32_t g = (uint32_t)it * kBatchBlock + threadIdx.x;
        const uint32_t row = g >> 3, part = g & 7u;
        if (row >= rows) continue;
        const uint32_t four = *reinterpret_cast<const uint32_t *>(tileB + row * kBatchRowBytes + part * 4u);
        int32_t v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int32_t b = (int32_t)(int8_t)(four >> (8 * c));
            v[c] = b == (int32_t)kBatchPadByte ? BCS_BATCH_PAD : b;
        }
        int32_t *out = dst + (uint64_t)row * BCS_BATCH_STRIDE + part * 4u;
        if (vec) {
            const v4i pack = {v[0], v[1], v[2], v[3]};
            *reinterpret_cast<v4i *>(out) = pack;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) out[c] = v[c];
        }
    }
}

// One entry of a work list of the batch kernel, as the lane that works on it sees it: the triple `who` of the
// workgroup (its p and rank from the sorted arrays), the entry's k, the to-neighbour t = (v + skips[k]) mod p, and
// a policy whose level loops run as far as the wave's largest q; kmax is the wave's largest k.  Lanes without an
// entry (has = false, kk = -1) stand in with p = 1.
struct BatchLane {
    PerLane pol;
    uint32_t t, orig;
    int kmax;
};
__device__ __forceinline__ BatchLane batch_lane(bool has, uint32_t who, int kk, const uint32_t *s_p, const uint32_t *s_v,
                                                const uint32_t *s_slot) {
    BatchLane e;
    const uint32_t p = has ? s_p[who] : 1u, v = has ? s_v[who] : 0u;
    e.orig = s_slot[who] & 0xffffu;
    const int q = ceil_log2(p);
    int kmax = kk, qtop = q;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const int ok = __shfl_xor(kmax, off, 64), oq = __shfl_xor(qtop, off, 64);
        kmax = ok > kmax ? ok : kmax;
        qtop = oq > qtop ? oq : qtop;
    }
    e.kmax = __builtin_amdgcn_readfirstlane(kmax);
    e.pol.pm1 = p - 1u;
    e.pol.ql = q;
    e.pol.wave_top = __builtin_amdgcn_readfirstlane(qtop) - 1;
    e.pol.odd = odd_levels(p, q);
    e.pol.low = g_lowtab + (size_t)low_shape(p, q) * kLowShapeBytes;
    const uint32_t t = v + (kk >= 0 ? e.pol.s(kk) : 0u);
    e.t = t >= p ? t - p : t;
    return e;
}

__global__ __launch_bounds__(kBatchBlock) void k_batch(int64_t count, const int32_t *__restrict__ pv,
                                                       const int32_t *__restrict__ rv,
                                                       const int32_t *__restrict__ rootv,
                                                       int32_t *__restrict__ recv_out, int32_t *__restrict__ send_out,
                                                       int32_t *__restrict__ q_out) {
    __shared__ uint32_t bins[33];                 // bins[q] for valid triples, bins[32] for the rest
    __shared__ uint32_t start[33];
    __shared__ uint32_t s_p[kBatchBlock], s_v[kBatchBlock], s_slot[kBatchBlock];
    __shared__ __align__(16) int8_t tileB[kBatchBlock * kBatchRowBytes];
    __shared__ uint32_t wcnt[kBatchBlock / 64][32];            // send entries left to Alg. 5: per wave and k, then their offsets
    __shared__ uint32_t kstart[33];
    __shared__ uint16_t queue[kQueue];                         // the work list: (lane << 5) | k
    const int64_t first = (int64_t)blockIdx.x * kBatchBlock;
    {
        const int64_t idx = first + threadIdx.x;
        const bool live = idx < count;
        const int32_t pi = live ? pv[idx] : 1, ri = live ? rv[idx] : 0, rooti = live ? rootv[idx] : 0;
        const bool valid = live && pi >= 1 && ri >= 0 && ri < pi && rooti >= 0 && rooti < pi;
        const uint32_t p = valid ? (uint32_t)pi : 1u;
        const int q = ceil_log2(p);
        const uint32_t v = !valid ? 0u
                           : ((uint32_t)ri >= (uint32_t)rooti ? (uint32_t)(ri - rooti)
                                                              : (uint32_t)ri + p - (uint32_t)rooti);
        if (threadIdx.x < 33) bins[threadIdx.x] = 0u;
        __syncthreads();
        const int bin = valid ? q : 32;
        const uint32_t rank_in_bin = atomicAdd(&bins[bin], 1u);
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t acc = 0;
            for (int k = 0; k < 33; ++k) {
                start[k] = acc;
                acc += bins[k];
            }
        }
        __syncthreads();
        const uint32_t pos = start[bin] + rank_in_bin;
        s_p[pos] = p;
        s_v[pos] = v;
        s_slot[pos] = threadIdx.x | (valid ? 0u : 0x80000000u) | (live ? 0u : 0x40000000u);
        __syncthreads();
    }
    // from here on this lane works on the triple that the sort put at its position
    const uint32_t p = s_p[threadIdx.x];
    const uint32_t v = s_v[threadIdx.x];
    const uint32_t slot = s_slot[threadIdx.x];
    const bool valid = (slot & 0x80000000u) == 0u;
    const bool live = (slot & 0x40000000u) == 0u;
    const uint32_t orig = slot & 0xffffu;                     // the triple's place among the workgroup's 1024
    const int64_t idx = first + orig;
    const int q = ceil_log2(p);
    if (live && q_out) q_out[idx] = valid ? q : -1;
    // largest q in this wave bounds the level loops of all its lanes
    int qmax = q;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const int other = __shfl_xor(qmax, off, 64);
        qmax = other > qmax ? other : qmax;
    }
    qmax = __builtin_amdgcn_readfirstlane(qmax);   // the same in every lane: a scalar, so the loops it bounds are scalar loops
    PerLane pol;
    pol.pm1 = p - 1u;
    pol.ql = q;
    pol.wave_top = qmax - 1;
    pol.odd = odd_levels(p, q);
    pol.low = g_lowtab + (size_t)low_shape(p, q) * kLowShapeBytes;
    const uint32_t rows = (count - first) < (int64_t)kBatchBlock ? (uint32_t)(count - first) : (uint32_t)kBatchBlock;
    int8_t *my = tileB + orig * kBatchRowBytes;
    uint32_t *my4 = reinterpret_cast<uint32_t *>(my);
    const uint32_t pad4 = 0x80808080u;
    if (recv_out) {
#pragma unroll
        for (int w = 0; w < BCS_BATCH_STRIDE / 4; ++w) my4[w] = pad4;
        recv_row(pol, v, qmax - 1, [&](int i, int val) { my[i] = (int8_t)val; });
        __syncthreads();
        batch_rows_out(tileB, rows, recv_out + first * BCS_BATCH_STRIDE);
        __syncthreads();
    }
    if (send_out) {
#pragma unroll
        for (int w = 0; w < BCS_BATCH_STRIDE / 4; ++w) my4[w] = pad4;
        // the entries that need none of the to-neighbour's rounds (send_row_direct); the others are left in `pending`
        const uint32_t pending = send_row_direct(pol, v, digits(pol, v), [&](uint32_t y) { return digits(pol, y); },
                                                 [&](int k, int val) { my[k] = (int8_t)val; });
        // Those are worked off as one list of the whole workgroup, one entry a lane.  (Each lane working down its
        // own entries made a wave run as many turns as its unluckiest lane has entries, each turn as far as the
        // largest k any lane asked for: five times the lane-operations the entries themselves need, by a count on
        // the C5 triples, where a triple leaves 1.8 entries on average, nearly all below level 8.)
        // Alg. 5 for the rest: rounds 0..k of the to-neighbour's receive row, of which entry k is kept (a wave
        // computes as many rounds as its largest k; receive rows are prefix-stable, the extra rounds change nothing)
        work_list<kBatchBlock, kQueue>(pending, wcnt, kstart, queue, [&](bool has, uint32_t who, int kk) {
            const BatchLane e = batch_lane(has, who, kk, s_p, s_v, s_slot);
            int32_t keep = 0;
            recv_row(e.pol, e.t, e.kmax, [&](int j, int val) { keep = (j == kk) ? val : keep; });
            if (has) tileB[e.orig * kBatchRowBytes + kk] = (int8_t)keep;
        });
        __syncthreads();
        batch_rows_out(tileB, rows, send_out + first * BCS_BATCH_STRIDE);
    }
}

}  // namespace

#endif  // BCS_KERNELS_SCHED_H
