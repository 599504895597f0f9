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
__device__ __align__(16) uint8_t g_lowtab[kLowTableBytes];   // read by k_build_lowrows

__global__ __launch_bounds__(kBlock) void k_build_lowtab() {
    const int e = blockIdx.x * kBlock + threadIdx.x;
    if (e >= kLowTableBytes) return;
    const int shape = e / kLowShapeBytes;
    const int rest = e - shape * kLowShapeBytes;
    g_lowtab[e] = (uint8_t)low_table_entry(shape, rest >> 7, rest & 127);
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

// n entries of the rank-major int32 table from a workgroup's LDS tile of bytes, which is laid out like the table's piece
// with one byte an entry: a lane reads four bytes, widens them and writes 16 bytes.
template <int LANES>
__device__ __forceinline__ void byte_tile_to_table(const int8_t *tile, uint32_t n, bool stream, int32_t *__restrict__ dst) {
    if ((reinterpret_cast<uintptr_t>(dst) & 15u) == 0) {
        const uint32_t n4 = n >> 2;
        for (uint32_t g = threadIdx.x; g < n4; g += LANES) {
            const int32_t w = reinterpret_cast<const int32_t *>(tile)[g];
            const v4i pack = {(int32_t)(int8_t)w, (int32_t)(int8_t)(w >> 8), (int32_t)(int8_t)(w >> 16), w >> 24};
            if (stream) __builtin_nontemporal_store(pack, reinterpret_cast<v4i *>(dst) + g);
            else reinterpret_cast<v4i *>(dst)[g] = pack;
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
// The entries of rounds 7 and up follow from a lane's own digits (about eight vector ops a level); those of the receive
// rounds below 7 are one 8-byte table entry, those of the send rounds below 7 seven such entries (of the ranks up to 64
// further on).  Rows are staged in LDS as bytes, laid out like the table, and leave widened to int32 in 16-byte stores.
// Nothing else of the tables' size is read or written: no table of all ranks in memory, no second pass, and a range of
// ranks costs the same a rank as all of them.
// Bound by the stores, and what a workgroup writes decides how fast they go.  Store-only kernels, whose workgroups take
// pieces of two 4 GB tables in turn, reach 6.3-7.0 TB/s with 4 KB pieces (64 to 256 lanes), 6.2-6.5 with 8 KB, and
// 5.6-5.8 with 6.9, 13.8 or 27.6 KB (64, 128 or 256 rows at q = 27).  So the tables are cut by entries, not by rows: a
// workgroup is one wave and takes 4 KB of ONE table, neighbouring workgroups take the two tables in turn, and a row that
// lies across two pieces is built twice.  2^24 ranks of 2^27-1 (3.6 GB): 0.55 ms so, 0.64 with 12 KB and 128 lanes or with
// whole rows; the construction without the stores takes 0.42 ms.  Plain stores beat streaming ones (by 17 % where the tables
// fit the memory-side cache) except where byte rows are left for an expansion, which then finds them in the caches.
// Measured: all ranks of 2^27-1, 29 GB, 7.30 ms before (digit table, receive rows by windows, send rows by look-up in a
// slot-major table), 4.38 ms now; all of 2^20+1 57 -> 31 us; 2^24 ranks of 2^27-1 1.11 -> 0.54 ms.
// ----------------------------------------------------------------------------------------------
constexpr int kSchedLanes = 64;
constexpr uint32_t kWantRecv = 1, kWantSend = 2;

// entries of one table that a workgroup writes (by_rows: whole rows, for the slot-major copy)
inline uint32_t sched_piece(int q, bool by_rows) {
    const bool fits = (kSchedLanes - 1) * q >= 1024;                        // a piece may begin inside a row; q >= 17
    return by_rows || !fits ? (uint32_t)(kSchedLanes * q) : 1024u;
}

template <int Q>
__global__ __launch_bounds__(kSchedLanes) void k_sched(const SkipTab tab, uint32_t root, uint32_t r0, uint32_t r1,
                                                       uint32_t want, uint32_t piece, int32_t *__restrict__ recv_out,
                                                       int32_t *__restrict__ send_out, slot_t *__restrict__ recvT,
                                                       uint64_t ldT, int8_t *__restrict__ recvB,
                                                       int8_t *__restrict__ sendB) {
    // a row begins up to Q - 1 entries before the piece: the piece's first entry sits at a 16-byte boundary behind them
    __shared__ __align__(16) int8_t tile_all[32 + kSchedLanes * Q + 16];
    int8_t *const tile = tile_all + 32;
    constexpr int kLow = Q < kLowLevels ? Q : kLowLevels;
    const bool both = want == (kWantRecv | kWantSend);
    const bool send = both ? (blockIdx.x & 1u) != 0u : want == kWantSend;
    const uint64_t e0 = (uint64_t)(both ? blockIdx.x >> 1 : blockIdx.x) * piece;      // first entry of the piece
    const uint32_t first = (uint32_t)(e0 / Q);                                         // its row, an offset inside [r0, r1)
    const uint32_t ahead = (uint32_t)(e0 - (uint64_t)first * Q);                       // entries of that row before it
    const uint32_t count = r1 - r0, left = count - first;                              // left > 0: the grid covers the table
    Uniform<Q> pol;
#pragma unroll
    for (int k = 0; k <= Q; ++k) pol.S[k] = tab.s[k];
    pol.tab = &tab;
    pol.low = nullptr;
    const uint32_t p = pol.p();
    const uint32_t r = r0 + first + (threadIdx.x < left ? threadIdx.x : 0u);           // lanes past the end repeat a rank
    const uint32_t v = r >= root ? r - root : r + p - root;
    const uint32_t base = row_base(pol);
    const RankPlace pl = rank_place(pol, v);
    const LowRow w = g_lowrows[base + pl.ctx * 128u + pl.low];
    const uint32_t own = place_own(pl, w);
    int8_t *my = tile + (int)(threadIdx.x * Q) - (int)ahead;
    auto read = [](uint32_t e) { return g_lowrows[e]; };
    auto keep = [&](int k, int32_t e) { my[k] = (int8_t)e; };
    auto drop = [](int, int32_t) {};
    if (send) {
        send_low_entries(pol, pl, base, read, [&](int k, int32_t e) { if (k < kLow) my[k] = (int8_t)e; });
        high_entries(pol, pl, own, drop, keep);
        send_fix(pol, v, pl, base, read, keep);
    } else {
        const LowRow b = row_bytes(w, pl.ctx, pl.J, (uint32_t)Q);
#pragma unroll
        for (int k = 0; k < kLow; ++k) my[k] = (int8_t)(k < 4 ? b.lo >> (8 * k) : b.hi >> (8 * (k - 4)));
        high_entries(pol, pl, own, keep, drop);
        recv_fix(pol, pl, w, keep);
    }
    __syncthreads();
    int32_t *const out = send ? send_out : recv_out;
    int8_t *const outB = send ? sendB : recvB;
    const uint64_t rest = (uint64_t)count * Q - e0;
    if (out) byte_tile_to_table<kSchedLanes>(tile, rest < piece ? (uint32_t)rest : piece, outB != nullptr, out + e0);
    if (outB) {
        // the rows that begin in the piece
        const uint32_t skip = ahead ? 1u : 0u;
        const uint32_t end = (ahead + piece + Q - 1u) / Q;                             // at most kSchedLanes
        byte_tile_to_byte_rows<Q, kSchedLanes>(tile + (int)(skip * Q) - (int)ahead, (end < left ? end : left) - skip,
                                               outB + ((uint64_t)first + skip) * byte_row_stride(Q));
    }
    if (!send && recvT) {
        // slot-major, a launch by whole rows: each slot's kSchedLanes bytes are one aligned piece of the table, whose rows
        // are padded to a multiple of them (the last tile writes its idle lanes' bytes into the padding)
        for (uint32_t g = threadIdx.x; g < (uint32_t)Q * (kSchedLanes / 4); g += kSchedLanes) {
            const uint32_t k = g / (kSchedLanes / 4), four = g % (kSchedLanes / 4);
            uint32_t packed = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) packed |= (uint32_t)(uint8_t)tile[(four * 4u + c) * Q + k] << (8 * c);
            *reinterpret_cast<uint32_t *>(recvT + (uint64_t)k * ldT + first + four * 4u) = packed;
        }
    }
}

// K3: unrelated (p, r, root) triples; rows of BCS_BATCH_STRIDE ints (one 128-byte line each), padded.  Lane = triple, in
// the closed form of bcs_rows.h with a p per lane.  A wave's level loops run to the largest q among its lanes; a step is
// a dozen vector ops, so ordering the triples by q first (which the construction by windows needed) would cost more than
// the idle steps.  The send entries below round 7 are read from the table entry by entry (seven 8-byte reads a lane
// within 1 KB of one another).  Rows are built as bytes in LDS, four levels to a word (entries lie in [-31, 30]; a byte
// of -128 stands for the padding); the workgroup then writes them as whole 128-byte lines, eight lanes a row and 16
// bytes a lane.  (Storing each entry straight into its row, 4 bytes at a time into a line of the lane's own, makes the
// memory system write five times the table's bytes as partial lines.)
// Bound by the stores: 2^20 triples of mixed q, both tables (268 MB written), 236 us by windows and Alg. 5, 54 us now.
constexpr int kBatchBlock = 256;
constexpr int kBatchRowBytes = BCS_BATCH_STRIDE + 4;       // LDS row stride: nine words, so lanes' rows spread over the banks
constexpr int8_t kBatchPadByte = -128;

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
            __builtin_nontemporal_store(pack, reinterpret_cast<v4i *>(out));
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) out[c] = v[c];
        }
    }
}

// bytes 0..n-1 of `four`, padding above (n may be any number)
__device__ __forceinline__ uint32_t batch_pad(uint32_t four, int n) {
    const uint32_t keep = n >= 4 ? 0xffffffffu : (n > 0 ? (1u << (8 * n)) - 1u : 0u);
    return (four & keep) | (0x80808080u & ~keep);
}

__global__ __launch_bounds__(kBatchBlock) void k_batch(int64_t count, const int32_t *__restrict__ pv,
                                                       const int32_t *__restrict__ rv,
                                                       const int32_t *__restrict__ rootv,
                                                       int32_t *__restrict__ recv_out, int32_t *__restrict__ send_out,
                                                       int32_t *__restrict__ q_out) {
    __shared__ __align__(16) int8_t tile_recv[kBatchBlock * kBatchRowBytes];
    __shared__ __align__(16) int8_t tile_send[kBatchBlock * kBatchRowBytes];
    const int64_t first = (int64_t)blockIdx.x * kBatchBlock;
    const int64_t idx = first + threadIdx.x;
    const bool live = idx < count;
    const int32_t pi = live ? pv[idx] : 1, ri = live ? rv[idx] : 0, rooti = live ? rootv[idx] : 0;
    const bool valid = live && pi >= 1 && ri >= 0 && ri < pi && rooti >= 0 && rooti < pi;
    const uint32_t p = valid ? (uint32_t)pi : 1u;             // an invalid triple stands in with p = 1: rows of padding
    const uint32_t v = !valid ? 0u
                       : ((uint32_t)ri >= (uint32_t)rooti ? (uint32_t)(ri - rooti)
                                                          : (uint32_t)ri + p - (uint32_t)rooti);
    const int q = ceil_log2(p);
    if (live && q_out) q_out[idx] = valid ? q : -1;
    if (!recv_out && !send_out) return;
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
    pol.low = nullptr;
    const uint32_t base = row_base(pol);
    const RankPlace pl = rank_place(pol, v);
    const LowRow w = g_lowrows[base + pl.ctx * 128u + pl.low];
    const LowRow b = row_bytes(w, pl.ctx, pl.J, (uint32_t)q);
    LowRow s = {0u, 0u};
    if (send_out)
        send_low_entries(pol, pl, base, [](uint32_t e) { return g_lowrows[e]; }, [&](int k, int32_t e) {
            if (k < 4) s.lo |= ((uint32_t)e & 0xffu) << (8 * k);
            else s.hi |= ((uint32_t)e & 0xffu) << (8 * (k - 4));
        });
    int8_t *my_recv = tile_recv + threadIdx.x * kBatchRowBytes, *my_send = tile_send + threadIdx.x * kBatchRowBytes;
    uint32_t *recv4 = reinterpret_cast<uint32_t *>(my_recv), *send4 = reinterpret_cast<uint32_t *>(my_send);
    // rounds 7 and up, largest first, as in high_entries; a word takes levels 4 i .. 4 i + 3
    const uint32_t bare = pl.up & ~(1u << (q & 31));
    int32_t next = (int32_t)place_own(pl, w);
#pragma unroll
    for (int i = BCS_BATCH_STRIDE / 4 - 1; i >= 1; --i) {
        if (4 * i >= qmax) {                                  // wave-uniform
            recv4[i] = send4[i] = 0x80808080u;
            continue;
        }
        uint32_t wr = 0, ws = 0;
#pragma unroll
        for (int c = 3; c >= 0; --c) {
            const int k = 4 * i + c;
            if (k < kLowLevels) continue;
            const int32_t set = -(int32_t)((bare >> (k & 31)) & 1u), here = k - q;
            const int32_t r = (set & next) | (~set & here);
            next = (set & here) | (~set & next);
            wr = __builtin_amdgcn_perm(wr, (uint32_t)r, 0x06050400u);        // the word up by a byte, r's byte below
            ws = __builtin_amdgcn_perm(ws, (uint32_t)next, 0x06050400u);
        }
        if (i == 1) {                                         // level 7 above the table's bytes 4..6
            wr = (wr << 24) | (b.hi & 0xffffffu);
            ws = (ws << 24) | (s.hi & 0xffffffu);
        }
        recv4[i] = batch_pad(wr, q - 4 * i);
        send4[i] = batch_pad(ws, q - 4 * i);
    }
    recv4[0] = batch_pad(b.lo, q);
    send4[0] = batch_pad(s.lo, q);
    recv_fix(pol, pl, w, [&](int k, int32_t e) { my_recv[k] = (int8_t)e; });
    if (send_out)
        send_fix(pol, v, pl, base, [](uint32_t e) { return g_lowrows[e]; }, [&](int k, int32_t e) { my_send[k] = (int8_t)e; });
    __syncthreads();
    const uint32_t rows = (count - first) < (int64_t)kBatchBlock ? (uint32_t)(count - first) : (uint32_t)kBatchBlock;
    if (recv_out) batch_rows_out(tile_recv, rows, recv_out + first * BCS_BATCH_STRIDE);
    if (send_out) batch_rows_out(tile_send, rows, send_out + first * BCS_BATCH_STRIDE);
}

}  // namespace

#endif  // BCS_KERNELS_SCHED_H
