// libbcsched: round-optimal broadcast schedules on a circulant graph, built on gfx950.
//
// Method: J. L. Traff, arXiv 2205.10072, Section 2 (Alg. 1, 2, 4, 5; index arithmetic of Alg. 6).
// One lane owns one rank.  Everything is 32-bit integer work on the vector ALU; block sets are
// 32-bit masks (q <= 31); the skips of a uniform-p launch live in scalar registers.
//
// The per-rank construction is in bcs_rows.h (its definition by windows in bcs_core.h), the kernels in bcs_kernels_*.h; this
// file holds the launch and timing helpers, the host logic and the C ABI.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <initializer_list>
#include <mutex>
#include <utility>

#include "bcsched.h"
#include "bcs_core.h"
#include "bcs_kernels_common.h"

namespace {

thread_local int g_last_hip = 0;

inline int hip_fail(hipError_t e) {
    g_last_hip = (int)e;
    return BCS_EHIP;
}

// Optional per-kernel device timing (bcs_timing_begin / bcs_timing_end): while it is on, a launch is
// given a start and a stop event from a fixed pool, so its duration is the device's own.
enum KernelId {
    kSched = 0, kBatch, kExpand, kFill, kValuPeak, kAllgather, kPackPlan, kPackCopy,
    kExpandRows, kRowsToBytes, kPartnerTables, kKernelCount
};
static_assert(kKernelCount == BCS_KERNEL_COUNT, "header and kernel list disagree");
const char *const kKernelNames[kKernelCount] = {"k_sched",       "k_batch",       "k_expand",      "k_fill",
                                                "k_valu_peak",   "k_allgather_tables", "k_pack_plan", "k_pack_copy",
                                                "k_expand_rows", "k_rows_to_bytes", "k_partner_tables"};
struct Timing {
    bool on = false;
    int used = 0;
    int created = 0;
    hipEvent_t start[BCS_TIMING_MAX_LAUNCHES];
    hipEvent_t stop[BCS_TIMING_MAX_LAUNCHES];
    int kid[BCS_TIMING_MAX_LAUNCHES];
};
Timing g_timing;

template <class... KArgs, class... Args>
void launch_lds(int kid, void (*kernel)(KArgs...), dim3 grid, dim3 block, unsigned lds_bytes, hipStream_t st,
                Args... args) {
    Timing &t = g_timing;
    if (t.on && t.used < BCS_TIMING_MAX_LAUNCHES) {
        if (t.used == t.created) {
            if (hipEventCreate(&t.start[t.created]) == hipSuccess) {
                if (hipEventCreate(&t.stop[t.created]) == hipSuccess) ++t.created;
                else (void)hipEventDestroy(t.start[t.created]);
            }
        }
        if (t.used < t.created) {
            const int slot = t.used++;
            t.kid[slot] = kid;
            hipExtLaunchKernelGGL(kernel, grid, block, lds_bytes, st, t.start[slot], t.stop[slot], 0, args...);
            return;
        }
    }
    hipLaunchKernelGGL(kernel, grid, block, lds_bytes, st, args...);
}

template <class... KArgs, class... Args>
void launch(int kid, void (*kernel)(KArgs...), dim3 grid, dim3 block, hipStream_t st, Args... args) {
    launch_lds(kid, kernel, grid, block, 0u, st, args...);
}

}  // namespace

#include "bcs_kernels_sched.h"
#include "bcs_kernels_expand.h"
#include "bcs_kernels_allgather.h"

namespace {

// Measurement aid: the practical ceiling the `alu` roofline is set against.  kValuChains independent chains of
// full-rate 32-bit integer vector ops of the kinds the construction is made of (add, xor, min, subtract), written
// as instructions so that the count is exact: `iters` rounds of 4 ops per chain and lane, no memory traffic
// until one word per lane at the end.
constexpr int kValuChains = 8;
static_assert(4 * kValuChains == BCS_VALU_PEAK_OPS_PER_ITER, "header and calibration kernel disagree");

__global__ __launch_bounds__(kBlock) void k_valu_peak(uint32_t iters, uint32_t seed, uint32_t *__restrict__ sink) {
    uint32_t x[kValuChains];
#pragma unroll
    for (int c = 0; c < kValuChains; ++c) x[c] = seed + threadIdx.x * (2u * c + 1u) + blockIdx.x;
    const uint32_t k1 = seed | 1u, k2 = seed ^ 0x9e3779b9u, k3 = 0xfffffff1u;
#pragma unroll 1
    for (uint32_t it = 0; it < iters; ++it) {
#pragma unroll
        for (int c = 0; c < kValuChains; ++c) asm volatile("v_add_u32 %0, %1, %0" : "+v"(x[c]) : "s"(k1));
#pragma unroll
        for (int c = 0; c < kValuChains; ++c) asm volatile("v_xor_b32 %0, %1, %0" : "+v"(x[c]) : "s"(k2));
#pragma unroll
        for (int c = 0; c < kValuChains; ++c) asm volatile("v_min_u32 %0, %1, %0" : "+v"(x[c]) : "s"(k3));
#pragma unroll
        for (int c = 0; c < kValuChains; ++c) asm volatile("v_subrev_u32 %0, %1, %0" : "+v"(x[c]) : "s"(k1));
    }
    uint32_t acc = 0;
#pragma unroll
    for (int c = 0; c < kValuChains; ++c) acc ^= x[c];
    sink[(size_t)blockIdx.x * kBlock + threadIdx.x] = acc;
}

__global__ void k_fill(int32_t *__restrict__ out, uint64_t n, int32_t value) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) out[e] = value;
}

// ----------------------------------------------------------------------------------------------
// Host side
// ----------------------------------------------------------------------------------------------
int host_q(int32_t p) {
    int q = 0;
    while (((int64_t)1 << q) < (int64_t)p) ++q;
    return q;
}

// The skips of Alg. 1 by the closed form its halving produces: skips[k] = ceil(p / 2^(q-k)).
int host_skips(int32_t p, SkipTab &t) {
    const int q = host_q(p);
    for (int k = 0; k <= q; ++k) t.s[k] = (((uint32_t)p - 1u) >> (q - k)) + 1u;
    for (int j = q + 1; j < kMaxQ + 2; ++j) t.s[j] = (uint32_t)p;
    t.odd = odd_levels((uint32_t)p, q);
    return q;
}

// Fills g_lowtab and g_lowrows on first use per device.  The fill is enqueued on the first caller's stream; until
// it has finished, callers on other streams are made to wait for it on the device.
struct LowTabState {
    bool launched = false;
    bool done = false;
    hipStream_t stream = nullptr;
    hipEvent_t ready = nullptr;
};
constexpr int kMaxDevices = 64;
LowTabState g_lowtab_state[kMaxDevices];
std::mutex g_lowtab_mutex;

int ensure_lowtab(hipStream_t st) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev < 0 || dev >= kMaxDevices) return BCS_EINVAL;
    std::lock_guard<std::mutex> lock(g_lowtab_mutex);
    LowTabState &s = g_lowtab_state[dev];
    if (s.done) return BCS_OK;
    if (!s.launched) {
        e = hipEventCreateWithFlags(&s.ready, hipEventDisableTiming);
        if (e != hipSuccess) return hip_fail(e);
        hipLaunchKernelGGL(k_build_lowtab, dim3((kLowTableBytes + kBlock - 1) / kBlock), dim3(kBlock), 0, st);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e);
        hipLaunchKernelGGL(k_build_lowrows, dim3((kRowsAll + kBlock - 1) / kBlock), dim3(kBlock), 0, st);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e);
        e = hipEventRecord(s.ready, st);
        if (e != hipSuccess) return hip_fail(e);
        s.launched = true;
        s.stream = st;
        return BCS_OK;
    }
    if (hipEventQuery(s.ready) == hipSuccess) {
        s.done = true;
        return BCS_OK;
    }
    (void)hipGetLastError();                       // hipErrorNotReady is not an error here
    if (st != s.stream) {
        e = hipStreamWaitEvent(st, s.ready, 0);
        if (e != hipSuccess) return hip_fail(e);
    }
    return BCS_OK;
}

// The per-device scratch of the plain calls.  One allocation serves every plain call on the device, so two of
// them on different streams must not overlap: when a call comes on another stream than the one before it, that
// earlier stream's work is made a dependency of the new one (an event recorded there now covers everything
// the earlier call enqueued).  A call holds the lock from scratch_get until its last launch is enqueued: an event recorded
// in between, by another thread's call, would not cover its kernels, and a larger block or bcs_release would free memory
// that they have yet to use.
struct Scratch {
    void *ptr = nullptr;
    size_t bytes = 0;
    bool used = false;
    hipStream_t last = nullptr;
    hipEvent_t order = nullptr;
};
Scratch g_scratch[kMaxDevices];
std::mutex g_scratch_mutex;

int scratch_get(size_t bytes, hipStream_t st, void **out, std::unique_lock<std::mutex> &held) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev < 0 || dev >= kMaxDevices) return BCS_EINVAL;
    held = std::unique_lock<std::mutex>(g_scratch_mutex);
    Scratch &s = g_scratch[dev];
    if (s.bytes < bytes) {
        if (s.ptr) {
            e = hipDeviceSynchronize();            // the one place a call waits: work may still use the old block
            if (e != hipSuccess) return hip_fail(e);
            e = hipFree(s.ptr);
            s.ptr = nullptr;
            s.bytes = 0;
            s.used = false;
            if (e != hipSuccess) return hip_fail(e);
        }
        e = hipMalloc(&s.ptr, bytes);
        if (e != hipSuccess) {
            s.ptr = nullptr;
            (void)hipGetLastError();
            g_last_hip = (int)e;
            return BCS_ENOMEM;
        }
        s.bytes = bytes;
    }
    if (s.used && s.last != st) {
        if (!s.order) {
            e = hipEventCreateWithFlags(&s.order, hipEventDisableTiming);
            if (e != hipSuccess) return hip_fail(e);
        }
        e = hipEventRecord(s.order, s.last);
        if (e == hipSuccess) {
            e = hipStreamWaitEvent(st, s.order, 0);
        } else {                                   // the earlier stream is gone: wait for whatever it left behind
            (void)hipGetLastError();
            e = hipDeviceSynchronize();
        }
        if (e != hipSuccess) return hip_fail(e);
    }
    s.used = true;
    s.last = st;
    *out = s.ptr;
    return BCS_OK;
}

inline uint64_t round_up(uint64_t v, uint64_t m) { return (v + m - 1) / m * m; }

// row length of the slot-major receive table (rows start on 256-byte boundaries)
inline uint64_t slot_ld(int32_t p) { return round_up((uint64_t)p, 256); }

// where the rows of a launch go besides the int32 tables: slot-major receive bytes (all ranks), byte rows of both tables
struct RowCopies {
    slot_t *recvT;
    uint64_t ldT;
    int8_t *recvB, *sendB;
};

template <int Q>
int launch_sched(const SkipTab &tab, uint32_t root, uint32_t r0, uint32_t r1, int32_t *recv_out, int32_t *send_out,
                 const RowCopies &to, hipStream_t st) {
    const uint32_t want = (recv_out || to.recvT || to.recvB ? kWantRecv : 0u) | (send_out || to.sendB ? kWantSend : 0u);
    const uint32_t piece = sched_piece(Q, to.recvT != nullptr);
    const uint64_t pieces = (((uint64_t)r1 - r0) * Q + piece - 1) / piece;
    // a launch takes fewer than 2^32 lanes: both tables together up to 274 GB, else one after the other
    const bool both = want == (kWantRecv | kWantSend), together = both && 2u * pieces * kSchedLanes <= 0xffffffffull;
    for (uint32_t part = together ? want : 1u; part <= (together ? want : 2u); ++part)
        if (together || (want & part))
            launch(kSched, k_sched<Q>, dim3((unsigned)(together ? 2u * pieces : pieces)), dim3(kSchedLanes), st, tab, root, r0,
                   r1, part, piece, recv_out, send_out, to.recvT, to.ldT, to.recvB, to.sendB);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BCS_OK : hip_fail(e);
}

typedef int (*LaunchFn)(const SkipTab &, uint32_t, uint32_t, uint32_t, int32_t *, int32_t *, const RowCopies &, hipStream_t);

template <int... Qs>
constexpr void fill_table(LaunchFn *t, std::integer_sequence<int, Qs...>) {
    ((t[Qs] = &launch_sched<Qs + 1>), ...);
}

LaunchFn launch_for_q(int q) {
    struct Table {
        LaunchFn fn[kMaxQ];
        Table() { fill_table(fn, std::make_integer_sequence<int, kMaxQ>{}); }
    };
    static const Table table;                  // initialised once, thread-safe
    return table.fn[q - 1];
}

ExpandArgs expand_args(uint64_t rows, uint64_t R, int q, int32_t n) {
    ExpandArgs ea;
    ea.total = rows * R;
    ea.rows = rows;
    ea.R = (uint32_t)R;
    ea.q = (uint32_t)q;
    ea.x = (uint32_t)((q - (int)(R % (uint64_t)q)) % q);
    ea.nm1 = n - 1;
    ea.step_rows = (uint32_t)((kBlock * 4u) / R);
    ea.step_j = (uint32_t)((kBlock * 4u) % R);
    ea.step_k = ea.step_j % (uint32_t)q;
    ea.wrap_k = (uint32_t)q - (uint32_t)(R % (uint64_t)q);
    ea.magic_R = (uint32_t)((1ull << 32) / R + 1ull);
    ea.magic_q = q >= 2 ? (uint32_t)((1ull << 32) / (uint64_t)q + 1ull) : 0u;
    ea.magic_w = (uint32_t)((1ull << 32) / (uint64_t)(q + kExpPad) + 1ull);
    return ea;
}

// A launch takes fewer than 2^32 lanes along a grid dimension, so kernels whose lanes write four entries each take at most
// this many entries (69 GB), whole workgroups: longer tables go by ranges of rows, multiples of four so that every range's
// piece of the table starts on 16 bytes.
constexpr uint64_t kMaxLanes = 0xffffffffull;
constexpr uint64_t kLaunchEntries = kMaxLanes / kBlock * kBlock * 4;
inline uint64_t rows_per_launch(uint64_t R) { return kLaunchEntries / R & ~(uint64_t)3; }      // R < 2^31: at least 4

// Bytes of one block table up to which both tables of a call are expanded by one launch (the calls say what it gives).
constexpr uint64_t kTogetherBytes = 128ull << 20;

int check_range(int32_t p, int32_t root, int32_t r0, int32_t r1) {
    if (p < 1 || root < 0 || root >= p || r0 < 0 || r0 > r1 || r1 > p) return BCS_EINVAL;
    return BCS_OK;
}

}  // namespace

extern "C" {

int bcs_q(int32_t p) { return p < 1 ? BCS_EINVAL : host_q(p); }

int bcs_skips(int32_t p, int32_t *skips_host) {
    if (p < 1 || !skips_host) return BCS_EINVAL;
    SkipTab t;
    const int q = host_skips(p, t);
    for (int k = 0; k <= q; ++k) skips_host[k] = (int32_t)t.s[k];
    return q;
}

int64_t bcs_rounds(int32_t p, int32_t n) {
    if (p < 1 || n < 1) return BCS_EINVAL;
    return (int64_t)n - 1 + host_q(p);
}

// The sizes that bcs_sched_workspace_bytes states: for all ranks with send rows a slot-major receive table (which the allgather
// tables keep in their workspace) and a word a rank, for a large part of the ranks the words alone.  The schedules
// themselves use none of it; callers' buffers and refusals go by these sizes.
inline uint64_t slot_table_bytes(int32_t p, int q) { return slot_ld(p) * (uint64_t)q * sizeof(slot_t); }
inline uint64_t digit_table_bytes(int32_t p) { return round_up((uint64_t)p * sizeof(uint32_t), 256); }

inline bool partial_range_tabled(int32_t p, int q, int32_t r0, int32_t r1) {
    return (uint64_t)(r1 - r0) * (uint64_t)(q * q) >= 8ull * (uint64_t)p;
}

int64_t bcs_sched_workspace_bytes(int32_t p, int32_t r0, int32_t r1, int want_send) {
    if (check_range(p, 0, r0, r1) != BCS_OK) return BCS_EINVAL;
    const int q = host_q(p);
    if (!want_send || q == 0) return 0;
    if (!(r0 == 0 && r1 == p)) return partial_range_tabled(p, q, r0, r1) ? (int64_t)digit_table_bytes(p) : 0;
    return (int64_t)(slot_table_bytes(p, q) + digit_table_bytes(p));
}

namespace {
// the rows themselves need no scratch; arguments are checked
int sched_rows(int32_t p, int32_t root, int32_t r0, int32_t r1, int32_t *recv_out, int32_t *send_out, hipStream_t st) {
    const int q = host_q(p);
    if (q == 0 || r0 == r1) return BCS_OK;
    SkipTab tab;
    host_skips(p, tab);
    const int rc = ensure_lowtab(st);
    if (rc != BCS_OK) return rc;
    return launch_for_q(q)(tab, (uint32_t)root, (uint32_t)r0, (uint32_t)r1, recv_out, send_out, RowCopies{}, st);
}
}  // namespace

int bcs_sched_rooted_ws(int32_t p, int32_t root, int32_t r0, int32_t r1, int32_t *recv_out, int32_t *send_out,
                        void *workspace, size_t workspace_bytes, void *stream) {
    const int rc = check_range(p, root, r0, r1);
    if (rc != BCS_OK) return rc;
    if (!recv_out && !send_out) return BCS_EINVAL;
    if (host_q(p) == 0 || r0 == r1) return BCS_OK;
    // the contract of the call: a workspace of the stated size, though this construction leaves it alone
    const int64_t need = bcs_sched_workspace_bytes(p, r0, r1, send_out != nullptr);
    if (need > 0 && (!workspace || workspace_bytes < (size_t)need)) return BCS_ENOMEM;
    if (need > 0 && (((uintptr_t)workspace) & 255u)) return BCS_EINVAL;
    return sched_rows(p, root, r0, r1, recv_out, send_out, (hipStream_t)stream);
}

int bcs_sched_rooted(int32_t p, int32_t root, int32_t r0, int32_t r1, int32_t *recv_out, int32_t *send_out,
                     void *stream) {
    const int rc = check_range(p, root, r0, r1);
    if (rc != BCS_OK) return rc;
    if (!recv_out && !send_out) return BCS_EINVAL;
    return sched_rows(p, root, r0, r1, recv_out, send_out, (hipStream_t)stream);
}

int bcs_sched_rooted_static(int32_t p, int32_t root, int32_t r0, int32_t r1, int32_t *recv_out, int32_t *send_out,
                            void *stream) {
    const int rc = check_range(p, root, r0, r1);
    if (rc != BCS_OK) return rc;
    if (!recv_out && !send_out) return BCS_EINVAL;
    // the stated limit of the call
    const int64_t need = bcs_sched_workspace_bytes(p, r0, r1, send_out != nullptr);
    if (need < 0) return (int)need;
    if ((uint64_t)need > (uint64_t)BCS_STATIC_SCRATCH_BYTES) return BCS_ETOOBIG;
    return sched_rows(p, root, r0, r1, recv_out, send_out, (hipStream_t)stream);
}

int bcs_sched(int32_t p, int32_t r0, int32_t r1, int32_t *recv_out, int32_t *send_out, void *stream) {
    return bcs_sched_rooted(p, 0, r0, r1, recv_out, send_out, stream);
}

int bcs_sched_batch(int64_t count, const int32_t *p, const int32_t *r, const int32_t *root, int32_t *recv_out,
                    int32_t *send_out, int32_t *q_out, void *stream) {
    if (count < 0 || !p || !r || !root) return BCS_EINVAL;
    if (!recv_out && !send_out && !q_out) return BCS_EINVAL;
    if (count == 0) return BCS_OK;
    const uint64_t blocks = ((uint64_t)count + kBatchBlock - 1) / kBatchBlock;
    if (blocks > 0x7fffffffull) return BCS_EINVAL;
    const int rc = ensure_lowtab((hipStream_t)stream);
    if (rc != BCS_OK) return rc;
    const int64_t step = (int64_t)(kMaxLanes / kBatchBlock * kBatchBlock);      // triples a launch: a lane each
    for (int64_t i = 0; i < count; i += step) {
        const int64_t part = count - i < step ? count - i : step, row = i * BCS_BATCH_STRIDE;
        launch(kBatch, k_batch, dim3((unsigned)((part + kBatchBlock - 1) / kBatchBlock)), dim3(kBatchBlock),
               (hipStream_t)stream, part, p + i, r + i, root + i, recv_out ? recv_out + row : nullptr,
               send_out ? send_out + row : nullptr, q_out ? q_out + i : nullptr);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BCS_OK : hip_fail(e);
}

int bcs_expand(int32_t p, int32_t n, int32_t r0, int32_t r1, const int32_t *recv, const int32_t *send,
               int32_t *recv_blocks, int32_t *send_blocks, void *stream) {
    if (check_range(p, 0, r0, r1) != BCS_OK || n < 1 || n > BCS_MAX_N) return BCS_EINVAL;
    const int q = host_q(p);
    if (q == 0) {                      // rows of the input tables are empty: only the outputs count
        recv = recv_blocks;
        send = send_blocks;
    }
    if ((recv == nullptr) != (recv_blocks == nullptr)) return BCS_EINVAL;
    if ((send == nullptr) != (send_blocks == nullptr)) return BCS_EINVAL;
    if (!recv && !send) return BCS_EINVAL;
    const uint64_t rows = (uint64_t)r1 - r0;
    const uint64_t R = (uint64_t)n - 1 + q;
    if (rows == 0 || R == 0) return BCS_OK;
    hipStream_t st = (hipStream_t)stream;
    if (q == 0) {
        for (int32_t *out : {recv_blocks, send_blocks})
            if (out) launch(kFill, k_fill, dim3(1024), dim3(kBlock), st, out, rows * R, (int32_t)BCS_NO_BLOCK);
        hipError_t e0 = hipGetLastError();
        return e0 == hipSuccess ? BCS_OK : hip_fail(e0);
    }
    // sixteen entries a lane: from 275 GB a table on, by ranges of rows
    const uint64_t most = kMaxLanes / kBlock * kExpChunk / R & ~(uint64_t)3;
    for (uint64_t a = 0; rows > most && a < rows; a += most) {
        const uint64_t b = rows - a < most ? rows : a + most;
        const int rc = bcs_expand(p, n, r0 + (int32_t)a, r0 + (int32_t)b, recv ? recv + a * q : nullptr,
                                  send ? send + a * q : nullptr, recv_blocks ? recv_blocks + a * R : nullptr,
                                  send_blocks ? send_blocks + a * R : nullptr, stream);
        if (rc != BCS_OK || b == rows) return rc;
    }
    // Both tables in one launch: a call of a few thousand ranks is bound by its launches (2 x 7.7 MB: 13.1 us with one for
    // each table, 9.3 us now; 2 x 81 MB 34.7 and 30.2 us).  From some hundred MB on it gives nothing (2 x 509 MB: 165 and
    // 170 us).
    ExpandArgs ea = expand_args(rows, R, q, n);
    const ExpandTables both = {{recv, send}, {recv_blocks, send_blocks}};
    auto aligned = [&](int t) { return (((uintptr_t)both.out[t]) & 15u) == 0 ? 1 : 0; };
    const uint64_t blocks = (ea.total + kExpChunk - 1) / kExpChunk;
    const bool together = recv && send && aligned(0) == aligned(1) && ea.total * sizeof(int32_t) <= kTogetherBytes;
    for (int t = 0; t < (together ? 1 : 2); ++t) {
        if (!both.in[t]) continue;
        const ExpandTables tables = together ? both : ExpandTables{{both.in[t], nullptr}, {both.out[t], nullptr}};
        const dim3 grid((unsigned)blocks, together ? 2u : 1u);
        ea.aligned = aligned(t);
        if (R >= kExpMinR && (uint32_t)q >= kExpMinQ) {
            // rows a chunk can touch, plus one that a lane past the end may address but never uses
            const uint64_t max_rows = (R - 1 + kExpChunk - 1) / R + 2;
            const unsigned lds_bytes = (unsigned)(max_rows * (uint64_t)(q + kExpPad) * sizeof(int32_t));
            if (R <= kExpNtMaxR) launch_lds(kExpand, k_expand<true>, grid, dim3(kBlock), lds_bytes, st, ea, tables);
            else launch_lds(kExpand, k_expand<false>, grid, dim3(kBlock), lds_bytes, st, ea, tables);
        } else {
            launch(kExpand, k_expand_small, grid, dim3(kBlock), st, ea, tables);
        }
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BCS_OK : hip_fail(e);
}

namespace {
// bytes of one rank-major byte table (p rows and one spare that the last row's lanes may read)
inline uint64_t byte_rows_bytes(int32_t p, int q) { return round_up(((uint64_t)p + 1) * byte_row_stride(q), 256); }
inline bool byte_rows_apply(int32_t p, int q, uint64_t R) {
    return q >= (int)kExpMinQ && R >= kExpMinR && byte_rows_bytes(p, q) <= kByteRowsMax;
}
}  // namespace

namespace {
// rows of the caller's tables from which an expansion through byte rows pays: the conversion is one more
// pass over the table and one more launch
constexpr uint64_t kExpandWsMinR = 256;
inline bool expand_ws_applies(int32_t rows, int q, uint64_t R) {
    return q >= (int)kExpMinQ && R >= kExpandWsMinR && rows > 0;
}
// ... and tables up to kTogetherBytes are better off without.  Both tables, with byte rows (four launches) against without
// (one): block tables of 7.7 MB 17.9 and 9.3 us, 81 MB 31.9 and 30.2, 161 MB 52.9 and 53.0, 266 MB 83 and 88, 1078 MB 300 and
// 319 us.  One table (two launches against one): 7.7 MB 6.7 and 4.2 us, 25 MB 8.3 and 6.1, 81 MB 16.1 and 14.8, 122 MB 21.7
// and 21.1, 137 MB 26.2 and 23.1
inline bool expand_ws_pays(int32_t rows, uint64_t R) { return (uint64_t)rows * R * sizeof(int32_t) > kTogetherBytes; }
// rows converted and expanded at a time: their byte table fits kByteRowsMax; a multiple of 4, so that every
// chunk's piece of the output starts on a 16-byte boundary
inline uint32_t expand_ws_chunk_rows(uint32_t rows, int q) {
    const uint32_t fit = (uint32_t)(kByteRowsMax / (uint64_t)byte_row_stride(q) - 1) & ~3u;
    return rows < fit ? rows : fit;
}

ExpandRowsArgs expand_rows_args(uint64_t rows, uint64_t R, int q, int32_t n) {
    ExpandRowsArgs ra;
    ra.total = rows * R;
    ra.magic_R64 = ~0ull / R + 1ull;
    ra.magic_R32 = (uint32_t)((1ull << 32) / R + 1ull);
    ra.magic_q = (uint32_t)((1ull << 32) / (uint64_t)q + 1ull);
    ra.R = (uint32_t)R;
    ra.q = (uint32_t)q;
    ra.x = (uint32_t)((q - (int)(R % (uint64_t)q)) % q);
    ra.RS = (uint32_t)byte_row_stride(q);
    ra.nm1 = n - 1;
    return ra;
}
}  // namespace

int64_t bcs_expand_workspace_bytes(int32_t p, int32_t n, int32_t r0, int32_t r1) {
    if (check_range(p, 0, r0, r1) != BCS_OK || n < 1 || n > BCS_MAX_N) return BCS_EINVAL;
    const int q = host_q(p);
    if (!expand_ws_applies(r1 - r0, q, (uint64_t)n - 1 + q)) return 0;
    return (int64_t)byte_rows_bytes((int32_t)expand_ws_chunk_rows((uint32_t)(r1 - r0), q), q);
}

int bcs_expand_ws(int32_t p, int32_t n, int32_t r0, int32_t r1, const int32_t *recv, const int32_t *send,
                  int32_t *recv_blocks, int32_t *send_blocks, void *workspace, size_t workspace_bytes, void *stream) {
    if (check_range(p, 0, r0, r1) != BCS_OK || n < 1 || n > BCS_MAX_N) return BCS_EINVAL;
    const int q = host_q(p);
    const uint64_t R = (uint64_t)n - 1 + q;
    const int64_t need = bcs_expand_workspace_bytes(p, n, r0, r1);
    const bool aligned = ((recv_blocks ? (uintptr_t)recv_blocks : 0) | (send_blocks ? (uintptr_t)send_blocks : 0)) % 16 == 0;
    const bool tables_ok = (recv == nullptr) == (recv_blocks == nullptr) && (send == nullptr) == (send_blocks == nullptr) &&
                           (recv || send);
    if (need <= 0 || !aligned || !tables_ok || !expand_ws_pays(r1 - r0, R) || !workspace || workspace_bytes < (size_t)need ||
        (((uintptr_t)workspace) & 15u))
        return bcs_expand(p, n, r0, r1, recv, send, recv_blocks, send_blocks, stream);
    hipStream_t st = (hipStream_t)stream;
    const uint32_t rows = (uint32_t)(r1 - r0);
    const uint64_t by_bytes = expand_ws_chunk_rows(rows, q), by_lanes = rows_per_launch(R);
    const uint32_t chunk = (uint32_t)(by_bytes < by_lanes ? by_bytes : by_lanes);
    const uint32_t RS = (uint32_t)byte_row_stride(q), w4 = RS / 4;
    const int32_t *ins[2] = {recv, send};
    int32_t *outs[2] = {recv_blocks, send_blocks};
    // the one workspace serves every chunk of both tables in turn (same stream: a conversion follows the
    // expansion that read the previous contents)
    for (int t = 0; t < 2; ++t) {
        if (!ins[t]) continue;
        for (uint32_t c0 = 0; c0 < rows; c0 += chunk) {
            const uint32_t rc = rows - c0 < chunk ? rows - c0 : chunk;
            const ExpandRowsArgs ra = expand_rows_args(rc, R, q, n);
            const uint64_t pieces = (ra.total + kBlock * 4 - 1) / (kBlock * 4);
            launch(kRowsToBytes, k_rows_to_bytes, dim3((rc * w4 + kBlock - 1) / kBlock), dim3(kBlock), st, rc, (uint32_t)q,
                   RS, (uint32_t)((1ull << 32) / w4 + 1ull), ins[t] + (uint64_t)c0 * q, (int8_t *)workspace);
            launch(kExpandRows, k_expand_rows, dim3((unsigned)pieces), dim3(kBlock), st, ra, (const int8_t *)workspace,
                   (const int8_t *)nullptr, outs[t] + (uint64_t)c0 * R, (int32_t *)nullptr);
        }
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BCS_OK : hip_fail(e);
}

int64_t bcs_sched_expand_workspace_bytes(int32_t p, int32_t n) {
    if (p < 1 || n < 1 || n > BCS_MAX_N) return BCS_EINVAL;
    const int q = host_q(p);
    const int64_t base = bcs_sched_workspace_bytes(p, 0, p, 1);
    if (byte_rows_apply(p, q, (uint64_t)n - 1 + q)) return base + (int64_t)(2 * byte_rows_bytes(p, q));
    // too many ranks for byte tables that stay in cache: the tables are expanded chunk by chunk (bcs_expand_ws)
    const int64_t extra = bcs_expand_workspace_bytes(p, n, 0, p);
    return base + (extra > 0 ? extra : 0);
}

namespace {
// Schedules of all ranks with byte rows in the workspace, and the expansion of the byte rows.
// Short calls are bound by launches: both tables at once, two launches.  Long ones go table by table, so that a table's
// byte rows are still cached when they are expanded.  Measured, together against table by table: block tables of 0.2 MB 13
// against 18 us, 65 MB 35 against 43 us, 218 MB 119 us both, 1158 MB 388 against 371 us.  Byte rows that exceed the
// workspace or kByteRowsMax are made and expanded a chunk of ranks at a time; any workspace that holds the schedules'
// scratch will do.  (Rows of up to 128 entries used to be expanded by the workgroup that built them, 256 ranks each: 43 us
// at 65 MB, 143 at 218 MB.)

int sched_expand_rows(int32_t p, uint32_t root, int32_t n, int q, uint64_t R, int32_t *recv_out, int32_t *send_out,
                      int32_t *recv_blocks, int32_t *send_blocks, int8_t *ws, size_t ws_bytes, hipStream_t st) {
    const uint64_t RS = (uint64_t)byte_row_stride(q), rows_bytes = byte_rows_bytes(p, q);
    const bool together = 2 * rows_bytes <= ws_bytes && (uint64_t)p * R * 4u <= kTogetherBytes;
    const uint64_t cap = ws_bytes < kByteRowsMax ? ws_bytes : kByteRowsMax;
    const uint64_t by_bytes = (cap / RS - 1u) & ~(uint64_t)3, by_lanes = rows_per_launch(R);      // multiples of 4
    const uint64_t fit = by_bytes < by_lanes ? by_bytes : by_lanes;
    const uint32_t chunk = together || (uint64_t)p <= fit ? (uint32_t)p : (uint32_t)fit;
    if (chunk == 0) return BCS_ENOMEM;
    SkipTab tab;
    host_skips(p, tab);
    int rc = ensure_lowtab(st);
    if (rc != BCS_OK) return rc;
    const LaunchFn rows = launch_for_q(q);
    if (together) {
        int8_t *const sendB = ws + rows_bytes;
        rc = rows(tab, root, 0u, (uint32_t)p, recv_out, send_out, RowCopies{nullptr, 0, ws, sendB}, st);
        if (rc != BCS_OK) return rc;
        const ExpandRowsArgs ra = expand_rows_args((uint64_t)p, R, q, n);
        const unsigned pieces = (unsigned)((ra.total + kBlock * 4 - 1) / (kBlock * 4));
        launch(kExpandRows, k_expand_rows, dim3(2 * pieces), dim3(kBlock), st, ra, (const int8_t *)ws, (const int8_t *)sendB,
               recv_blocks, send_blocks);
    } else {
        for (int t = 0; t < 2; ++t) {
            int32_t *const out = t ? send_out : recv_out, *const blocks = t ? send_blocks : recv_blocks;
            for (uint32_t c0 = 0; c0 < (uint32_t)p; c0 += chunk) {
                const uint32_t c1 = (uint32_t)p - c0 < chunk ? (uint32_t)p : c0 + chunk;
                int32_t *const to = out + (uint64_t)c0 * q;
                rc = rows(tab, root, c0, c1, t ? nullptr : to, t ? to : nullptr,
                          RowCopies{nullptr, 0, t ? nullptr : ws, t ? ws : nullptr}, st);
                if (rc != BCS_OK) return rc;
                const ExpandRowsArgs ra = expand_rows_args((uint64_t)(c1 - c0), R, q, n);
                launch(kExpandRows, k_expand_rows, dim3((unsigned)((ra.total + kBlock * 4 - 1) / (kBlock * 4))), dim3(kBlock),
                       st, ra, (const int8_t *)ws, (const int8_t *)nullptr, blocks + (uint64_t)c0 * R, (int32_t *)nullptr);
            }
        }
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BCS_OK : hip_fail(e);
}
}  // namespace

int bcs_sched_expand_ws(int32_t p, int32_t root, int32_t n, int32_t *recv_out, int32_t *send_out,
                        int32_t *recv_blocks, int32_t *send_blocks, void *workspace, size_t workspace_bytes,
                        void *stream) {
    if (p < 1 || root < 0 || root >= p || n < 1 || n > BCS_MAX_N) return BCS_EINVAL;
    const int q = host_q(p);
    const uint64_t R = (uint64_t)n - 1 + q;
    if (R == 0) return BCS_OK;                     // one process, one block: every table is empty
    if (!recv_blocks || !send_blocks) return BCS_EINVAL;
    if (q > 0 && (!recv_out || !send_out)) return BCS_EINVAL;
    if (workspace && workspace_bytes > 0 && (((uintptr_t)workspace) & 255u)) return BCS_EINVAL;
    const int64_t base = q > 0 ? bcs_sched_workspace_bytes(p, 0, p, 1) : 0;
    if (base > 0 && (!workspace || workspace_bytes < (size_t)base)) return BCS_ENOMEM;
    const bool aligned = ((((uintptr_t)recv_blocks) | ((uintptr_t)send_blocks)) & 15u) == 0;
    // Tables of up to kTogetherBytes whose byte rows exceed the workspace (the schedules' size alone) would take eight launches
    // or more in chunks; the schedules and bcs_expand take two.  p = 1000, n = 16 21.6 and 7.8 us; p = 20000, n = 200 31.7 and
    // 11.1; p = 200003, n = 64 57.5 and 40.5 (34.2 with byte rows of both tables at once)
    const bool chunks_pay = q > 0 && ((uint64_t)p * R * sizeof(int32_t) > kTogetherBytes ||
                                      2 * byte_rows_bytes(p, q) <= workspace_bytes);
    if (q >= (int)kExpMinQ && R >= kExpMinR && aligned && chunks_pay)
        return sched_expand_rows(p, (uint32_t)root, n, q, R, recv_out, send_out, recv_blocks, send_blocks,
                                 (int8_t *)workspace, workspace_bytes, (hipStream_t)stream);
    if (q > 0) {
        const int rc = sched_rows(p, root, 0, p, recv_out, send_out, (hipStream_t)stream);
        if (rc != BCS_OK) return rc;
    }
    return bcs_expand(p, n, 0, p, recv_out, send_out, recv_blocks, send_blocks, stream);
}

int bcs_sched_expand(int32_t p, int32_t root, int32_t n, int32_t *recv_out, int32_t *send_out, int32_t *recv_blocks,
                     int32_t *send_blocks, void *stream) {
    if (p < 1 || root < 0 || root >= p || n < 1 || n > BCS_MAX_N) return BCS_EINVAL;
    if ((uint64_t)n - 1 + host_q(p) > 0) {         // nothing is required of an empty result
        if (!recv_blocks || !send_blocks) return BCS_EINVAL;
        if (p > 1 && (!recv_out || !send_out)) return BCS_EINVAL;
    }
    const int64_t need = bcs_sched_expand_workspace_bytes(p, n);
    void *ws = nullptr;
    std::unique_lock<std::mutex> held;             // until the call below has enqueued everything
    if (need > 0) {
        const int rc = scratch_get((size_t)need, (hipStream_t)stream, &ws, held);
        if (rc != BCS_OK) return rc;
    }
    return bcs_sched_expand_ws(p, root, n, recv_out, send_out, recv_blocks, send_blocks, ws, (size_t)need, stream);
}

int bcs_release(void) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev < 0 || dev >= kMaxDevices) return BCS_EINVAL;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    Scratch &s = g_scratch[dev];
    if (s.ptr) {
        e = hipDeviceSynchronize();
        if (e != hipSuccess) return hip_fail(e);
        e = hipFree(s.ptr);
        s.ptr = nullptr;
        s.bytes = 0;
        s.used = false;
        if (e != hipSuccess) return hip_fail(e);
    }
    return BCS_OK;
}

int64_t bcs_allgather_workspace_bytes(int32_t p) {
    if (p < 1) return BCS_EINVAL;
    return bcs_sched_workspace_bytes(p, 0, p, 1);
}

int bcs_allgather_tables_ws(int32_t p, int32_t n, int32_t r, int32_t *pack_idx, int32_t *unpack_idx, void *workspace,
                            size_t workspace_bytes, void *stream) {
    if (p < 1 || n < 1 || n > BCS_MAX_N || r < 0 || r >= p) return BCS_EINVAL;
    if (!pack_idx && !unpack_idx) return BCS_EINVAL;
    const int q = host_q(p);
    const uint64_t R = (uint64_t)n - 1 + q;
    if (R == 0) return BCS_OK;
    hipStream_t st = (hipStream_t)stream;
    if (q == 0) {                                  // one process: nothing ever moves
        if (pack_idx) launch(kFill, k_fill, dim3(64), dim3(kBlock), st, pack_idx, R, (int32_t)BCS_NO_BLOCK);
        if (unpack_idx) launch(kFill, k_fill, dim3(64), dim3(kBlock), st, unpack_idx, R, (int32_t)BCS_NO_BLOCK);
        hipError_t e0 = hipGetLastError();
        return e0 == hipSuccess ? BCS_OK : hip_fail(e0);
    }
    const int64_t need = bcs_allgather_workspace_bytes(p);
    if (!workspace || workspace_bytes < (size_t)need) return BCS_ENOMEM;
    if (((uintptr_t)workspace) & 255u) return BCS_EINVAL;
    SkipTab tab;
    host_skips(p, tab);
    int rc = ensure_lowtab(st);
    if (rc != BCS_OK) return rc;
    const uint64_t ld = slot_ld(p);
    slot_t *recvT = (slot_t *)workspace;
    rc = launch_for_q(q)(tab, 0u, 0u, (uint32_t)p, nullptr, nullptr, RowCopies{recvT, ld, nullptr, nullptr}, st);
    if (rc != BCS_OK) return rc;
    const unsigned bx = (unsigned)(((uint64_t)p + kAgChunk - 1) / kAgChunk);
    const uint32_t x = (uint32_t)((q - (int)(R % (uint64_t)q)) % q);
    const bool vec = ((((uintptr_t)pack_idx) | ((uintptr_t)unpack_idx)) & 15u) == 0;
    if (vec && R * (uint64_t)p <= kLaunchEntries) {
        AgFlatArgs fa;
        fa.total = R * (uint64_t)p;
        fa.magic_p = ~0ull / (uint64_t)p + 1ull;
        fa.p = (uint32_t)p;
        fa.q = (uint32_t)q;
        fa.r = (uint32_t)r;
        fa.x = x;
        fa.nm1 = n - 1;
        fa.magic_q = (uint32_t)((1ull << 32) / (uint64_t)q + 1ull);
        const uint64_t pieces = (fa.total + kBlock * 4 - 1) / (kBlock * 4);
        launch(kAllgather, k_allgather_tables_flat, dim3((unsigned)pieces, (pack_idx && unpack_idx) ? 2u : 1u),
               dim3(kBlock), st, tab, fa, (const slot_t *)recvT, ld, pack_idx, unpack_idx);
    } else {
        launch(kAllgather, k_allgather_tables, dim3(bx, (unsigned)q), dim3(kBlock), st, tab, q, (uint32_t)r, x,
               (int32_t)(n - 1), R, (const slot_t *)recvT, ld, pack_idx, unpack_idx);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BCS_OK : hip_fail(e);
}

int bcs_allgather_tables(int32_t p, int32_t n, int32_t r, int32_t *pack_idx, int32_t *unpack_idx, void *stream) {
    if (p < 1 || n < 1 || n > BCS_MAX_N || r < 0 || r >= p) return BCS_EINVAL;
    if (!pack_idx && !unpack_idx) return BCS_EINVAL;
    const int64_t need = bcs_allgather_workspace_bytes(p);
    void *ws = nullptr;
    std::unique_lock<std::mutex> held;             // until the call below has enqueued everything
    if (need > 0) {
        const int rc = scratch_get((size_t)need, (hipStream_t)stream, &ws, held);
        if (rc != BCS_OK) return rc;
    }
    return bcs_allgather_tables_ws(p, n, r, pack_idx, unpack_idx, ws, (size_t)need, stream);
}

int bcs_allgather_plan(int32_t p, int32_t r, int32_t *to, int32_t *from, int32_t *count, int32_t *recv_first) {
    if (p < 1 || r < 0 || r >= p || !to || !from || !count || !recv_first) return BCS_EINVAL;
    SkipTab t;
    const int q = host_skips(p, t);
    for (int k = 0; k < q; ++k) {
        const uint32_t s = t.s[k];
        to[k] = (int32_t)((uint32_t)r >= s ? (uint32_t)r - s : (uint32_t)r + (uint32_t)p - s);
        const uint32_t f = (uint32_t)r + s;
        from[k] = (int32_t)(f >= (uint32_t)p ? f - (uint32_t)p : f);
        count[k] = (int32_t)(t.s[k + 1] - s);
        recv_first[k] = (int32_t)s;
    }
    return q;
}

int bcs_census_plan(int32_t p, int32_t r, int32_t *to, int32_t *from, int32_t *own) {
    if (p < 1 || r < 0 || r >= p || !to || !from || !own) return BCS_EINVAL;
    SkipTab t;
    const int q = host_skips(p, t);
    for (int k = 0; k < q; ++k) {
        const bool odd = ((t.odd >> k) & 1u) != 0;             // 2 skips[k] - skips[k+1] = 1
        const uint32_t s = t.s[k] - (odd ? 1u : 0u);            // partner distance
        to[k] = (int32_t)((uint32_t)r >= s ? (uint32_t)r - s : (uint32_t)r + (uint32_t)p - s);
        const uint32_t f = (uint32_t)r + s;
        from[k] = (int32_t)(f >= (uint32_t)p ? f - (uint32_t)p : f);
        own[k] = odd ? 0 : 1;
    }
    return q;
}

}  // extern "C"

namespace {
int partner_tables(int32_t p, int32_t r0, int32_t r1, uint32_t census, int32_t *to, int32_t *from, void *stream) {
    if (p < 1 || r0 < 0 || r0 > r1 || r1 > p) return BCS_EINVAL;
    const int q = host_q(p);
    const uint64_t total = (uint64_t)(r1 - r0) * (uint64_t)q;
    if (total == 0) return BCS_OK;                                          // p = 1 or an empty range
    if (!to && !from) return BCS_EINVAL;
    const bool vec = ((((uintptr_t)to) | ((uintptr_t)from)) & 15u) == 0;
    const uint64_t step = kLaunchEntries / (uint64_t)q & ~(uint64_t)3;      // rows a launch; 31 * 2^31 entries take four
    for (uint64_t row = 0; row < (uint64_t)(r1 - r0); row += step) {
        const uint64_t rest = total - row * q, count = rest < step * q ? rest : step * q;
        const dim3 grid((unsigned)((count + kBlock * 4 - 1) / (kBlock * 4)));
        int32_t *const t = to ? to + row * q : nullptr, *const f = from ? from + row * q : nullptr;
        if (vec)
            launch(kPartnerTables, k_partner_tables<true>, grid, dim3(kBlock), (hipStream_t)stream, (uint32_t)p,
                   (uint32_t)q, census, (uint32_t)r0 + (uint32_t)row, count, t, f);
        else
            launch(kPartnerTables, k_partner_tables<false>, grid, dim3(kBlock), (hipStream_t)stream, (uint32_t)p,
                   (uint32_t)q, census, (uint32_t)r0 + (uint32_t)row, count, t, f);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BCS_OK : hip_fail(e);
}
}  // namespace

extern "C" {

int bcs_allgather_partners(int32_t p, int32_t r0, int32_t r1, int32_t *to, int32_t *from, void *stream) {
    return partner_tables(p, r0, r1, 0u, to, from, stream);
}

int bcs_census_partners(int32_t p, int32_t r0, int32_t r1, int32_t *to, int32_t *from, void *stream) {
    return partner_tables(p, r0, r1, 1u, to, from, stream);
}

int64_t bcs_pack_workspace_bytes(int32_t p) {
    if (p < 1) return BCS_EINVAL;
    const uint64_t groups = ((uint64_t)p + kPlanRoots - 1) / kPlanRoots;
    return (int64_t)(((uint64_t)p + groups + 1) * sizeof(int64_t));
}

namespace {
int pack_args(int32_t p, int32_t n, const int32_t *idx, const int64_t *displs, const int64_t *offsets, const void *workspace,
              size_t workspace_bytes) {
    if (p < 1 || n < 1 || !idx || !displs || !offsets) return BCS_EINVAL;
    const int64_t need = bcs_pack_workspace_bytes(p);
    if (!workspace || workspace_bytes < (size_t)need || (((uintptr_t)workspace) & 7u)) return BCS_ENOMEM;
    return BCS_OK;
}

int pack_plan(int32_t p, int32_t n, const int32_t *idx, const int64_t *displs, int64_t *offsets, void *workspace,
              hipStream_t st, PackPlan &plan) {
    const uint32_t groups = (uint32_t)(((uint64_t)p + kPlanRoots - 1) / kPlanRoots);
    plan.offsets = offsets;
    plan.src = (int64_t *)workspace;
    plan.totals = plan.src + p;
    if ((uint32_t)p <= kPlanOneMaxP) {
        launch(kPackPlan, k_pack_plan_one, dim3(1), dim3(kBlock), st, (uint32_t)p, (uint32_t)n, idx, displs, plan);
    } else {
        launch(kPackPlan, k_pack_plan_local, dim3(groups), dim3(kBlock), st, (uint32_t)p, (uint32_t)n, idx, displs,
               plan);
        launch(kPackPlan, k_pack_plan_totals, dim3(1), dim3(kBlock), st, (uint32_t)p, groups, plan);
        launch(kPackPlan, k_pack_plan_finish, dim3(((unsigned)p + kBlock - 1) / kBlock), dim3(kBlock), st, (uint32_t)p,
               plan);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BCS_OK : hip_fail(e);
}
}  // namespace

}  // extern "C"

namespace {
// the payload kernel of one round: PACK moves blocks into the message, !PACK the message into the blocks
template <bool PACK>
int launch_copy(int32_t p, int64_t limit, const int64_t *offsets, const int64_t *src, int32_t *data, int32_t *message,
                hipStream_t st) {
    const int aligned = (int)((((uintptr_t)message) & 15u) == 0);
    if (limit < kCopyShort) {
        const uint64_t blocks = ((uint64_t)limit + kBlock * 4 - 1) / (kBlock * 4);
        launch(kPackCopy, k_pack_copy<PACK, 1>, dim3((unsigned)blocks), dim3(kBlock), st, (uint32_t)p, limit, offsets, src,
               data, message, aligned);
    } else {
        const uint64_t chunk = (uint64_t)kCopyIter * kBlock * 4;
        const uint64_t blocks = ((uint64_t)limit + chunk - 1) / chunk;
        launch(kPackCopy, k_pack_copy<PACK, kCopyIter>, dim3((unsigned)blocks), dim3(kBlock), st, (uint32_t)p, limit,
               offsets, src, data, message, aligned);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BCS_OK : hip_fail(e);
}
// plan and payload of one round: one launch where the round is short, else the plan's launches and the payload's
template <bool PACK>
int launch_round(int32_t p, int32_t n, const int32_t *idx, const int64_t *displs, int64_t limit, int64_t *offsets,
                 void *workspace, int32_t *data, int32_t *message, hipStream_t st) {
    if ((uint32_t)p <= kRoundMaxP && limit > 0 && limit <= kRoundMaxElements) {
        const int aligned = (int)((((uintptr_t)message) & 15u) == 0);
        launch(kPackCopy, k_pack_round<PACK>, dim3((unsigned)((limit + kBlock * 4 - 1) / (kBlock * 4))), dim3(kBlock), st,
               (uint32_t)p, (uint32_t)n, limit, idx, displs, offsets, data, message, aligned);
        hipError_t e = hipGetLastError();
        return e == hipSuccess ? BCS_OK : hip_fail(e);
    }
    PackPlan plan;
    const int rc = pack_plan(p, n, idx, displs, offsets, workspace, st, plan);
    if (rc != BCS_OK || limit == 0) return rc;
    return launch_copy<PACK>(p, limit, offsets, plan.src, data, message, st);
}
// a launch of the payload kernel covers 2^36 elements (275 GB), which with their buffers no card holds
inline bool copy_size_ok(int64_t limit) { return (uint64_t)limit <= kMaxLanes / kBlock * ((uint64_t)kCopyIter * kBlock * 4); }
}  // namespace

extern "C" {

int bcs_pack_round(int32_t p, int32_t n, const int32_t *idx, const int64_t *displs, const int32_t *data,
                   int32_t *packed, int64_t capacity, int64_t *offsets, void *workspace, size_t workspace_bytes,
                   void *stream) {
    if (!data || capacity < 0 || (!packed && capacity > 0)) return BCS_EINVAL;
    if (!copy_size_ok(capacity)) return BCS_EINVAL;
    const int rc = pack_args(p, n, idx, displs, offsets, workspace, workspace_bytes);
    if (rc != BCS_OK) return rc;
    return launch_round<true>(p, n, idx, displs, capacity, offsets, workspace, const_cast<int32_t *>(data), packed,
                              (hipStream_t)stream);
}

int bcs_unpack_round(int32_t p, int32_t n, const int32_t *idx, const int64_t *displs, int32_t *data,
                     const int32_t *packed, int64_t length, int64_t *offsets, void *workspace, size_t workspace_bytes,
                     void *stream) {
    if (!data || length < 0 || (!packed && length > 0)) return BCS_EINVAL;
    if (!copy_size_ok(length)) return BCS_EINVAL;
    const int rc = pack_args(p, n, idx, displs, offsets, workspace, workspace_bytes);
    if (rc != BCS_OK) return rc;
    return launch_round<false>(p, n, idx, displs, length, offsets, workspace, data, const_cast<int32_t *>(packed),
                               (hipStream_t)stream);
}

int bcs_pack_plan_rounds(int32_t p, int32_t n, int64_t rounds, const int32_t *idx_table, const int64_t *displs,
                         int64_t *offsets_all, int64_t *src_all, void *stream) {
    if (p < 1 || n < 1 || rounds < 0 || rounds > 0x7fffffffll || !idx_table || !displs || !offsets_all || !src_all)
        return BCS_EINVAL;
    if ((((uintptr_t)offsets_all) | ((uintptr_t)src_all)) & 7u) return BCS_EINVAL;
    if (rounds == 0) return BCS_OK;
    const int64_t step = (int64_t)(kMaxLanes / kBlock);             // rounds a launch: a workgroup each
    for (int64_t j = 0; j < rounds; j += step) {
        PackPlan part;
        part.offsets = offsets_all + j * ((int64_t)p + 1);
        part.src = src_all + j * (int64_t)p;
        part.totals = nullptr;
        launch(kPackPlan, k_pack_plan_one, dim3((unsigned)(rounds - j < step ? rounds - j : step)), dim3(kBlock),
               (hipStream_t)stream, (uint32_t)p, (uint32_t)n, idx_table + j * (int64_t)p, displs, part);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BCS_OK : hip_fail(e);
}

int bcs_pack_round_planned(int32_t p, const int64_t *offsets, const int64_t *src, const int32_t *data, int32_t *packed,
                           int64_t capacity, void *stream) {
    if (p < 1 || !offsets || !src || !data || capacity < 0 || (!packed && capacity > 0)) return BCS_EINVAL;
    if (!copy_size_ok(capacity)) return BCS_EINVAL;
    if (capacity == 0) return BCS_OK;
    return launch_copy<true>(p, capacity, offsets, src, const_cast<int32_t *>(data), packed, (hipStream_t)stream);
}

int bcs_unpack_round_planned(int32_t p, const int64_t *offsets, const int64_t *src, int32_t *data,
                             const int32_t *packed, int64_t length, void *stream) {
    if (p < 1 || !offsets || !src || !data || length < 0 || (!packed && length > 0)) return BCS_EINVAL;
    if (!copy_size_ok(length)) return BCS_EINVAL;
    if (length == 0) return BCS_OK;
    return launch_copy<false>(p, length, offsets, src, data, const_cast<int32_t *>(packed), (hipStream_t)stream);
}

int bcs_valu_peak_launch(uint32_t blocks, uint32_t iters, uint32_t *sink, void *stream) {
    if (blocks == 0 || blocks > kMaxLanes / kBlock || iters == 0 || !sink) return BCS_EINVAL;
    launch(kValuPeak, k_valu_peak, dim3(blocks), dim3(kBlock), (hipStream_t)stream, iters, 0x2205u, sink);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BCS_OK : hip_fail(e);
}

int bcs_timing_begin(void) {
    g_timing.used = 0;
    g_timing.on = true;
    return BCS_OK;
}

int bcs_timing_stats(double *ms_sum, int64_t *launches, double *ms_min, double *ms_max) {
    Timing &t = g_timing;
    t.on = false;
    if (!ms_sum || !launches) return BCS_EINVAL;
    for (int k = 0; k < kKernelCount; ++k) {
        ms_sum[k] = 0.0;
        launches[k] = 0;
        if (ms_min) ms_min[k] = 0.0;
        if (ms_max) ms_max[k] = 0.0;
    }
    for (int i = 0; i < t.used; ++i) {
        hipError_t e = hipEventSynchronize(t.stop[i]);
        if (e != hipSuccess) return hip_fail(e);
        float ms = 0.f;
        e = hipEventElapsedTime(&ms, t.start[i], t.stop[i]);
        if (e != hipSuccess) return hip_fail(e);
        const int k = t.kid[i];
        if (ms_min && (launches[k] == 0 || (double)ms < ms_min[k])) ms_min[k] = (double)ms;
        if (ms_max && (launches[k] == 0 || (double)ms > ms_max[k])) ms_max[k] = (double)ms;
        ms_sum[k] += (double)ms;
        launches[k] += 1;
    }
    t.used = 0;
    return BCS_OK;
}

int bcs_timing_end(double *ms_sum, int64_t *launches) { return bcs_timing_stats(ms_sum, launches, nullptr, nullptr); }

const char *bcs_kernel_name(int id) { return (id >= 0 && id < kKernelCount) ? kKernelNames[id] : "?"; }

const char *bcs_strerror(int code) {
    switch (code) {
        case BCS_OK: return "success";
        case BCS_EINVAL: return "invalid argument";
        case BCS_EHIP: return "HIP call failed (see bcs_last_hip_error)";
        case BCS_ENOMEM: return "scratch memory unavailable or workspace too small";
        case BCS_ETOOBIG: return "problem needs more scratch than the fixed array of the no-allocation call holds";
        default: return "unknown bcsched error code";
    }
}

int bcs_last_hip_error(void) { return g_last_hip; }

}  // extern "C"
