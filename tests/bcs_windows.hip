// Checks rows in device memory against their definition: receive rounds from their windows (Alg. 4, csrc/bcs_core.h); send
// entries of all ranks by look-up in the receive rows that are checked with them (Alg. 9, second loop), of a part of the
// ranks from the to-neighbour's rounds (Alg. 5).  One rank a lane: the construction shares with the library's rows the table
// of the low levels and no more.  Test support; not part of libbcsched.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "bcs_core.h"

using namespace bcs;

namespace {
__global__ __launch_bounds__(256) void k_check(uint32_t p, int q, uint32_t odd, uint32_t root, uint32_t r0, uint32_t count,
                                               const uint8_t *__restrict__ low, const int32_t *__restrict__ recv,
                                               const int32_t *__restrict__ send, unsigned long long *__restrict__ bad) {
    const uint64_t i = (uint64_t)blockIdx.x * 256u + threadIdx.x;
    const bool live = i < count;
    const uint32_t at = live ? (uint32_t)i : 0u;                      // lanes past the end repeat a rank and count nothing
    const uint32_t r = r0 + at, v = r >= root ? r - root : r + (p - root);
    PerLane pol;
    pol.pm1 = p - 1u;
    pol.ql = q;
    pol.wave_top = q - 1;
    pol.odd = odd;
    pol.low = low;
    uint32_t wrong = 0;
    const uint64_t row = (uint64_t)at * (uint32_t)q;
    if (recv) recv_row(pol, v, q - 1, [&](int k, int e) { wrong += recv[row + k] != e ? 1u : 0u; });
    const bool look_up = recv && count == p;                          // all ranks: the to-neighbour's row is here
    if (send)
        for (int k = 0; k < q; ++k) {
            const uint32_t s = pol.s(k);
            if (look_up) {
                const uint32_t t = r + s >= p ? r + s - p : r + s;
                wrong += send[row + k] != recv[(uint64_t)t * (uint32_t)q + k] ? 1u : 0u;
                continue;
            }
            const uint32_t t = v + s >= p ? v + s - p : v + s;
            recv_row(pol, t, k, [&](int j, int e) { wrong += j == k && send[row + k] != e ? 1u : 0u; });
        }
    if (live && wrong) atomicAdd(bad, (unsigned long long)wrong);
}

uint8_t *g_low = nullptr;                                             // the low-level table on the device
unsigned long long *g_bad = nullptr;
}  // namespace

// Enqueues (on the default stream) the check of the rows of ranks [r0, r1); recv, send: device, rows of q entries, either may
// be NULL.  0, or -1 for bad arguments or a HIP error.
extern "C" int bw_check(int32_t p, int32_t root, int32_t r0, int32_t r1, const int32_t *recv, const int32_t *send) {
    if (p < 2 || root < 0 || root >= p || r0 < 0 || r0 > r1 || r1 > p) return -1;
    if (r0 == r1) return 0;
    if (!g_low) {
        std::vector<uint8_t> table(kLowTableBytes);
        for (int e = 0; e < kLowTableBytes; ++e) {
            const int shape = e / kLowShapeBytes, rest = e - shape * kLowShapeBytes;
            table[e] = (uint8_t)low_table_entry(shape, rest >> 7, rest & 127);
        }
        const unsigned long long none = 0;
        uint8_t *dev;
        if (hipMalloc(&g_bad, sizeof *g_bad) != hipSuccess || hipMalloc(&dev, kLowTableBytes) != hipSuccess) return -1;
        if (hipMemcpy(g_bad, &none, sizeof none, hipMemcpyHostToDevice) != hipSuccess) return -1;
        if (hipMemcpy(dev, table.data(), kLowTableBytes, hipMemcpyHostToDevice) != hipSuccess) return -1;
        g_low = dev;
    }
    const int q = ceil_log2((uint32_t)p);
    const uint32_t count = (uint32_t)(r1 - r0);
    hipLaunchKernelGGL(k_check, dim3((unsigned)(((uint64_t)count + 255) / 256)), dim3(256), 0, 0, (uint32_t)p, q,
                       odd_levels((uint32_t)p, q), (uint32_t)root, (uint32_t)r0, count,
                       (const uint8_t *)(g_low + (size_t)low_shape((uint32_t)p, q) * kLowShapeBytes), recv, send, g_bad);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Entries found to differ since the last call, or -1; waits for the checks.
extern "C" int64_t bw_result() {
    unsigned long long bad = 0, none = 0;
    if (!g_bad) return 0;
    if (hipMemcpy(&bad, g_bad, sizeof bad, hipMemcpyDeviceToHost) != hipSuccess) return -1;
    if (hipMemcpy(g_bad, &none, sizeof none, hipMemcpyHostToDevice) != hipSuccess) return -1;
    return (int64_t)bad;
}
