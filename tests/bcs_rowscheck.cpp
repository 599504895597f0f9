// Host build of the closed-form rows in bcs_rows.h and of their definition by windows, for the CPU tests.  Test support; not part of libbcsched.
#include <stddef.h>
#include <stdint.h>
#include <vector>

#include "bcs_core.h"
#include "bcs_rows.h"

using namespace bcs;

namespace {
std::vector<uint8_t> g_low;
std::vector<LowRow> g_rows;

void ready() {
    if (!g_rows.empty()) return;
    g_low.resize(kLowTableBytes);
    for (int e = 0; e < kLowTableBytes; ++e) {
        const int shape = e / kLowShapeBytes, rest = e - shape * kLowShapeBytes;
        g_low[e] = (uint8_t)low_table_entry(shape, rest >> 7, rest & 127);
    }
    g_rows.resize(kRowsAll);
    for (uint32_t e = 0; e < kRowsAll; ++e) g_rows[e] = low_row_entry(e, g_low.data());
}

PerLane per_lane(uint32_t p, int wave_q) {
    PerLane pol;
    pol.pm1 = p - 1u;
    pol.ql = ceil_log2(p);
    pol.wave_top = (wave_q > pol.ql ? wave_q : pol.ql) - 1;
    pol.odd = odd_levels(p, pol.ql);
    pol.low = g_low.data() + (size_t)low_shape(p, pol.ql) * kLowShapeBytes;
    return pol;
}

LowRow read(uint32_t e) { return g_rows.at(e); }          // throws where a kernel would read past the table

// Receive and send rows the way the kernels make them.  Returns false where the low send entries, which come from v's own
// block and the next one, differ from those of the to-neighbours' own rows.
template <class Pol>
bool rows(const Pol &pol, uint32_t v, int32_t *recv, int32_t *send) {
    const uint32_t q = (uint32_t)pol.q(), base = row_base(pol);
    const RankPlace pl = rank_place(pol, v);
    const LowRow w = read(base + pl.ctx * 128u + pl.low);
    const LowRow b = row_bytes(w, pl.ctx, pl.J, q);
    auto byte = [](const LowRow &x, uint32_t k) { return (int32_t)(int8_t)((k < 4 ? x.lo >> (8 * k) : x.hi >> (8 * k - 32)) & 0xffu); };
    bool same = true;
    for (uint32_t k = 0; k < q && k < (uint32_t)kLowLevels; ++k) recv[k] = byte(b, k);
    send_low_entries(pol, pl, base, read, [&](int k, int32_t e) { if (k < (int)q) send[k] = e; });
    for (uint32_t k = 0; k < q && k < (uint32_t)kLowLevels; ++k) {
        const uint32_t t = (uint32_t)(((uint64_t)v + pol.s((int)k)) % pol.p());
        const RankPlace pt = rank_place(pol, t);
        same &= send[k] == byte(row_bytes(read(base + pt.ctx * 128u + pt.low), pt.ctx, pt.J, q), k);
    }
    high_entries(pol, pl, place_own(pl, w), [&](int k, int32_t e) { recv[k] = e; }, [&](int k, int32_t e) { send[k] = e; });
    recv_fix(pol, pl, w, [&](int k, int32_t e) { recv[k] = e; });
    send_fix(pol, v, pl, base, read, [&](int k, int32_t e) { send[k] = e; });
    return same;
}

template <int Q>
bool uniform_rows(uint32_t p, uint32_t v, int32_t *recv, int32_t *send) {
    SkipTab t;
    for (int k = 0; k <= Q; ++k) t.s[k] = ((p - 1u) >> (Q - k)) + 1u;
    t.odd = odd_levels(p, Q);
    Uniform<Q> pol;
    for (int k = 0; k <= Q; ++k) pol.S[k] = t.s[k];
    pol.tab = &t;
    pol.low = g_low.data() + (size_t)low_shape(p, Q) * kLowShapeBytes;
    return rows(pol, v, recv, send);
}

template <int Q>
bool uniform_for(int q, uint32_t p, uint32_t v, int32_t *recv, int32_t *send) {
    if constexpr (Q > 0) {
        return q == Q ? uniform_rows<Q>(p, v, recv, send) : uniform_for<Q - 1>(q, p, v, recv, send);
    }
    return false;
}
}  // namespace

// rows of virtual ranks v[0..count): recv and send, 32 entries apart; wave_q 0: the one-p form, else the per-lane form
// in a wave whose largest q is wave_q
extern "C" int rc_rows(int32_t p, const int32_t *v, int64_t count, int wave_q, int32_t *recv, int32_t *send) {
    if (p < 2) return -1;
    ready();
    for (int64_t i = 0; i < count; ++i) {
        const bool same = wave_q ? rows(per_lane((uint32_t)p, wave_q), (uint32_t)v[i], recv + i * 32, send + i * 32)
                                 : uniform_for<kMaxQ>(ceil_log2((uint32_t)p), (uint32_t)p, (uint32_t)v[i], recv + i * 32,
                                                      send + i * 32);
        if (!same) return 1;
    }
    return 0;
}

// the same rows by their definition: every receive round from its windows (Alg. 4), every send entry from the receive row
// of the to-neighbour (Alg. 5)
extern "C" int rc_windows(int32_t p, const int32_t *v, int64_t count, int32_t *recv, int32_t *send) {
    if (p < 2) return -1;
    ready();
    const PerLane pol = per_lane((uint32_t)p, 0);
    for (int64_t i = 0; i < count; ++i) {
        recv_row(pol, (uint32_t)v[i], pol.ql - 1, [&](int k, int e) { recv[i * 32 + k] = e; });
        for (int k = 0; k < pol.ql; ++k) {
            const uint32_t t = (uint32_t)(((uint64_t)(uint32_t)v[i] + pol.s(k)) % (uint32_t)p);
            recv_row(pol, t, k, [&](int j, int e) { if (j == k) send[i * 32 + k] = e; });
        }
    }
    return 0;
}
