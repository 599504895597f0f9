// Host build of the closed-form rows in bcs_rows.h, for the CPU tests.  Test support; not part of libbcsched.
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

template <class Pol>
void rows(const Pol &pol, uint32_t v, int32_t *recv, int32_t *send) {
    const uint32_t q = (uint32_t)pol.q(), base = row_base(pol);
    const RankPlace pl = rank_place(pol, v);
    const LowRow w = g_rows[base + (q >= 7 ? pl.ctx * 128u : 0u) + pl.low];
    const LowRow b = row_bytes(w, pl.ctx, pl.J, q);
    auto byte = [](const LowRow &x, uint32_t k) { return (int32_t)(int8_t)((k < 4 ? x.lo >> (8 * k) : x.hi >> (8 * k - 32)) & 0xffu); };
    int32_t across[7];                                       // the batch kernel's way to the low send entries
    send_low_entries(pol, pl, base, [&](uint32_t e) { return g_rows[e]; }, [&](int k, int32_t e) { across[k] = e; });
    for (uint32_t k = 0; k < q && k < 7; ++k) {
        recv[k] = byte(b, k);
        if (!Pol::kScalarSkips) {
            send[k] = across[k];
            continue;
        }
        const uint32_t t = (uint32_t)(((uint64_t)v + pol.s((int)k)) % pol.p());
        const RankPlace pt = rank_place(pol, t);
        send[k] = byte(row_bytes(g_rows[base + (q >= 7 ? pt.ctx * 128u : 0u) + pt.low], pt.ctx, pt.J, q), k);
    }
    high_entries(pol, pl, place_own(pl, w), [&](int k, int32_t e) { recv[k] = e; }, [&](int k, int32_t e) { send[k] = e; });
    recv_fix(pol, pl, w, [&](int k, int32_t e) { recv[k] = e; });
    send_fix(pol, v, pl, base, [&](uint32_t e) { return g_rows[e]; }, [&](int k, int32_t e) { send[k] = e; });
}

template <int Q>
void uniform_rows(uint32_t p, uint32_t v, int32_t *recv, int32_t *send) {
    SkipTab t;
    for (int k = 0; k <= Q; ++k) t.s[k] = ((p - 1u) >> (Q - k)) + 1u;
    t.odd = odd_levels(p, Q);
    Uniform<Q> pol;
    for (int k = 0; k <= Q; ++k) pol.S[k] = t.s[k];
    pol.tab = &t;
    pol.low = g_low.data() + (size_t)low_shape(p, Q) * kLowShapeBytes;
    rows(pol, v, recv, send);
}

template <int Q>
void uniform_for(int q, uint32_t p, uint32_t v, int32_t *recv, int32_t *send) {
    if constexpr (Q > 0) {
        if (q == Q) uniform_rows<Q>(p, v, recv, send);
        else uniform_for<Q - 1>(q, p, v, recv, send);
    }
}
}  // namespace

// rows of virtual ranks v[0..count): recv and send, 32 entries apart; wave_q 0: the one-p form, else the per-lane form
// in a wave whose largest q is wave_q
extern "C" int rc_rows(int32_t p, const int32_t *v, int64_t count, int wave_q, int32_t *recv, int32_t *send) {
    if (p < 2) return -1;
    ready();
    for (int64_t i = 0; i < count; ++i) {
        if (wave_q) rows(per_lane((uint32_t)p, wave_q), (uint32_t)v[i], recv + i * 32, send + i * 32);
        else uniform_for<kMaxQ>(ceil_log2((uint32_t)p), (uint32_t)p, (uint32_t)v[i], recv + i * 32, send + i * 32);
    }
    return 0;
}
