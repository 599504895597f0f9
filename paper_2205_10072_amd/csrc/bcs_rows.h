// bcs_rows.h: receive and send rows in closed form, without windows (the definition by windows is in bcs_core.h).
// Written once for the GPU lanes and for the host build of the CPU tests.
//
// A rank v is read as its greedy sum of skips (the digit mask D(v) of bcs_core.h), cut at level 7: H is the part made
// of skips[7] and up, low the rest, low < skips[7] <= 128.  The ranks with one H are a block; its first rank (low = 0)
// holds baseblock j, the lowest digit of H (the lap digit q, which is no block, for H = 0).
// Notation: o(a, b) = number of odd levels k (2 skips[k] - skips[k+1] = 1) with a <= k < b.
//
// Rounds below 7.  Their windows reach skips[7] + 7 ranks back at most: into v's block, the block before it and a few
// ranks of the one before that.  What these look like follows from skips[7], low and
//   - digit 7 of v clear (H's lowest digit is J > 7): the block before lacks its last o(7, J) ranks and begins with a
//     rank that holds block 7; the one before it is whole;
//   - digit 7 set (J the next digit above it): the block before is whole and begins with a rank that holds J; the one
//     before that lacks its last o(7, J) ranks;
//   - whether J is the lap digit.
// So the seven entries are read from a table of 64 shapes (skips[7]) x 4 families x 25 values of o(7, J) x low, eight
// bytes an entry, with J as the one symbol that is filled in.  q = 7 (the ring is one block, which precedes itself) has
// a context of its own and each p <= 64 a shape of its own.  The table is filled by Alg. 4 on the smallest system that
// shows the context.
//
// Rounds i >= 7 of the receive row, `next` the next digit of v above i:
//   - digit i set: the entry is next - q, or v's baseblock when there is none (the home round);
//   - digit i clear: i - q, except for v = A + skips[j] + low with digits 7..j-1 clear (A the digits above j) and low
//     small.  There block i's last holder lies low + skips[i] - o(i, j) ranks back (the blocks before v's are cut),
//     which is in round i's window for low >= o(i, j) and has been in round i-1's otherwise: a rank whose rounds below
//     7 already took block 7 goes on taking i + 1 in round i while low < o(i+1, j), then catches up with the one
//     block x of 0..6 that it lacks and is regular from there.  x is kept in the table (7: none is lacking).
// Rounds k >= 7 of the send row: entry k of the receive row of t = v + skips[k].
//   - digit k set: the addition carries to the lowest clear digit z above k and t's digit k is clear: k - q;
//   - digit k clear: t has v's digits and digit k: next - q, or v's baseblock when there is none (k itself for v = 0);
//   - the one exception of each kind: for k = the lowest clear digit from 7 up, with z the lowest clear digit above k,
//     the upper copy that t would lie in ends skips[7] - o(7, z) into its last block.  For low beyond that t is z's
//     head plus dl = low + o(7, z) - skips[7], whose entry k is k + 1 - q for dl < o(k+1, z), else t's x - q;
//     and for k = 7 set with low = 0 t's round 7 is the one that catches up where t's x is not 7.
// The argument covers where the holders lie; that Alg. 4 then acts as described is checked against its definition by
// windows (bcs_core.h, made for every rank on the GPU; send rows by look-up in those rows, of slices by Alg. 5): every rank
// of every p up to 200 000 and of 140 000 larger p up to 2^23, and 40 000 slices of 2^16 ranks of p up to 2^31, at and
// around both ends of blocks, the p with few, many and random odd levels, under random roots (3.0 10^11 ranks): no
// difference.  The CPU and GPU tests repeat this against windows and the oracle at smaller counts.
#ifndef BCS_ROWS_H
#define BCS_ROWS_H

#include "bcs_core.h"

namespace bcs {

constexpr int kCtxD = kMaxQ - kLowLevels + 1;            // values of o(7, J): 0..24
constexpr int kCtxRing = 4 * kCtxD;                      // q = 7
constexpr int kCtxCount = kCtxRing + 1;
constexpr int kRowShapes = 64;                           // skips[7] = 65..128
constexpr uint32_t kCatchUpMinD = 17;                    // see send_fix
constexpr uint32_t kRowsPerShape = kCtxCount * 128u;
constexpr uint32_t kRowsBig = kRowShapes * kRowsPerShape;
constexpr uint32_t kRowsAll = kRowsBig + 64u * 64u;      // then p = 1..64, 64 entries each

// One table entry.  Byte i < 7, bits 0..2: the block of round i; hi bits 19..21: x; hi bits 24..26: the baseblock of
// `low` (7: low is 0); hi bits 27..29: the round that gets an extra term (7: none): J (its byte is 0) or, in the
// contexts without higher digits, q in the home round, which turns "block - q" into the baseblock.
struct LowRow {
    uint32_t lo, hi;
};

BCS_HD uint32_t row_own(const LowRow &w) { return (w.hi >> 24) & 7u; }
BCS_HD uint32_t row_pos(const LowRow &w) { return (w.hi >> 27) & 7u; }
BCS_HD uint32_t row_lacks(const LowRow &w) { return (w.hi >> 19) & 7u; }

// Entry `e` of the table; lowtab: the low-level table of bcs_core.h (all shapes), which Alg. 4 reads.
BCS_HD LowRow low_row_entry(uint32_t e, const uint8_t *lowtab) {
    LowRow w = {0u, 0u};
    uint32_t p, H = 0u, low;
    int J = 32;
    if (e >= kRowsBig) {
        p = ((e - kRowsBig) >> 6) + 1u;
        low = e & 63u;
    } else {
        const uint32_t S = e / kRowsPerShape + 65u, rest = e % kRowsPerShape;
        const int ctx = (int)(rest >> 7), fam = ctx / kCtxD, d = ctx % kCtxD;
        low = rest & 127u;
        if (ctx == kCtxRing) {
            p = S;
        } else {
            // J = 7 + d with d odd levels below it.  Where digit 7 is set the odd levels start at 8 if there is room:
            // with level 7 even the block is whole and every low occurs.
            const bool lap = (fam & 1) != 0, upper = fam >= 2;
            const int top = lap ? kMaxQ : kMaxQ - 1;
            const int from = upper && d > 0 && 8 + d <= top ? 8 : 7;
            J = d > 0 ? from + d : 8;
            if (J > top) return w;                             // no such system
            uint64_t s = S;
            for (int l = 7; l < J; ++l) s = 2u * s - (l >= from && l < from + d ? 1u : 0u);
            H = (lap ? 0u : (uint32_t)s) + (upper ? S : 0u);
            const uint64_t pp = lap ? s : 2u * s;               // level J is even
            if (pp > 0x80000000ull) return w;                   // no such system
            p = (uint32_t)pp;
            if (lap) J = 32;                                    // no block
        }
    }
    const uint32_t v = H + low;
    if (v >= p || v < H) return w;
    PerLane pol;
    pol.pm1 = p - 1u;
    pol.ql = ceil_log2(p);
    pol.wave_top = kMaxQ - 1;
    pol.odd = odd_levels(p, pol.ql);
    pol.low = lowtab + (size_t)low_shape(p, pol.ql) * kLowShapeBytes;
    const int q = pol.ql;
    const uint32_t dv = digits(pol, v);
    const int home = 31 - BCS_CLZ(dv);
    const uint32_t dlow = dv & 127u;
    const uint32_t own = dlow ? (uint32_t)__builtin_ctz(dlow) : 7u;
    uint32_t have = dlow ? 1u << own : 0u, pos = 7u;
    recv_row(pol, v, kLowLevels - 1, [&](int i, int val) {
        uint32_t b = (uint32_t)(i == home ? val : val + q);
        if (i == home || (int)b == J) pos = (uint32_t)i;
        have |= 1u << (b & 31u);
        if ((int)b == J) b = 0u;
        if (i < 4) w.lo |= (b & 7u) << (8 * i);
        else w.hi |= (b & 7u) << (8 * (i - 4));
    });
    const uint32_t lacks = ~have & 127u;
    w.hi |= (lacks ? (uint32_t)__builtin_ctz(lacks) : 7u) << 19 | own << 24 | pos << 27;
    return w;
}

// Where a rank stands: its block and its place in it.
struct RankPlace {
    uint32_t low;                        // value of the digits below 7
    uint32_t up;                         // digits 7 and up with the lap digit q (q >= 7)
    uint32_t J;                          // the digit that the context depends on
    uint32_t ctx;
};

BCS_HD uint32_t odd_between(uint32_t odd, uint32_t from, uint32_t to) {           // o(from, to), from <= to <= 31
    return (uint32_t)__builtin_popcount((odd & ((1u << (to & 31u)) - 1u)) >> (from & 31u));
}

// context of a block: up = its digits from 7 up with the lap digit
template <class Pol>
BCS_HD void place_context(const Pol &pol, RankPlace &pl) {
    const uint32_t q = (uint32_t)pol.q();
    const uint32_t upper = (pl.up >> kLowLevels) & 1u;
    const uint32_t rest = pl.up & ~(1u << kLowLevels);
    pl.J = rest ? (uint32_t)__builtin_ctz(rest) : q;
    const uint32_t d = odd_between(pol.odd_mask(), kLowLevels, pl.J);
    pl.ctx = (2u * upper + (pl.J == q ? 1u : 0u)) * (uint32_t)kCtxD + d;
    if (q == (uint32_t)kLowLevels) pl.ctx = kCtxRing;
}

// digits 7 and up of v, largest first: two vector ops a level take the skip off (the difference wraps to a large
// number when the skip is larger) and one collects the sign
template <class Pol>
BCS_HD RankPlace rank_place(const Pol &pol, uint32_t v) {
    RankPlace pl;
    const int q = pol.q();
    uint32_t y = v, clear = 0u;
    if constexpr (Pol::kScalarSkips) {
#pragma unroll
        for (int k = pol.top(); k >= kLowLevels; --k) {
            const uint32_t t = y - pol.s(k);
            y = t < y ? t : y;
            clear = (clear << 1) | (t >> 31);
        }
        const int n = pol.top() + 1 - kLowLevels;
        pl.up = n > 0 ? (~clear & (0xffffffffu >> (32 - (n > 0 ? n : 1)))) << kLowLevels : 0u;
    } else {
        // level q-1-m in step m, whose skip is ((p-1) >> (m+1)) + 1; a lane past its level 7 takes nothing off
        const int steps = pol.top() + 1 - kLowLevels, mine = q - kLowLevels;
        uint32_t g = pol.pm1;
#pragma unroll 1
        for (int m = 0; m < steps; ++m) {
            g = m < mine ? g >> 1 : 0x7fffffffu;
            const uint32_t t = y + ~g;
            y = t < y ? t : y;
            clear = (clear << 1) | (t >> 31);
        }
        pl.up = mine > 0 ? ((~clear & (0xffffffffu >> (32 - steps))) >> (steps - mine)) << kLowLevels : 0u;
    }
    pl.low = y;
    pl.up |= 1u << (q & 31);
    if (q < kLowLevels) {
        pl.J = (uint32_t)q;
        pl.ctx = 0u;
    } else {
        place_context(pol, pl);
    }
    return pl;
}

// index of the row of (context, low) in the table of this p
template <class Pol>
BCS_HD uint32_t row_base(const Pol &pol) {
    const int q = pol.q();
    const uint32_t p = pol.p();
    return q >= kLowLevels ? ((p - 1u) >> (q - kLowLevels)) * kRowsPerShape - 64u * kRowsPerShape : kRowsBig + (p - 1u) * 64u;
}

// the seven entries of a row as bytes (bytes 0..3 in lo, 4..6 in hi)
BCS_HD LowRow row_bytes(const LowRow &w, uint32_t ctx, uint32_t J, uint32_t q) {
    const bool in_low = ctx - (uint32_t)kCtxD < (uint32_t)kCtxD || ctx == (uint32_t)kCtxRing || q < (uint32_t)kLowLevels;
    const uint32_t extra = in_low ? q : J;                            // no digit from 7 up: the home round is one of these
    const uint32_t sh = 8u * row_pos(w);
    const uint64_t add = (uint64_t)extra << (sh & 63u);
    const uint32_t qs = q * 0x01010101u, top = 0x80808080u;
    LowRow r;
    r.lo = ((((w.lo & 0x07070707u) + (uint32_t)add) | top) - qs) ^ top;
    r.hi = ((((w.hi & 0x00070707u) + ((uint32_t)(add >> 32) & 0x00ffffffu)) | top) - qs) ^ top;
    return r;
}

// Receive entries from round 7 up that the digits alone do not give; fix(i, value).  w: v's row of the table.
template <class Pol, class Fix>
BCS_HD void recv_fix(const Pol &pol, const RankPlace &pl, const LowRow &w, Fix fix) {
    const uint32_t q = (uint32_t)pol.q();
    if (pl.ctx >= 2u * (uint32_t)kCtxD || row_lacks(w) == 7u || q <= (uint32_t)kLowLevels) return;
    uint32_t i = kLowLevels;
    for (; i + 1u < pl.J && pl.low < odd_between(pol.odd_mask(), i + 1u, pl.J); ++i) fix((int)i, (int)(i + 1u - q));
    if (i < pl.J) fix((int)i, (int)(row_lacks(w) - q));
}

// lowest clear digit of `up` (with the lap digit) at or above k, at most q
BCS_HD uint32_t clear_digit(uint32_t up, uint32_t k, uint32_t q) {
    const uint32_t c = (~up >> k) << k;
    const uint32_t z = c ? (uint32_t)__builtin_ctz(c) : 32u;
    return z < q ? z : q;
}

// The block after v's: how many ranks v's block holds and the context that follows it.
struct NextBlock {
    uint32_t size, ctx, J;
};

template <class Pol>
BCS_HD NextBlock next_block(const Pol &pol, const RankPlace &pl) {
    const uint32_t q = (uint32_t)pol.q(), p = pol.p();
    NextBlock nb;
    if (q <= (uint32_t)kLowLevels) {                                      // the ring is one block
        nb.size = p;
        nb.ctx = pl.ctx;
        nb.J = pl.J;
        return nb;
    }
    const uint32_t bare = pl.up & ~(1u << (q & 31u));
    const bool upper = (bare >> kLowLevels) & 1u;
    const uint32_t z = clear_digit(bare, kLowLevels, q);                   // upper: where the next head's digit is
    const uint32_t cut = odd_between(pol.odd_mask(), kLowLevels, z);       // 0 for digit 7 clear (z = 7)
    nb.size = ((p - 1u) >> (q - (uint32_t)kLowLevels)) + 1u - cut;
    nb.ctx = upper ? (z == q ? (uint32_t)kCtxD : 0u) + cut : pl.ctx + 2u * (uint32_t)kCtxD;   // digit 7 clear: it gets set
    nb.J = upper ? z : pl.J;
    return nb;
}

// Send entries below round 7 without other lanes' help: entry k is the low round k of rank v + skips[k], which lies in
// v's block or in the next one.
template <class Pol, class Read, class Emit>
BCS_HD void send_low_entries(const Pol &pol, const RankPlace &pl, uint32_t base, Read read, Emit emit) {
    const uint32_t q = (uint32_t)pol.q();
    const NextBlock nb = next_block(pol, pl);
    auto extra_of = [&](uint32_t ctx, uint32_t J) {
        return q <= (uint32_t)kLowLevels || ctx - (uint32_t)kCtxD < (uint32_t)kCtxD ? q : J;
    };
    const uint32_t here = base + pl.ctx * 128u, next = base + nb.ctx * 128u;
    const uint32_t extra_here = extra_of(pl.ctx, pl.J), extra_next = extra_of(nb.ctx, nb.J);
#pragma unroll
    for (uint32_t k = 0; k < (uint32_t)kLowLevels; ++k) {
        const uint32_t s = k < q ? ((pol.p() - 1u) >> (q - k)) + 1u : 0u;   // lanes with fewer rounds: some entry, not used
        const uint32_t to = pl.low + s;
        const bool over = to >= nb.size;
        const LowRow w = read(over ? next + to - nb.size : here + to);
        const uint32_t block = (k < 4u ? w.lo >> (8u * k) : w.hi >> (8u * k - 32u)) & 7u;
        const uint32_t add = row_pos(w) == k ? (over ? extra_next : extra_here) : 0u;
        emit((int)k, (int32_t)(block + add - q));
    }
}

// Rounds 7 and up from the digits, largest first; own = v's baseblock.  Three vector ops a level for both entries.
template <class Pol, class EmitR, class EmitS>
BCS_HD void high_entries(const Pol &pol, const RankPlace &pl, uint32_t own, EmitR emit_recv, EmitS emit_send) {
    const int q = pol.q();
    const uint32_t bare = pl.up & ~(1u << (q & 31));
    int32_t next = (int32_t)own;                                          // what a round without a digit above it gets
#pragma unroll
    for (int k = pol.top(); k >= kLowLevels; --k) {
        const int32_t set = -(int32_t)((bare >> (k & 31)) & 1u), here = k - q;
        const int32_t r = (set & next) | (~set & here);
        next = (set & here) | (~set & next);
        if (k < q) {
            emit_recv(k, r);
            emit_send(k, next);
        }
    }
}

// v's baseblock: the lowest digit (any value for v = 0)
BCS_HD uint32_t place_own(const RankPlace &pl, const LowRow &w) {
    const uint32_t low = row_own(w);
    return low < 7u ? low : (uint32_t)__builtin_ctz(pl.up);
}

// Send entries from round 7 up that the digits alone do not give; read(row index) reads the table.
template <class Pol, class Read, class Fix>
BCS_HD void send_fix(const Pol &pol, uint32_t v, const RankPlace &pl, uint32_t base, Read read, Fix fix) {
    const uint32_t q = (uint32_t)pol.q(), odd = pol.odd_mask();
    if (q <= (uint32_t)kLowLevels) return;
    const uint32_t bare = pl.up & ~(1u << (q & 31u));                    // without the lap digit
    if (v == 0u)
        for (uint32_t k = kLowLevels; k < q; ++k) fix((int)k, (int)k);
    const uint32_t k = clear_digit(bare, kLowLevels, q);
    // a head with digit 7 set: t's x is 7 (nothing to mend) for fewer than kCatchUpMinD odd levels, in all 64 shapes
    const bool head = pl.low == 0u && k > (uint32_t)kLowLevels && odd_between(odd, kLowLevels, k) >= kCatchUpMinD;
    const uint32_t z = head ? k : clear_digit(bare, k + 1u < q ? k + 1u : q, q);
    const uint32_t d = odd_between(odd, kLowLevels, z);
    const uint32_t s7 = ((pol.p() - 1u) >> (q - (uint32_t)kLowLevels)) + 1u;
    const bool past = !head && k < q && pl.low + d >= s7;
    if (!head && !past) return;
    const uint32_t dl = head ? d : pl.low + d - s7;
    if (past && dl < odd_between(odd, k + 1u, z)) {
        fix((int)k, (int)(k + 1u - q));
        return;
    }
    const LowRow w = read(base + ((z == q ? (uint32_t)kCtxD : 0u) + d) * 128u + dl);
    fix(head ? kLowLevels : (int)k, (int)(row_lacks(w) - q));
}

}  // namespace bcs
#endif  // BCS_ROWS_H
