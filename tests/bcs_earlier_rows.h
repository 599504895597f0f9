// Earlier forms of the rows, which no kernel uses any more and the host tests hold against the oracle entry by entry: rounds
// taken from the rank's own digits, receive rows from a table of all ranks' digit masks, send entries without the
// to-neighbour's rounds.  The kernels' form is csrc/bcs_rows.h, its definition by windows csrc/bcs_core.h.  Test support; not
// part of libbcsched.
#ifndef BCS_EARLIER_ROWS_H
#define BCS_EARLIER_ROWS_H

#include "bcs_core.h"

namespace bcs {

// One round of Alg. 4 for callers that keep B themselves: the new block joins B, the entry goes to emit.
template <class Pol, class DigitsOf, class Emit>
BCS_HD void recv_round(const Pol &pol, uint32_t v, int i, uint32_t s_n, uint32_t d_lo, uint32_t d_hi, int home,
                       int own, uint32_t &B, DigitsOf digits_of, Emit emit) {
    const int q = pol.q();
    int blk;
    const int val = recv_round_value(pol, v, i, s_n, d_lo, d_hi, home, own, B, digits_of, blk);
    const bool active = i < q;
    // one emit for both kinds of round, so that a wave with lanes of both kinds does not run it twice
    B |= active ? (1u << (blk & 31)) : 0u;
    if (active) emit(i, val);
}

// Rounds that need no window (one p per launch).  With D(v) the digit mask of the rank, low the value of its
// digits below i and c the number of odd levels below i, round i's entry is
//   - the rank's baseblock when i is its highest digit (Alg. 4's first branch);
//   - (next digit j of v above i) - q when digit i is set and low >= c.  The rank w = v - skips[i] - low has the
//     digits of v above i and nothing below (taking digits out of a greedy sum leaves a greedy sum), so its
//     baseblock is j; low < skips[i+1] - skips[i] puts it into the round's first window, whose other end has digit
//     j clear, so j is the window's largest block; and v cannot have come by block j before: its own baseblock
//     is at or below i, the earlier rounds' windows lie above v - skips[i] except for round i-1's second range,
//     which reaches fewer than c ranks below it (and w lies low ranks below), and the next rank with baseblock j
//     is more than 2 skips[i] above w;
//   - i - q when digit i is clear and low keeps clear of the ends of its range: taking skips[i] from v borrows
//     from the next digit j above (the lap digit when there is none), which sets digits i..j-1 and lowers the low
//     part by the number o of odd levels in [i, j) (skips[j] - skips[i] = sum of skips[i..j-1] minus o).  With
//     low' = low - o >= 0: the rank w = v - skips[i] - low' has lowest digit i and lies in the first window when
//     low' < skips[i+1] - skips[i]; every other rank of the window shares the digits above i and has a lower
//     lowest digit; and block i is new: v's baseblock is not i, the earlier rounds reach down to
//     v - skips[i] - c + 1 only, which misses w when low' >= c, and the next rank with lowest digit i lies
//     skips[i+1] - (odd levels in [i+1, j)) above w, past v.  The test allows for every o from 0 to the number of
//     odd levels from i up and keeps twice the margin this needs (it is case (b) of send_row_direct below).
// Both are also checked against the oracle (every rank of every p the CPU tests run this code on, the full-size
// configurations on the GPU while kernels used this form).  Low rounds rarely agree
// across the 64 ranks of a wave, so the test starts at round kDigitRoundsFrom.
constexpr int kDigitRoundsFrom = 6;
constexpr int kTabAhead = 10;                           // recv_row_tab reads the end points of rounds below this ahead

// dl = D(v) with the lap digit (so that there always is a digit above round i); returns whether the entry could
// be taken from the digits and leaves it in val, its block (the lap digit's index q for the home round, which
// Alg. 4's set B never holds) in blk.  Written with masks instead of conditions: one straight run of vector ops.
template <class Pol>
BCS_HD bool round_from_digits(const Pol &pol, uint32_t dl, int i, uint32_t s_i, uint32_t low, int home, int own,
                              int &val, int &blk) {
    const int q = pol.q();
    const uint32_t odd = pol.odd_mask();
    const int mrg = 2 * __builtin_popcount(odd & ((2u << (i & 31)) - 1u)) + 2;
    const int c1 = mrg + __builtin_popcount(odd >> (i & 31));          // low must exceed this ...
    const int c2 = (int)s_i - mrg - 1;                                  // ... and stay below this
    const uint32_t width = c2 > c1 + 1 ? (uint32_t)(c2 - c1 - 1) : 0u;
    const uint32_t m = 0u - ((dl >> (i & 31)) & 1u);                    // all ones when digit i is set
    const uint32_t above = (dl >> (i & 31)) >> 1;                       // never 0: the lap digit
    const uint32_t next = (uint32_t)(__builtin_ctz(above) + i + 1);
    blk = (int)((m & next) | (~m & (uint32_t)i));
    val = i == home ? own : blk - q;
    const uint32_t x = (low - (uint32_t)c1 - 1u) & ~m;
    const uint32_t cbelow = (uint32_t)__builtin_popcount(odd & ((1u << (i & 31)) - 1u));   // odd levels below i
    return (m != 0u && low >= cbelow) || x < width;
}

template <class Pol, class Emit>
BCS_HD void recv_row_mixed_from(const Pol &pol, uint32_t v, uint32_t dv, int last, Emit emit);

// Alg. 4's row with the rounds that the digits give taken from them (one p), the others from windows.
template <class Pol, class Emit>
BCS_HD void recv_row_mixed(const Pol &pol, uint32_t v, int last, Emit emit) {
    recv_row_mixed_from(pol, v, digits(pol, v), last, emit);
}

// recv_row_mixed for a caller that already has dv = digits(pol, v)
template <class Pol, class Emit>
BCS_HD void recv_row_mixed_from(const Pol &pol, uint32_t v, uint32_t dv, int last, Emit emit) {
    const uint32_t p = pol.p();
    const int q = pol.q();
    const uint32_t lap = 1u << (q & 31);
    const int home = 31 - BCS_CLZ(dv);                    // -1 for the root
    const int own = dv ? __builtin_ctz(dv) : 0;
    uint32_t B = v ? (1u << own) : 0u;
    // Digits of v - skips[n] with the lap digit.  When skips[n] is part of v's greedy sum, taking it out leaves the
    // greedy sum of v - skips[n] (the ranks below it were below skips[n] before and still are), and for n = q the
    // end point is v itself: no walk.  The high digits of consecutive ranks agree, so whole waves take this path.
    // (Lanes with unrelated p never agree on it, so the per-lane policy does not ask.)
    auto end_digits = [&](int n, uint32_t s) -> uint32_t {
        const bool ahead = v >= s;
        const uint32_t y = ahead ? v - s : v + p - s;
        if constexpr (Pol::kScalarSkips) {
            const uint32_t nbit = 1u << (n & 31);
            const bool direct = (n == q) || (dv & nbit) != 0u;
            uint32_t d = (n == q) ? dv : ((dv & ~nbit) | lap);
            if (BCS_WAVE_ANY(!direct)) d = digits(pol, y) | (ahead ? lap : 0u);
            return d;
        } else {
            return digits(pol, y) | (ahead ? lap : 0u);
        }
    };
    uint32_t s_i = pol.sdyn(0);
    uint32_t d_hi = end_digits(0, s_i);
    bool have_hi = true;                                  // wave-uniform: d_hi holds the digits of v - skips[i]
    uint32_t low = 0;                                     // value of v's digits below round i
#pragma unroll 1
    for (int i = 0; i <= last; ++i) {
        const uint32_t s_n = pol.sdyn(i + 1);
        int val = 0, blk = 0;
        bool easy = false, window = true;
        if constexpr (Pol::kScalarSkips) {
            easy = i >= kDigitRoundsFrom && round_from_digits(pol, dv | lap, i, s_i, low, home, own, val, blk);
            window = BCS_WAVE_ANY(!easy);
        }
        if (window) {
            if (!have_hi) d_hi = end_digits(i, s_i);
            const uint32_t d_lo = end_digits(i + 1, s_n);
            int wb;
            const int w = recv_round_value(pol, v, i, s_n, d_lo, d_hi, home, own, B,
                                           [&](uint32_t r) { return digits(pol, r); }, wb);
            val = easy ? val : w;
            blk = easy ? blk : wb;
            d_hi = d_lo;
        }
        have_hi = window;
        const bool active = i < q;                        // per-lane q may be below the wave's bound
        B |= active ? (1u << (blk & 31)) : 0u;
        if (active) emit(i, val);
        low += (0u - ((dv >> (i & 31)) & 1u)) & s_i;
        s_i = s_n;
    }
}

// The same row with every digit mask read from a table of all ranks' masks (dtab[y] = digits of rank y, filled
// by one walk per rank beforehand): every end point of every window is some rank.  All q rounds, unrolled, so that
// the skips are the policy's registers and the reads of later rounds can be issued ahead of the rounds that use
// them.
template <class Pol, class Emit>
BCS_HD void recv_row_tab(const Pol &pol, const uint32_t *__restrict__ dtab, uint32_t v, Emit emit) {
    static_assert(Pol::kScalarSkips, "one p per launch: the inert skips of the per-lane policy are no table indices");
    constexpr int kQ = Pol::kTopLevel + 1;
    const uint32_t p = pol.p();
    const uint32_t lap = 1u << (kQ & 31);
    // d(n): digits of v - skips[n] with the lap digit.  Those of the low rounds, which always need their windows,
    // are read ahead; the others only by the few waves that need a window in a high round.
    constexpr int kAhead = kQ < kTabAhead ? kQ : kTabAhead;
    auto end_point = [&](int n) -> uint32_t {
        const uint32_t s = pol.s(n);
        const bool ahead = v >= s;
        return dtab[ahead ? v - s : v + p - s] | (ahead ? lap : 0u);
    };
    uint32_t d[kAhead + 1];
#pragma unroll
    for (int n = 0; n <= kAhead; ++n) d[n] = end_point(n);
    const uint32_t dv = dtab[v];                         // skips[q] = p: the rank itself, no lap
    const int home = 31 - BCS_CLZ(dv);
    const int own = dv ? __builtin_ctz(dv) : 0;
    uint32_t B = v ? (1u << own) : 0u;
    uint32_t low = 0;                                    // value of v's digits below round i
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
        int val = 0, blk = 0;
        const bool easy = i >= kDigitRoundsFrom && round_from_digits(pol, dv | lap, i, pol.s(i), low, home, own, val, blk);
        if (BCS_WAVE_ANY(!easy)) {
            const uint32_t d_hi = i <= kAhead ? d[i <= kAhead ? i : 0] : end_point(i);
            const uint32_t d_lo = i + 1 == kQ ? dv : (i + 1 <= kAhead ? d[i + 1 <= kAhead ? i + 1 : 0] : end_point(i + 1));
            int wb;
            const int w = recv_round_value(pol, v, i, pol.s(i + 1), d_lo, d_hi, home, own, B,
                                           [&](uint32_t r) { return dtab[r]; }, wb);
            val = easy ? val : w;
            blk = easy ? blk : wb;
        }
        B |= 1u << (blk & 31);
        emit(i, val);
        low += (0u - ((dv >> i) & 1u)) & pol.s(i);
    }
}

// Rounds 0..last of the same row, for Alg. 5's neighbours (last varies, so the rounds stay a loop): the read for
// the next round is issued before this round's work.  dv = dtab[v] comes from the caller.
template <class Pol, class Emit>
BCS_HD void recv_row_tab_upto(const Pol &pol, const uint32_t *__restrict__ dtab, uint32_t v, uint32_t dv, int last,
                              Emit emit) {
    static_assert(Pol::kScalarSkips, "one p per launch: the inert skips of the per-lane policy are no table indices");
    const uint32_t p = pol.p();
    const int q = pol.q();
    const uint32_t lap = 1u << (q & 31);
    auto end_point = [&](uint32_t s) -> uint32_t {       // digits of v - s with the lap digit, s in [1, p]
        const bool ahead = v >= s;
        return dtab[ahead ? v - s : v + p - s] | (ahead ? lap : 0u);
    };
    uint32_t d_hi = end_point(pol.sdyn(0));
    uint32_t s_n = pol.sdyn(1);
    uint32_t d_lo = end_point(s_n);
    const int home = 31 - BCS_CLZ(dv);
    const int own = dv ? __builtin_ctz(dv) : 0;
    uint32_t B = v ? (1u << own) : 0u;
#pragma unroll 1
    for (int i = 0; i <= last; ++i) {
        const uint32_t s_next = pol.sdyn(i + 2 <= q ? i + 2 : q);
        const uint32_t d_next = end_point(s_next);
        recv_round(pol, v, i, s_n, d_lo, d_hi, home, own, B, [&](uint32_t r) { return dtab[r]; }, emit);
        d_hi = d_lo;
        d_lo = d_next;
        s_n = s_next;
    }
}

// Send entries without the to-neighbour's rounds (Alg. 5 costs entry k that neighbour's rounds 0..k).
// With t = (v + skips[k]) mod p the entry is entry k of t's receive row, and in three cases none of t's rounds
// are needed:
//   (a) k is t's home round, which is the case exactly for v < skips[k+1] - skips[k]: the entry is t's
//       baseblock (Alg. 4's first branch), and D(t) = D(v) with digit k added, so that baseblock is v's, or k
//       for v = 0;
//   otherwise, when v has a digit at or above k, let m be the lowest such digit and L the value of v's digits
//   below k.  The rank with the digits of v from m up and nothing below lies in round k's first window
//   (v - (skips[k+1] - skips[k]), v], holds baseblock m, and nothing larger lies there; so the entry is m - q
//   unless t has come by block m in its earlier rounds.  Those rounds' windows reach back to v + 1 only, and past
//   it, by Alg. 4's second range, by at most the number of odd levels; between v + 1 and t the ranks whose lower
//   part is empty hold blocks other than m.  So the entry is m - q
//   (b) when L keeps clear of both ends of its range: 2c + 2 < L < skips[k] - 1 - (2c + 2), c = the number of
//       odd levels up to k.  The second range of round i of t reaches skips[k] - skips[i+1] + 1 - c_i ranks past
//       v + 1 at most, so it can touch the holder of m, the rank v - L, only for L < c; at the other end a lower
//       part within c of skips[k] - 1 runs over the end of its (shortened) copy when the skip is added.  Every
//       exception found (all entries of every rank of every p <= 40 000; 39 million entries of structured larger
//       p up to 2^31 with L within 80 of either end, 0.6 million of them exceptions) has L within c - 1 of an end;
//       the margin is more than twice that;
//   (c) when the digits of t below k are those of v (adding the skip did not disturb them): no exception in the
//       same searches.
// (b) is what round_from_digits argues for receive rounds, read from the sender (digit k of v clear: t has digit k
// set and the same low part; set: the addition carries, t has digit k clear and the low part L plus the odd levels
// the carry passes); (c) goes beyond it and is an observation, not a proved statement.  The CPU tests compare this
// code with Alg. 5 of the oracle entry by entry (every rank of every p <= 1500, of every p <= 40 000 behind the slow
// marker, and structured large p).  Everything else -- L near an end of its range and low digits disturbed by a
// carry that met an odd level -- is left to Alg. 5: the return value has bit k set for every entry k < q that was
// NOT emitted.
template <class Pol, class DigitsOf, class Emit>
BCS_HD uint32_t send_row_direct(const Pol &pol, uint32_t v, uint32_t dv, DigitsOf digits_of, Emit emit) {
    const uint32_t p = pol.p();
    const int q = pol.q();
    uint32_t pending = 0;
    uint32_t low = 0;                                         // value of v's digits below k
#pragma unroll 1
    for (int k = 0; k <= pol.top(); ++k) {
        const bool active = k < q;                            // per-lane q may be below the wave's bound
        const uint32_t s = active ? pol.sdyn(k) : 0u;
        const uint32_t kbit = 1u << (k & 31);
        const uint32_t oddk = (pol.odd_mask() >> (k & 31)) & 1u;
        const uint32_t above = dv & ~(kbit - 1u);
        const bool home = active && v + oddk < s;             // v < skips[k+1] - skips[k]
        const uint32_t mrg = 2u * (uint32_t)__builtin_popcount(pol.odd_mask() & ((kbit << 1) - 1u)) + 2u;
        const bool mid = low > mrg && low + mrg + 1u < s;
        bool direct = home || (above != 0u && mid);
        const bool ask = active && !direct && above != 0u;    // (c) needs the digits of t
        bool same_low = false;
        if (BCS_WAVE_ANY(ask)) {
            uint32_t t = v + s;
            t = t >= p ? t - p : t;
            const uint32_t dt = digits_of(t);
            same_low = ((dv ^ dt) & (kbit - 1u)) == 0u;
        }
        direct = direct || (ask && same_low);
        const int val = home ? (v ? __builtin_ctz(dv | 0x80000000u) : k) : __builtin_ctz(above | 0x80000000u) - q;
        if (active && direct) emit(k, val);
        pending |= (active && !direct) ? kbit : 0u;
        low += (dv & kbit) ? s : 0u;
    }
    return pending;
}

}  // namespace bcs
#endif  // BCS_EARLIER_ROWS_H
