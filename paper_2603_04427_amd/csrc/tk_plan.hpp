// Which form of a kernel a call takes: pure functions of the sizes, without HIP, so
// that a host program can check them too (constexpr functions serve both sides).
#pragma once

namespace tk {

constexpr unsigned kXcds = 8;   // workgroups are dealt to the XCDs round-robin
constexpr unsigned kXcdCus = 32; // CUs of an XCD

constexpr int gcd4(int g) { return (g % 4 == 0) ? 4 : (g % 2 == 0 ? 2 : 1); }

// Heads of a KV group per workgroup: as many of gcd(G, 4) as its GW waves hold.
constexpr int heads_per_group(int G, int GW) { return gcd4(G) < GW ? gcd4(G) : GW; }

// An attention call's sizes, forward or backward.
struct AttnSizes {
    int B, Hkv, G, Sq, Sk, r, dv;
    bool causal;
};

// ------------------------------------------------------------------ order of the workgroups
//
// The workgroups of a prefill kernel are `pairs` walkers (a KV sequence and some of
// its heads) times `n` blocks of rows (or keys), block rank 0 with the longest walk.
enum Order : int {
    kRanked = 0,      // the longest walk of every pair, then the next: round-robin dispatch puts pair i on XCD i % 8
    kOwned = 1,       // each XCD the longest walks of its own eighth of the pairs first (pairs a multiple of 8)
    kBySequence = 2,  // each XCD its share of the pairs one after the other
};

struct Place {
    int pair, rank;  // pair < 0: no work
};

constexpr Place place_workgroup(int order, unsigned block, unsigned pairs, unsigned n) {
    if (order == kRanked) return {(int)(block % pairs), (int)(block / pairs)};
    const unsigned xcd = block % kXcds, i = block / kXcds;
    if (order == kOwned) {
        const unsigned own = pairs / kXcds;
        return {(int)(xcd * own + i % own), (int)(i / own)};
    }
    const unsigned total = pairs * n, at = xcd * ((total + kXcds - 1) / kXcds) + i;
    return at < total ? Place{(int)(at / n), (int)(at % n)} : Place{-1, 0};
}
// Workgroups to launch (by sequence every XCD gets the same number, the last ones empty).
constexpr long order_launch(int order, long workgroups) {
    return order == kBySequence ? (workgroups + kXcds - 1) / kXcds * kXcds : workgroups;
}

// The order of the forward and of the dQ kernel with four heads or row blocks a
// workgroup and one key group. Longest walks first over all sequences lets the
// lightest workgroups start last, which balances the end of a causal call; but every
// sequence that an XCD has in flight streams its K and V through that XCD's L2 at
// once. Where a KV sequence has several head groups, round-robin would also spread
// them over the XCDs, each fetching the sequence anew: there each XCD owns its pairs.
// us per call, by sequence / longest first (two input sets in turn, spread under 1 %
// below 1 ms and 2 % above; r 32, d_v 128 unless stated):
//   * all resident at once: longest first. 12 heads, d_v 64, 1 x 8192 tokens 133 / 96
//   * equal walks (no mask), unless owned: nothing to balance. 32 heads, 8 x 2048 354 / 398,
//     4 x 4096 659 / 689; 32 over 8, 8 x 4096 1299 / 1318, 16 x 1024 192 / 198
//   * over 24 MB of K and V an XCD: 32 heads, 4 x 8192 1369 / 1494, 8 x 2048 (21 MB)
//     231 / 225, 2 x 8192 (21 MB) 701 / 668; r 128, 29 x 1598 (95 MB) 813 / 1186
//   * over 6 MB where the blocks of one sequence fill the XCD twice over, so that only
//     light ones are left at its end: 64 heads over 8, 4 x 8192 2582 / 2664; 32 over 8,
//     8 x 6400 1610 / 1643, 4 x 8192 with inputs from HBM 1294 / 1309 (0.47 against
//     1.57 GB read and written), 2 x 8192 (5.2 MB) 656 / 653, 2 x 4096 190 / 176
//   * several head groups: owned, 64 over 8, 2 x 4096 354 / 346. Pairs that are no
//     multiple of 8 go longest first round-robin while K and V are few (40 over 5, 2 x
//     6000, 2.4 MB an XCD 483 / 456; 28 over 4, 9 x 5381, 7.8 MB 1195 / 1385) and a pair
//     has some blocks to balance (25 x 123 tokens, 40 over 5, r 128 24.6 / 29.8). At r
//     128, whose key rows weigh most, by sequence past four rounds of workgroups (dQ, 64
//     over 8, 29 x 311 190 / 209; 28 over 4, 1 x 2629, 1.2 rounds 100 / 73)
constexpr int walk_order(const AttnSizes& s, int slots_per_cu) {
    const int heads = heads_per_group(s.G, 4), rows = 32 * (4 / heads);
    const long kv_sequences = (long)s.B * s.Hkv, per_kv = s.G / heads, pairs = kv_sequences * per_kv;
    const long n = ((long)s.Sq + rows - 1) / rows, slots = (long)kXcdCus * slots_per_cu;
    const long bytes = kv_sequences * s.Sk * (s.r + s.dv) * 2 / kXcds;  // K and V of an XCD
    const bool wide = s.r + s.dv >= 256;
    if (per_kv > 1 && ((wide && pairs * n > 4 * kXcds * slots) ||
                       (pairs % kXcds != 0 && (n < (wide ? 5 : 4) || bytes > 3000000L))))
        return kBySequence;
    const int longest_first = per_kv > 1 && pairs % kXcds == 0 ? kOwned : kRanked;
    if (pairs * n <= kXcds * slots) return longest_first;
    if ((!s.causal && longest_first != kOwned) || bytes > 24000000L || (n >= 2 * slots && bytes > 6000000L)) return kBySequence;
    return longest_first;
}

// The order of the dK/dV kernel (pairs: KV sequences; n: key blocks of 32 KW keys).
// Longest first over all sequences balances the CUs: with the workgroups of one
// sequence after the other, a CU's two resident workgroups were both of the longest or
// both of the shortest (606 against 522 us at 2 x 4096 tokens, 954 against 723 us at
// 4 x 4096; r 32, d_v 128, 32 query heads over 8). Where the key blocks of one sequence
// fill an XCD by themselves (64 slots) and read the same G heads' tiles, keeping to one
// sequence at a time serves those reads from its L2: 2.84 against 2.95 ms at 4 x 8192.
// With r + d_v of 192 or more (one workgroup per CU, more work per byte) the balance
// counts more (5.50 against 5.73 ms there at r 128), and with G = 1 as well (1.40 against
// 1.42 ms at 2 x 8192, 32 heads). Without a mask every walk is the same (32 heads, 19 x
// 2295 tokens 2.33 against 2.52 ms, 64 over 8, 10 x 2152 2.23 against 2.27 ms).
constexpr int dkdv_order(const AttnSizes& s, int KW) {
    const long nkb = ((long)s.Sk + 32 * KW - 1) / (32 * KW);
    return KW == 4 && (!s.causal || (s.r + s.dv < 192 && s.G >= 4 && nkb >= 64)) ? kBySequence : kRanked;
}

}  // namespace tk
