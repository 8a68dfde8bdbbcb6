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
    int pair, rank;
};

// The walk of one of pairs x n workgroups. (Every workgroup has one: a check for empty
// ones before the rest of the arguments are read would cost a short kernel their round
// trip a second time, 0.5 of 13.7 us in a small backward.)
constexpr Place place_workgroup(int order, unsigned block, unsigned pairs, unsigned n) {
    if (order == kRanked) return {(int)(block % pairs), (int)(block / pairs)};
    const unsigned xcd = block % kXcds, i = block / kXcds;
    if (order == kOwned) {
        const unsigned own = pairs / kXcds;
        return {(int)(xcd * own + i % own), (int)(i / own)};
    }
    const unsigned total = pairs * n, over = total % kXcds;  // the first `over` XCDs have one more
    const unsigned at = xcd * (total / kXcds) + (xcd < over ? xcd : over) + i;
    return {(int)(at / n), (int)(at % n)};
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

// ------------------------------------------------------------------ forward: workgroup shape
//
// A unit is one wave's rows: 32 query rows of one head. With four units per workgroup
// and one wave per unit, a call of few units leaves CUs idle and gives a busy CU's SIMDs
// one wave each, which exposes the tile's dependent score -> softmax -> value chain (0.9
// us per 64-key tile against 0.35 with three waves per SIMD). Key groups split that
// walk; fewer waves per tile spread the units over more CUs, at the price of more tile
// copies and, where the workgroups no longer fit the CUs at once, of a second round.
struct PrefillForm {
    int waves, groups;  // waves that share a tile, key groups of them that walk the tiles in turn
};

// Walks of about the same length for every row: no mask, or a prefix at least as long as
// the rows are many.
constexpr bool even_walks(const AttnSizes& s) { return !s.causal || s.Sk - s.Sq >= s.Sq; }
// Workgroups of GW units a key group (rows and heads past the end included).
constexpr long row_workgroups(const AttnSizes& s, int GW) {
    const int heads = heads_per_group(s.G, GW), rows = 32 * (GW / heads);
    return (long)s.B * s.Hkv * (s.G / heads) * (((long)s.Sq + rows - 1) / rows);
}
// Workgroups of KW blocks of 32 keys.
constexpr long key_workgroups(const AttnSizes& s, int KW) {
    return (long)s.B * s.Hkv * (((long)s.Sk + 32 * KW - 1) / (32 * KW));
}
// Whether one launch takes them (threads in 32 bits).
constexpr bool launchable(long workgroups, int waves) { return workgroups * 64 * waves <= 0xffffffffL; }
// LDS of one key group's two K and V tiles, and the most key groups in one CU's LDS (up to 4).
constexpr int prefill_tile_lds(int r, int dv) { return 2 * 64 * (r + dv) * 2; }
constexpr int prefill_most_groups(int r, int dv) {
    return 160 * 1024 / prefill_tile_lds(r, dv) < 4 ? 160 * 1024 / prefill_tile_lds(r, dv) : 4;
}

//   up to 256 units    one unit per workgroup, as many key groups as the LDS holds
//   up to 512          two units, as many key groups, in at most 256 workgroups (one a CU)
//   up to 1280         two units x 2 where two workgroups share a CU's LDS
//                      (r + d_v <= 160); else, and up to 1024 units in 256 workgroups
//                      where every row walks about the same number of keys (no causal
//                      ramp to balance) over wide values, so that sharing the tiles
//                      counts, four units x 2
//   up to 1536         two units x 2 for d_v 64, three workgroups per CU (r 64: two)
//   up to 2048         as up to 1280 for long walks on a causal ramp (20 tiles or more)
//   beyond             four units, one key group
// A walk of one tile has nothing to split, and one of two or three tiles is split in two
// at most. Where splitting leaves no room on the CUs at once (two units x 2: two a CU at r
// + d_v 128 and 160, three below), the walk has to be a ramp of 8 tiles or more; at r +
// d_v 160 one of under 4 tiles is split in up to 256 workgroups; and equal walks of under
// 6 tiles that already fit the CUs whole stay whole. Measured, us per call, four units x 1 against the
// adopted shape (r 32, d_v 128 unless stated; 32 query heads over 8 KV heads):
//   128 queries over 8192 keys     111.6 / 44.3      500 over 7700     103.4 / 52.6
//   1000 over 8000                 107.5 / 90.1      1100 causal        21.0 / 15.4
//   2048 causal                     36.9 / 35.4      r 128, 500 over 7700  145.4 / 91.7
//   12 heads, r 32, d_v 64: 2 x 500 causal 9.6 / 7.0; 4096 causal 48.9 / 32.9
// and, on the other side of the lines, the shape not taken second: 2 x 1024 causal 22.2 /
// 23.4 with two units x 2, 2000 over 8000 158 / 170, 4 x 512 causal 15.1 / 17.2; 8 x 1000
// causal, 12 heads, d_v 64, 21.2 / 21.7 (r 64: 23.9 / 28.7). Short walks: 5 x 207 causal
// 8.8 / 12.0, 5 x 265 9.3 / 11.9, 28 heads over 4, 15 x 71 8.2 / 11.5 (two units x 2); 9 x
// 178, r 16, 32 heads over 4 of d_v 64, 3 tiles 7.7 / 8.8; 32 heads, r 64, 5 x 94 6.8 / 8.8
// (320 workgroups of two units x 3); 32 over 4 of d_v 64, r 64, 9 x 158 8.2 / 10.4; equal
// walks in 392 workgroups: 28 over 4, 7 x 131 over 508 16.2 / 20.0 (four units x 2).
constexpr PrefillForm prefill_form(const AttnSizes& s) {
    const int most = prefill_most_groups(s.r, s.dv);
    const bool pair = 4 * prefill_tile_lds(s.r, s.dv) <= 160 * 1024;  // two workgroups of two key groups share a CU
    const long units = (long)s.B * s.Hkv * s.G * (((long)s.Sq + 31) / 32);
    const long tiles = ((long)s.Sk + 63) / 64, two = row_workgroups(s, 2), four = row_workgroups(s, 4);
    const bool even = even_walks(s);
    if (tiles < 2) return {4, 1};
    if (units <= 512 && tiles < 4 && two <= 256) return {2, 2};
    if (units <= 256) return {1, most};
    if (units <= 512 && tiles >= 4 && two <= 256) return {2, most};
    if (pair && s.dv == 64) {
        const bool resident = two <= (s.r < 64 ? 768 : 512) || (!even && tiles >= 8);
        return units <= 1536 && resident && !(even && two > 256 && four <= 256 && tiles < 6) ? PrefillForm{2, 2}
                                                                                            : PrefillForm{4, 1};
    }
    if (!even && (units <= 1280 || (units <= 2048 && tiles >= 20))) {
        if (pair && two <= (tiles >= 8 ? 2048 : tiles >= 4 ? 512 : 256)) return {2, 2};
        if (!pair && tiles >= 8) return {4, 2};
    }
    if (even && tiles >= 8 && units <= 1024 && four <= 256) return {4, 2};
    return {4, 1};
}

// ------------------------------------------------------------------ backward: workgroup shapes
//
// A unit is one wave's block of 32 query rows of one head (dQ) or of 32 keys of one KV
// head (dK/dV). As in the forward, a call of few units leaves CUs idle, or all its
// workgroups resident at once so that the longest walk sets its time: fewer units per
// workgroup and several groups that walk the tiles in turn shorten it, as long as the
// CUs still hold the workgroups at once (two units x 2: three a CU at r + d_v 96, two
// at 128 and 160, one above, where two groups' tiles fill the LDS). Past that a long
// causal ramp still gains, because its longest walks bound the call; equal walks and
// short ones lose. us per call, four units x 1 group against the adopted shape (r 32,
// 32 query heads over 8, d_v 128, unless stated):
//   512 tokens 14.9 / 10.8, 1024 tokens 24.9 / 18.2; r 128, 1024 tokens 39.0 / 30.8; 12
//   heads, d_v 64, 2 x 2048 tokens 36.5 / 24.7; four units x 2, 2048 tokens 48.4 / 40.4
// and on the other side of the lines, the shape not taken second: 3 x 500 tokens, 32 KV
// heads, 16.4 / 19.2; r 64, 28 over 4, 5 x 104 8.6 / 12.6 (280 workgroups of two units);
// 11 x 47 over 65 6.9 / 8.1; 7 x 125 7.9 / 9.3; r 64, 10 x 86 over 447 16.3 / 23.6;
// 2 x 2684 without a mask, 8 heads over 2, 68.1 / 75.9 (four units x 2, which without a
// ramp pays at r + d_v 96 in up to 512 workgroups: 12 heads, 5129 tokens 6 % of the whole).
struct DqForm {
    int waves, groups;
};
constexpr DqForm dq_form(const AttnSizes& s) {
    const int wide = s.r + s.dv;
    const long units = (long)s.B * s.Hkv * s.G * (((long)s.Sq + 31) / 32);
    const long tiles = ((long)s.Sk + 63) / 64, two = row_workgroups(s, 2), four = row_workgroups(s, 4);
    const bool even = even_walks(s);
    if (tiles < 2) return {4, 1};
    if (two <= (wide <= 96 ? 768 : wide <= 128 ? 512 : 256)) return {2, 2};
    if (wide <= 128 ? !even && tiles >= 8 && units <= 1536
                    : tiles >= (wide >= 192 ? 10 : even ? 8 : 6) && units <= 1024 && two <= 512 && (wide < 192 || !even))
        return {2, 2};
    if (wide >= 192 && even && tiles >= 12 && four <= 256) return {4, 2};
    if (tiles >= 20 && (even ? wide <= 96 && four <= 512 : units <= 2048)) return {4, 2};
    return {4, 1};
}

// dK/dV: KW waves of 32 keys share each query tile of `rows` rows, `groups` query groups
// of them. us per call, four units x 1 against the adopted shape:
//   r + d_v < 192 (two waves per SIMD), d_v 128: two units x 4 on 32-row tiles, one
//     workgroup per CU, 1024 tokens 129 / 54, 2048 tokens 253 / 100; up to 512 of them on
//     a ramp of 16 tiles, 9 x 1513 over 1713, 8 heads over 2, 194 / 107. Else two
//     units x 2, 32-row tiles (two per CU), up to 3072 units: 2 x 4096 tokens 520 / 394,
//     10 x 952 142 / 122, 32 KV heads, 4 x 153 11.9 / 11.5 (x 4: 18.2). Without a ramp
//     only where they are no second round or save one of the whole shape's: 3 x 1428 over
//     1742 235 / 229; 7 x 877, 64 over 8, 286 / 326 with them, 13 x 104, 32 KV heads, 13.9 / 17.9
//   d_v 64: x 4 in one workgroup per CU for walks of 16 tiles or more (on a ramp of 24
//     up to 768 units); else two units x 2, 64-row tiles, three per CU: 12 heads, 4096
//     tokens 92.8 / 57.8, 8 x 1000 tokens 37 / 40; 9 x 267 without a mask, 16 heads, 14.7
//     / 17.5, 15 x 99 over 166 17.8 / 20.1 (whole backward)
//   r + d_v >= 192 (one wave per SIMD): two units x 2, 64-row tiles, one workgroup per
//     CU: r 128, 2048 tokens 339 / 192; 13 x 157, r 128, 39.2 / 48.2 (312 workgroups); up
//     to 1024 units on a ramp of 8 tiles: 2 x 1122, r 64, 170 / 95, 32 KV heads, 512
//     over 518 53 / 42 (whole backward); r 128, 2048 tokens 104 / 123
struct DkdvForm {
    int waves, groups, rows;
};
constexpr DkdvForm dkdv_form(const AttnSizes& s) {
    const int wide = s.r + s.dv;
    const long units = key_workgroups(s, 1), two = key_workgroups(s, 2), four = key_workgroups(s, 4);
    const long walk = ((long)s.Sq + 63) / 64 * s.G;  // 64-row query tiles of the longest walk
    const bool even = even_walks(s);
    if (walk < 2) return {4, 1, 64};
    if (wide >= 192) {
        if (two <= 256 || (!even && walk >= 8 && units <= 1024)) return {2, 2, 64};
    } else if (s.dv == 64) {
        if ((two <= 256 && walk >= 16) || (!even && walk >= 24 && units <= 768)) return {2, 4, 32};
        if (two <= (walk < 8 ? 512 : 768)) return {2, 2, 64};
    } else {
        if (two <= 256 || (!even && walk >= 16 && two <= 512)) return {2, 4, 32};
        if (even ? two <= 736 || (four > 512 && two <= 1536) : units <= 3072) return {2, 2, 32};
    }
    return {4, 1, 64};
}

// ------------------------------------------------------------------ projection: tile ladder
//
// Tile shape of a call of M tokens x N columns over K = d_model: the smallest of a ladder
// of tiles (columns x tokens) with which every CU gets at most one workgroup. A
// workgroup's time grows with its columns plus tokens (both are read over all of
// d_model), so small tiles win as long as CUs are free to take more of them, and a
// second workgroup on some CUs costs more than the next larger tile on all. Up to 32 x 64
// the waves split d_model each for itself (project_split_kernel), from 64 x 64 to 128 x
// 128 in groups that share a tile's rows (project_kernel with KG > 1); the larger ones
// take d_model whole. Measured, us per call (weights from HBM), with the shapes of one
// group only (16 x 16 ... 64 x 64 by single waves, 128 x 128 up to 256 workgroups of the
// next) / with this ladder:
//   d_model 4096: 200 x 2048 columns 18.5 / 16.5, 600 x 1024 21.5 / 16.4, 1043 x 1024
//     35.1 / 23.5, 600 x 2048 42.2 / 23.8, 4500 x 256 33.7 / 22.7, 2202 x 1024
//     41.5 / 34.6, 9810 x 1024 118 / 97, 3000 x 4096 138 / 105
//   d_model 768: 1043 x 768 6.5 / 5.8, 2202 x 768 9.8 / 7.5, 6500 x 768 16.9 / 15.2
// Where a line lies:
//   * 32 x 64 / 64 x 64: at d_model 4096 they cross between 120 and 200 tiles of the
//     former, by tokens and columns (637 x 384, 120 tiles 15.2 / 15.0; 1177 x 228, 152
//     14.5 / 14.7; 418 x 768, 168 16.6 / 15.8; 158 x 2048, 192 17.8 / 19.4; 1706 x 256,
//     216 16.9 / 15.1), at 2048 by 256 (94 x 4096 13.3 / 12.4), at 8192 by 192 (332 x 1024
//     30.3 / 30.4), at 1024 and 1536 between 192 and 256 (255 x 2048 from 1536, 256 tiles
//     9.6 / 8.9; 196 x 2048 from 1024 7.4 / 7.2), and at 768 past 256 (2035 x 256 5.9 / 6.2)
//   * 64 x 128 / 128 x 64 (half the groups, twice the waves to a group): d_model 4096,
//     1500 x 1024 23.3 / 27.4; 3072, 1500 x 768 19.7 / 21.9; 2048, 1500 x 1024 14.8 / 15.9;
//     1536, 2202 x 768 11.7 / 10.8; 768, 2202 x 768 8.6 / 7.4
//   * past 256 tiles of 128 x 128: these without groups, two workgroups a CU, while 256 x
//     128 would leave CUs idle and the weights are over 8 MiB, so that their stream from
//     HBM needs the second workgroup to hide behind: d_model 4096, 1400 x 3072 (25 MB) 67.6
//     / 80.8 with 256 x 128, 3004 x 2048 (17 MB) 70.5 / 80.9; 2048, 1816 x 3072 (13 MB) 40.0
//     / 42.7; 4096, 6276 x 1024 (8.4 MB) 70.5 / 64.2, 12534 x 512 72.5 / 62.8
//   * just past 256 tiles of 256 x 256 their last ones run alone, and 256 x 128 are
//     faster: 22000 x 768 from d_model 768 54.3 / 47.2, 9810 x 2048 from 2048 110 / 102,
//     4500 x 4096 from 4096 200 / 193 (288 tiles); at 416 tiles 206 / 258
enum class ProjShape : int {
    k16x16, k16x32, k32x32, k32x64, k64x64, k64x128, k128x64, k128x128, k128x128whole, k256x128, k256x256
};

struct ProjTileSize {
    int columns, tokens;
};
constexpr ProjTileSize project_tile(ProjShape s) {
    switch (s) {
        case ProjShape::k16x16: return {16, 16};
        case ProjShape::k16x32: return {16, 32};
        case ProjShape::k32x32: return {32, 32};
        case ProjShape::k32x64: return {32, 64};
        case ProjShape::k64x64: return {64, 64};
        case ProjShape::k64x128: return {64, 128};
        case ProjShape::k128x64: return {128, 64};
        case ProjShape::k128x128:
        case ProjShape::k128x128whole: return {128, 128};
        case ProjShape::k256x128: return {256, 128};
        case ProjShape::k256x256: break;
    }
    return {256, 256};
}
constexpr long project_tiles_of(long M, long N, ProjShape s) {
    const ProjTileSize t = project_tile(s);
    return ((M + t.tokens - 1) / t.tokens) * ((N + t.columns - 1) / t.columns);
}

constexpr ProjShape project_shape(long M, long N, long K) {
    const auto tiles = [=](ProjShape s) { return project_tiles_of(M, N, s); };
    if (tiles(ProjShape::k16x16) <= 256) return ProjShape::k16x16;
    if (tiles(ProjShape::k16x32) <= 256) return ProjShape::k16x32;
    if (tiles(ProjShape::k32x32) <= 256) return ProjShape::k32x32;
    if (tiles(ProjShape::k32x64) <= (K < 1024 ? 256 : K < 2048 ? 192 : 160)) return ProjShape::k32x64;
    if (tiles(ProjShape::k64x64) <= 256) return ProjShape::k64x64;
    if (K < 2048 && tiles(ProjShape::k128x64) <= 256) return ProjShape::k128x64;
    if (tiles(ProjShape::k64x128) <= 256) return ProjShape::k64x128;
    if (tiles(ProjShape::k128x128) <= 256) return ProjShape::k128x128;
    if (tiles(ProjShape::k256x128) < 256 && N * K * 2 > (8L << 20)) return ProjShape::k128x128whole;
    if (tiles(ProjShape::k256x128) <= 256) return ProjShape::k256x128;
    const long large = tiles(ProjShape::k256x256);
    return large > 256 && large <= 320 ? ProjShape::k256x128 : ProjShape::k256x256;
}
constexpr long project_tiles(long M, long N, long K) { return project_tiles_of(M, N, project_shape(M, N, K)); }

}  // namespace tk
