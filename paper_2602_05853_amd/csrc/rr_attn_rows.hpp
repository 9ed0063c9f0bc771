// Rules of the attention launches in plain C++ (HIP compiles constexpr functions for host and device), so that they can be checked
// without a GPU: which row a workgroup of a launch without a row order takes where every XCD has KV groups of its own, and how
// decode-sized steps are shared out.
#pragma once

namespace rr {

// The order of a dense call's rows, for NG KV groups of L keys, the Lq / 128 last query blocks and `rows` rows in all.
enum DenseOrder {
    kSetsOfGroups = 0,  // over all XCDs
    kGroupByGroup = 1,  // XCDs have KV groups of their own and take one after the other
    kRankByRank = 2     // ... and take the heaviest row of each, then the second, ..
};
// Groups of their own: where the groups divide into the XCDs or the XCDs into the groups.  The rows of a chunk all walk
// nearly the whole context, so the keys and values of the groups in flight, one to an XCD, must fit the memory-side cache
// of 256 MB; those of a prompt are half as long in the mean.
// Sets of groups over all XCDs / this, us:
//   chunks: 4096 of 65536, 32 / 8 heads (256 MB) 3698 / 3668, 8192 7193 / 7092, two sequences of 45000 (175) 3185 / 3111,
//     4096 of 131072, 28 / 4 (256) 7358 / 7227; not taken: 2048 of 80000, 64 / 8 (312) 4565 / 4732, 8192 of 80000, 32 / 8
//     8826 / 8956, 4096 of 131072 (512) 7452 / 7655, 16384 28547 / 28969, 64 / 8 14937 / 15372, 1024 of 400000, 32 / 2
//     (390) 5719 / 5820
//   whole prompts: 65536, two of 32 / 8 (256) 60563 / 59704, 80000 (312) level, 98304 (384) 67351 / 67105, 131072 (512)
//     119887 / 119418, 16 / 8 61205 / 59332
// Several groups to an XCD: one after the other their tiles stay in its L2 longer, but the last one's heavy rows start
// late.  It pays from ten rows on to each of the 512 workgroups that run at once, and the earlier the less the rows differ:
// by Lq of L blocks, of which one share is how many rows are unlike and one how late they are.  Packed prompts: heavy rows
// in the middle of a group.
// Sets / group by group / rank by rank, us:
//   32 / 32 heads, 1531 tokens (0.8 rows to a workgroup) 37.7 / 42.3 / 37.5, 3195 92.4 / 108.9 / 92.1, 4096
//     159 / 166 / 139, 8192 (4) 560 / 515 / 503, 16379 (8) 2159 / 1960 / 1949, 24059 (11.8) 4231 / 4155 / 4239; 24 / 24,
//     2171 49.5 / 57.3 / 49.1; 32 / 8, four of 379 19.4 / 21.4 / 19.0, of 8192 (16) 2083 / 1975 / 1970, sixteen of 4096
//     (32) 2294 / 2131 / 2218; 24 / 12, eight of 507 33.4 / 38.7 / 33.2, of 10875 (32) 5910 / 5219 / 5916
//   chunks: 2000 of 20000, 32 / 32 (1.1) 811 / 754 / 811, 512 of 12000, sixteen of 32 / 8 (5) 1851 / 1721 / 1866, 1500 of
//     3000, eight of 8 / 8 (1.6) 131 / 144 / 131
//   packed: 32 / 32, forty of 8 blocks (20) 568 / 575 / 518, 64 / 16, two of 100 (25) 4899 / 4708 / 4723, 16 / 16, 6, 24, 1
//     and 2 59.9 / 61.4 / 60.4
constexpr DenseOrder dense_order(int NG, int L, int d, int Lq, bool packed, long long rows) {
    const long long in_flight = (NG < 8 ? NG : 8) * 4ll * L * d;
    const bool own = ((NG & 7) == 0 || 8 % NG == 0) && (Lq == L || in_flight <= 256ll << 20);
    if (!own || NG <= 8) return own ? kGroupByGroup : kSetsOfGroups;
    const double differ = (double)Lq / L;
    return !packed && rows >= 512 && rows >= 5120.0 * differ * differ ? kGroupByGroup : kRankByRank;
}

struct RowPlace {
    int grp;            // KV group, batch * Hkv of them
    int hl;             // query head inside the group
    int mr;             // query block, counted from the heaviest; from Nb on: no row
};

// NG a multiple of eight: XCD x (workgroup mod 8) takes the groups x, x + 8, .., rows by descending weight, the heads of a query
// block together; one group after the other, or all of them rank by rank.
constexpr RowPlace row_of_whole_groups(int bid, int G, int Nb) {
    const int x = bid & 7, s = bid >> 3, per = Nb * G, r = s % per;
    return {x + 8 * (s / per), r % G, r / G};
}
constexpr RowPlace row_of_groups_by_rank(int bid, int NG, int G) {
    const int x = bid & 7, s = bid >> 3, per = (NG >> 3) * G, r = s % per;
    return {x + 8 * (r / G), r % G, s / per};
}

// NG a divisor of eight: k = 8 / NG XCDs share a group, and each takes one of every k query blocks (a level) for all heads,
// whose tiles then meet in its L2.  Levels are taken forth and back: with the same place in every level the heaviest of k
// rows always went to one XCD, which had 21 % more key blocks than the mean for one KV head and 32 query blocks.  Of less
// than two whole levels the place moves on from head to head instead, so that no XCD is left without rows.
// Dense, us, sets of groups over all XCDs / the same place in every level / this:
//   32 / 1 heads: 2048 tokens 51.5 / 55.8 / 45.7, 3500 124 / 124 / 113, 4096 151.8 / 169.5 / 143.0, 8192 521 / 553 / 516,
//     20000 2920 / 2921 / 2840
//   64 / 1: 1500 70.2 / 70.0 / 58.6, 4096 288.7 / 317.7 / 276.3; 128 / 1, 4096 566 / 621 / 549; 8 / 1, 9000
//     186 / 186 / 177, 16384 529 / 538 / 517
//   32 / 2: 4096 152.1 / 155.3 / 142.8, 8192 519 / 531 / 509; 64 / 2, 2300 113 / 113 / 99; 28 / 4: 8192 453 / 455 / 445,
//     10000 660 / 660 / 651, 16384 1715 / 1706 / 1690
//   chunks: 1500 of 60000, 16 / 1, 854 / 855 / 710, 3000 of 20000 481 / 481 / 471, 4096 of 100000 level for 1, 2 and 4 KV
//     heads
//   lists without an order, 4900 tokens (blocks no multiple of eight), same place / this: 32 / 1 131 / 127, 32 / 2
//     109 / 104; 9999, 16 / 1, 204 / 194; 20300, 28 / 4, 885 / 889
// (The place that moves on from head to head in all levels: 32 / 1, 2048 tokens 51.1, 4096 154.5, 20000 2990, 28 / 4, 16384
// 1742; only in a last level without a partner or that k does not fill: 32 / 1, 3500 124, 64 / 2, 2300 106, 4096 of 100000,
// 16 / 1, 4029 instead of 3854.)
// Packed prompts: a row's weight jumps where a prompt starts, and the XCDs on the heavy side of that level would have it
// for all heads; the second half of the heads is therefore taken k / 2 places on.  Packed dense calls, us, sets of groups
// over all XCDs / the same place in every level / forth and back / and halves:
//   32 / 1: four prompts of 50 blocks 1252 / 1215 / 1349 / 1271, of 101 and 37 1394 / 1393 / 1475 / 1394, forty of 8
//     517 / 638 / 501 / 478; 8 / 1: 65 and 28 179 / 180 / 191 / 184; 16 / 2: forty of 8 267 / 271 / 248 / 244; 28 / 4: 12,
//     80 and 33 825 / 826 / 836 / 821; 75 packings of 1, 2 and 4 KV heads: 1 / 1.000 / 0.986 / 0.980 in the geometric mean,
//     at worst 1.21 / 1.08 / 1.04 (8 / 1, seventeen of 13 blocks, 1768 rows)
// (Halves without forth and back 0.985, quarters 0.982, eighths 0.982; single prompts with halves, 32 / 1, 4096 135 instead
// of 131, 8 / 1, 8192 135 instead of 131.)
constexpr RowPlace row_of_shared_group(int bid, int NG, int G, int Nb, bool packed) {
    const int k = 8 / NG, x = bid & 7, s = bid >> 3, q = s / G, c = x / NG;
    const int hl = s - q * G, beyond = packed && 2 * hl >= G ? k / 2 : 0;
    const int at = Nb < 2 * k ? (c + s) % k : ((q & 1 ? k - 1 - c : c) + beyond) % k;
    return {x % NG, hl, q * k + at};
}

// Whether a sparse launch draws its rows by KV group (queue q of min(NG, 8): the groups q, q + 8, ..): `resident`
// workgroups at once; interleave: the groups to a set in the other order, rank by rank over all XCDs.
// At least eight rows to a workgroup, four where every queue has the same number of several groups or where the other order
// has sets of two groups at most (below that the queues' different lengths cost what the L2 hits give), and as long as the
// keys and values of the groups in flight, one to a queue, fit the memory-side cache of 256 MB.  Estimate and attention,
// gain of the inputs 3, tau 0.9, us, rows in rank order over all XCDs / by group:
//   32 / 8 heads: 16384 tokens 708 / 681, 24000 1518 / 1430, 31907 3142 / 3034, 40000 4068 / 3864, 50000, weaker structure,
//     8088 / 7776; 64 / 8: 9000 533 / 521, 20000 2124 / 2040, 60000 17788 / 17407; 28 / 4: 20000 911 / 902, 32000
//     2247 / 2176, 50000 5442 / 5221; 16 / 4: 60000 4537 / 4312, 90000 10911 / 10725; 8 / 2: 40000 1087 / 1068
//   batches: 32 / 8, four of 2000 162 / 152, sixteen 585 / 554, three of 12000 1360 / 1260, two of 45000 10346 / 9835;
//     28 / 4, eight of 3000 357 / 342; packed prompts of 311 blocks, 28 / 4, 1452 / 1382, forty of 6 blocks, 32 / 8,
//     403 / 373
//   queues of different numbers of groups: nine KV heads, 9 / 9, 30000 (8.3) 657 / 613, 36 / 9, 10000 (5.5, not taken)
//     309 / 318, 16000 (8.8) 689 / 660; ten, 40 / 10, 14000 (8.6) 625 / 611; eleven, 22 / 11, 13000 (4.4) 454 / 404 and
//     329 / 333; seventeen, 68 / 17, 4100 (4.4) 226 / 180; not taken: 36 / 9, 8000 (4.4) 223 / 246, 40 / 10, 7000 (4.3)
//     199 / 223, 36 / 18, 8000 (4.4) 227 / 240
//   not taken: 32 / 8, 2500 (1.3 rows to a workgroup) 76 / 82, 6500 (3.2) 172 / 180, 8192 (4) level, 12000 (5.9) level;
//     28 / 4, 8000 (3.4) 217 / 229; 16 / 4, 16384 (4) 411 / 428; 64 / 8, 65536 21131 / 21141; 32 / 8, 98304 25889 / 25944,
//     131072 31994 / 32199
constexpr bool rows_by_group(long long rows, int resident, int NG, int interleave, int L, int d) {
    const bool four = NG > 8 && (NG % 8 == 0 || interleave <= 2);
    return rows >= (four ? 4ll : 8ll) * resident && (NG < 8 ? NG : 8) * 4ll * L * d < 256ll << 20;
}
// Rows of each group's order that a queue of several groups takes rank by rank, before the others group by group.
// Queues of as many groups each: the heaviest, 16 G of a queue in all (at least G of a group): more of them mix the tiles
// of many groups in L2 for long.  Others: all, since the last group of a longer queue would start late (heaviest
// first / all: 36 / 9, 16000 671 / 631, 30000 1968 / 1891, 24 / 12, 18000 582 / 563).
// Queues of as many, rank order over all XCDs / none first / 8 G of each group / 2 G of each:
//   32 groups to a queue: 32 / 32, eight of 7424 1488 / 1423 / 1557 / 1448, of 12000 3290 / 3039 / 3346 / 3076; 16: 8 / 2,
//     sixty-four of 2000 541 / 498 / 512 / 495, 32 / 32, four of 7424 797 / 783 / 760 / 749; 8: 32 / 8, eight of 3000
//     373 / 373 / 368 / 361, of 8000 1592 / 1537 / 1523 / 1508
//   4: 32 / 8, four of 4096 268 / 273 / 262 / 255, of 9000 979 / 914 / 874 / 861; 2: 16 / 16, 20000 559 / - / 546 / 563,
//     16 / 1, sixteen of 1500 163 / 162 / 162 / 166
constexpr int front_rows_of_groups(int NG, int G, int Nb) {
    const int n = NG / 8 > 2 ? NG / 8 : 2, each = n < 16 ? 16 / n : 1;
    return NG > 8 && NG % 8 ? G * Nb : (each < Nb ? each * G : 0);
}

// Decode-sized steps (rr_attn_decode.hip): how many waves take a part of the context and in how many workgroups, for R query rows
// to a KV head and `parts` parts in all of `len` blocks each.
struct DecodeForm {
    bool eight;         // waves: eight, or four
    bool halves;        // two workgroups to a part, 16 of its rows each
};
// Eight waves, two blocks at a time: fewer parts than compute units, of some length (at 64K, 32 / 8 heads, 8 tokens, 128
// parts 75 -> 56 us; 256 parts 51 and 52).
// Halves, of more than 16 rows: where both fit the compute units at once, one of eight waves to a unit.  Both read the
// part's keys, the second from L2, and use the matrix and vector units of twice as many compute units; sparse, each walks
// the blocks of its own rows only.  32 rows in one workgroup / halves, us:
//   estimate and attention: 8 tokens of 64512, 32 / 8 heads, 90.2 / 84.4, of 30000 51.3 / 47.1, of 4000 (four waves)
//     40.8 / 38.2, of 90000, 8 / 2, 65.6 / 57.7
//   dense: 4 tokens of 131072, 28 / 4 90.4 / 83.8, 64 / 8 193.5 / 181.7, eight sequences of 5000, 28 / 4, 28.1 / 26.1 (31
//     with the two on different XCDs)
//   not taken, more than 128 parts, where halves make a second round of the launch: 8 tokens of 30000, 32 / 8, three
//     sequences (144 parts) 78.0 / 122.4, five, 16 / 4 (140) 63.4 / 99.0; of 16435, 3 / 1, twelve (180) 24.3 / 32.8
// (The values of the next keys requested with these, which one tile of rows has registers for: 86.2 instead of 83.7, one
// token of 128K 97.3 instead of 95.9.)
constexpr DecodeForm decode_form(int R, long long parts, int len) {
    return {parts < 256 && len >= 8, R > 16 && 2 * parts <= 256};
}

}  // namespace rr
