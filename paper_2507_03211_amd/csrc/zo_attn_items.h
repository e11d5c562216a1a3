// How the causal attention's work items are listed and dealt to workgroups: what the kernel and its launcher share.
//
// Work items: (128 query rows, head, sequence).  The hardware deals consecutive workgroup ids round-robin to the 8 XCDs, so
// workgroup b sits on XCD b % 8 and is that XCD's slot b / 8.  Every (head, sequence) pair goes to one XCD with all its query
// tiles, so the XCDs hold equal shares of the causal triangle and the K and V of a pair are fetched into one L2 instead of eight.
// An XCD's items are listed in groups of pairs, long rows first within a group.  Persistent workgroups: slot j takes entry j of
// the even rounds and entry slots - 1 - j of the odd ones, so that a long tile is followed by a short one.  One workgroup per
// item: the list is one round, and a workgroup that ends makes room for the next entry.
#pragma once
#include <hip/hip_runtime_api.h>

namespace zo {

constexpr int kAttnRows = 128;

struct AttnItems {
    int n_qt, n_pairs, pairs_xcd, group_pairs, group_items, n_lin;      // n_lin: entries of an XCD's list, empty ones among them
    // `fill`: as many of an XCD's items as a group is to have at least, if that is more than one pair
    __host__ __device__ __forceinline__ AttnItems(int seq, int n_heads, int n_seq, int fill)
    {
        n_qt = (seq + kAttnRows - 1) / kAttnRows;
        n_pairs = n_heads * n_seq, pairs_xcd = (n_pairs + 7) / 8;
        group_pairs = fill / n_qt > 1 ? fill / n_qt : 1, group_items = group_pairs * n_qt;
        n_lin = (pairs_xcd + group_pairs - 1) / group_pairs * group_items;
    }
    // the (head, sequence) pair of an entry, -1 if it is empty, and its query tile
    __host__ __device__ __forceinline__ int pair_at(int lin, int xcd, int &qt) const
    {
        if (lin >= n_lin) return -1;
        const int grp = lin / group_items, r = lin % group_items;
        const int gp = pairs_xcd - grp * group_pairs < group_pairs ? pairs_xcd - grp * group_pairs : group_pairs;
        if (r >= gp * n_qt) return -1;
        qt = n_qt - 1 - r / gp;
        const int pair = (grp * group_pairs + r % gp) * 8 + xcd;
        return pair < n_pairs ? pair : -1;
    }
};

// Slots an XCD's workgroups have (persistent: as many as are resident at once), the list's `fill` and workgroups a CU.
struct AttnPlan { int slots, fill, per_cu = 0; };

// When the query tiles of a sequence divide the resident workgroups, rounds of the list are whole groups, the zigzag gives every
// slot the same number of key tiles, and persistent workgroups save an item's start.  When they don't, a group's long tiles come
// to lie at both ends of a round and some slots get two of them: then a workgroup per item, for which the hardware finds the free
// place.  us, persistent / per item, heads of 128 unless said: 1500 tokens (12 tiles, 64 slots) x 64 (sequence, head) pairs
// 67 / 50, x 320 259 / 236; 1100 x 320 172 / 137; 600 x 160 35 / 28; but 1024 x 160 63 / 72.
// From some round on the dynamic order wins there as well: with heads of 64 (up to 5 tiles, three workgroups a CU) from the fourth,
// with larger heads from the fifth up to 4 tiles a sequence, else the seventh.  One and two tiles stay persistent: an
// item's start is most of it.  Persistent time over per item's, whole tiles | a ragged last one:
//   rounds             4           4.5         5           6           7           8           12.5
//   heads of 64,  3 t  1.03 | 1.05 1.03 | 0.98 1.06 | 1.04 1.09 | 1.08 1.08 | 1.08 1.07 | 1.08 1.09 | 1.08
//   heads of 128, 4 t  1.00 | 1.02 0.94 | 0.95 1.01 | 1.06 1.02 | 1.05 1.02 | 1.07 1.01 | 1.08 1.02 | 1.06
//                16 t  0.97 | 0.99 0.93 | 0.94 1.00 | 1.01 1.00 | 1.00 1.02 | 1.04 1.01 | 1.01
//   heads of 80,  8 t  0.98 | 0.99 0.95 | 0.91 1.00 | 0.99 1.00 | 1.01 1.02 | 1.01 1.02 | 1.04 1.01 | 1.02
//
// The list of a workgroup per item: a group keeps few pairs' K and V in the L2, but the last one begins with its longest rows when
// the others are nearly done.  Over few rounds that tail is the longer, and all pairs make one group: the longest rows of all
// come first.  us, persistent / groups / one group: heads of 128, 3328 x 56 (2.8 rounds) 179 / 187 / 166, 3584 x 40 (2.2) 154 / 156 /
// 135.  Up to three rounds from 8 tiles on; shorter sequences leave groups sooner: groups / one group, heads of 128, 640 x 128
// (1.2) 1.01, x 160 (1.6) 0.98, x 224 (2.2) 0.96.  Two whole groups that fill the slots have no such tail, and with large heads
// two groups' K and V are twice the L2: heads of 128, 1792 x 64 62.7 / 66.8, 1408 x 80 52.9 / 54.8, of 112 68.1 / 69.9
// (heads of 80: 63.1 / 61.9, 53.1 / 51.8).
inline AttnPlan attention_plan(long long pairs, int n_qt, int slots_max, int d_head)
{
    const long long pairs_xcd = (pairs + 7) / 8, items = pairs_xcd * n_qt;
    if (items <= slots_max) return {(int)items, (int)items};
    const int rounds = d_head == 64 ? 4 : n_qt <= 4 ? 5 : 7;
    const bool per_item = slots_max % n_qt != 0 || (n_qt >= 3 && items / slots_max >= rounds);
    if (!per_item) return {slots_max, slots_max};
    const long long in_slots = slots_max / n_qt > 1 ? slots_max / n_qt : 1;          // pairs
    const bool even = d_head > 80 && n_qt <= slots_max && pairs_xcd == 2 * in_slots && 7 * in_slots * n_qt >= 6 * slots_max;
    const bool one_group = 2 * items <= (n_qt >= 8 ? 6 : d_head == 64 ? 5 : 3) * (long long)slots_max && !even;
    const long long group = one_group ? pairs_xcd : in_slots;
    return {(int)((pairs_xcd + group - 1) / group * group * n_qt), one_group ? (int)items : slots_max};
}

// Heads of 64 channels and six query tiles or more, where a CU has room for four workgroups (S slots an XCD, F with one workgroup less,
// P pairs of n tiles).  us of 1024 tokens (8 tiles) unless said, F and S slots x persistent / groups / one group:
//   P x n up to S                   all at once: 16 pairs 32.8 / 34.7 / 30.1, 27.5 / 27.6 / 27.6; but where one pair more than F holds
//                                   is all there is, its items fill in behind short ones: 13 pairs 31.6 / 32.7 / 24.6, 25.1 / 25.1 / 25.1
//   two to three rounds of S        n divides S, n <= 8: persistent with S: 40 pairs 70.5 / 70.6 / 69.4, 64.3 / 69.9 / 68.9
//   2.25 to three rounds of F       n divides F, n <= 8: persistent with F: 32 pairs 51.7 / 58.5 / 55.1, 53.7 / 56.8 / 54.2; 6 tiles,
//                                   40 pairs 43.3 / 47.7 / 45.2, 52.0 / 47.6 / 44.9
//   up to 20 pairs past a round     (22 for up to 10 tiles) one group of all pairs with S: 17 pairs 34.2 / 36.9 / 31.7, 39.6 / 39.6 / 30.3;
//                                   16 tiles, 25 pairs 142 / 144 / 132, 147 / 144 / 129; 32 tiles, 14 pairs 281 / 292 / 264, 280 / 280 / 258;
//                                   while the chip's K and V stay in 256 MiB of cache, eight rounds: 64 tiles, 15 pairs 1174 / 1145 / 1143,
//                                   1140 / 1119 / 1105, 19 pairs 1486 / 1439 / 1488, 1451 / 1406 / 1449
//   up to three rounds of S         those are four whole ones of F, in groups: 9 tiles, 40 pairs 98.6 / 79.8 / 84.9, 86.0 / 81.9 / 84.4
//   more                            groups with S: 58 pairs 94.2 / 94.2 / 105, 96.9 / 92.5 / 106; 16 tiles, 30 pairs 169 / 167 / 167, 166 / 159 / 167
// Over 562 sizes (6 - 64 tiles, 0.7 - 11 rounds) 0.2 % behind the best of the six on average, 6 % at the most.
inline AttnPlan attention_plan_64(long long pairs, int n_qt, int cus_xcd)
{
    const int slots = 4 * cus_xcd, fewer = 3 * cus_xcd;
    const long long pairs_xcd = (pairs + 7) / 8, items = pairs_xcd * n_qt;
    auto grouped = [&](int per_cu) {
        const int filled = per_cu * cus_xcd;
        const long long group = filled / n_qt > 1 ? filled / n_qt : 1;
        return AttnPlan{(int)((pairs_xcd + group - 1) / group * group * n_qt), filled, per_cu};
    };
    if (items <= slots) return {(int)items, (int)items, items > fewer && items <= fewer + n_qt ? 3 : 4};
    if (n_qt <= 8 && slots % n_qt == 0 && items > 2 * slots && items <= 3 * slots) return {slots, slots, 4};
    if (n_qt <= 8 && fewer % n_qt == 0 && 4 * items > 9 * fewer && items <= 3 * fewer) return {fewer, fewer, 3};
    if (items <= slots + (n_qt <= 10 ? 22 : 20) * n_qt && items <= 8 * slots) return {(int)items, (int)items, 4};
    return grouped(items <= 3 * slots ? 3 : 4);
}

// How many workgroups share a CU, and the plan.  Heads of 64 channels leave room for four, of 80 for three, larger ones for two.  One
// less is better where the rounds of persistent workgroups come out so, and with heads of 64 for sequences of up to five tiles: those
// take the time that their operands need, and more pairs at a time leave the L2 (3 tiles x 1024 pairs, us, three / four 50.1 / 51.1, 4 x
// 976 77.5 / 80.9, 3 x 2432 105 / 110), unless all items fit at once (2 tiles x 444 18.2 / 15.6).
// Heads of 80: a round of three a CU takes about 1.3 times as long as one of two.  Time with two over time with three, persistent:
// 16 tiles x 128 pairs (4 rounds or 3) 1.05, x 96 (3 or 2) 1.10, 4 x 448 1.07, 3 x 512 1.06, but 6 x 400 (5 or 4) 0.96, 1 x 832 0.96, 4
// x 248 0.95; all items at once, 7 tiles and less 1.02 - 1.20, 10 x 64 0.96 (the longest item's chain is all there is).
// Three a CU: a workgroup per item from the fourth round on (persistent over per item's time, 4 tiles 1.05, 6 tiles, 4 rounds 1.04, 6
// 1.05; 8 and more only from the sixth: 16 tiles, 4 rounds 0.98, 6 1.03), and all pairs in one group, over few rounds, also where the
// tiles divide the slots (over persistent's, 16 tiles, 1.3 rounds 1.06, 2 1.02, 2.7 1.03, 6 tiles, 1.1 1.16, 1.6 0.99, 3.1 0.98).
// Five tiles, groups / one group, us: 29 pairs an XCD (1.5 rounds) 48.5 / 42.1, 36 (1.9) 51.1 / 49.5, 38 (2.0) 52.8 / 54.3.
inline AttnPlan attention_plan_on(long long pairs, int n_qt, int cus_xcd, int d_head)
{
    const int full = d_head == 64 ? 4 : d_head == 80 ? 3 : 2, slots = full * cus_xcd, fewer = slots - cus_xcd;
    const long long pairs_xcd = (pairs + 7) / 8, items = pairs_xcd * n_qt;
    if (d_head == 64 && n_qt >= 6) return attention_plan_64(pairs, n_qt, cus_xcd);
    bool more = full > 2;
    if (d_head == 64) more = items <= slots;
    if (d_head == 80 && items <= slots) more = n_qt < 8;
    else if (d_head == 80 && slots % n_qt == 0 && (n_qt < 6 || items >= 2 * slots))
        more = 13 * ((items + slots - 1) / slots) <= 10 * ((items + fewer - 1) / fewer);
    if (!more) {
        AttnPlan plan = attention_plan(pairs, n_qt, full > 2 ? fewer : slots, d_head);
        plan.per_cu = full > 2 ? full - 1 : full;
        return plan;
    }
    if (items <= slots) return {(int)items, (int)items, full};
    const int rounds = n_qt <= 6 ? 4 : 6;                                             // from here on heads of 80
    const bool few = (n_qt >= 16 && items <= 3 * slots) || (n_qt >= 6 && items < 2 * slots);
    const bool per_item = slots % n_qt != 0 || few || (n_qt >= 3 && items >= rounds * slots);
    if (!per_item) return {slots, slots, full};
    const long long in_slots = slots / n_qt > 1 ? slots / n_qt : 1;
    const bool one_group = few || (n_qt >= 8 ? items <= 3 * slots : 8 * items <= 15 * slots);
    const long long group = one_group ? pairs_xcd : in_slots;
    return {(int)((pairs_xcd + group - 1) / group * group * n_qt), one_group ? (int)items : slots, full};
}

}  // namespace zo
