// Which kernel serves which call: the rules that go by sizes alone.  Plain host code without the HIP runtime, so that a
// test can compile it and ask.
#pragma once
#include <stdint.h>

namespace ie {

// Items (workgroups of 256 threads) of a launch that the hardware deals out: a HIP launch has fewer than 2^32 threads.
// Persistent launches draw up to 2^31 - 1 items from their queues, so a call of more than this goes to them.
constexpr int64_t kDealtItems = ((int64_t)1 << 32) / 256 - 1;

// Backward pass at head dimension 64: a persistent launch for each kind of item (kTwo), one launch that the hardware deals out
// (kDealt, two workgroups per CU) or one with queues (kQueued)?  As at head dimension 128 (below) the shared launch has one
// tail instead of two, and its dQ items run at two waves per SIMD instead of three.  The estimated time of one launch is
// its longest item or the work per resident workgroup, whichever is longer; two launches come to 2.3 times the dK/dV items
// alone.  Before (queued or two) : now: 8192 x 8, 8 per group, bidirectional 1791 : 1144 us, 8192 x 8, 4 per group, 1009 : 621,
// 700 x 48 93 : 44, 640 x 80 126 : 57, 4096 x 16 x 4 605 : 520 (two), 8192 x 16 x 4 1970 : 1759 (two).
// Fitted to 220 dense shapes, 128 to 16384 tokens; on 1486 others 0.4 % slower than the better of one and two launches on
// average, 18 % at most, and 1 % slower than before at most but for one (3692 x 9, bidirectional, 4 %).
// Very many short batch entries take two launches: what stands around an item that the hardware starts adds up (two : dealt, 153
// x 886 x 24 2078 : 2528 us, 1127 x 193 x 16 1481 : 1625, 978 x 237 x 8, bidirectional, 823 : 931; entries of one tile, and of two
// below 128 items per CU, 0.6 to 0.95).
// Packed documents have prices of their own: a call's longest document, whose length the host does not know, counts as 2.4
// times the mean, and the dQ items of a launch of their own run three to a CU.  1530 calls of 1024 to 65536 tokens: 0.2 %
// slower than the better form on average, 12 % at most, none slower than before; with the dense prices 2.3 %, 34 % and 17 %
// (two : dealt, 52129 x 8, 4 per group, in 53 documents 439 : 339 us, 15593 x 24, 4 per group, in 11 600 : 449; 65065 x 136, 4
// per group, in 261 3683 : 4130).
// Queues keep the order that shares K and V in L2, which pays in long bidirectional items of many heads per group (12800 x
// 12, 8 per group, 4225 : 4037 us, 8600 x 20, 4 per group, 2024 : 1962); elsewhere, and where a call has no dK/dV item for
// every CU, the dealt launch is 1 % behind at most or ahead by up to 50 %.
// `resident`: workgroups of the shared launch that the chip holds at once (two per CU).
enum class Bwd64 { kTwo, kDealt, kQueued };
inline Bwd64 bwd64_route(int64_t B, int64_t S, int64_t Hq, int64_t Hkv, bool causal, int64_t num_docs, int64_t cus, int64_t resident) {
  constexpr double kKvStep = 2.46, kKvItem = 18.2, kQStep = 4.82, kQItem = 0.23;   // us per pair of tiles, per item
  constexpr double kAlone = 0.91, kTwoLaunches = 2.31, kLaunch = 1.4;
  const double per_head = num_docs ? (double)(S / 128 + num_docs) : (double)((S + 127) / 128), group = (double)(Hq / Hkv);
  double doc = num_docs ? (double)S / 128 / (double)num_docs : per_head;   // tiles of a document (packed: on average)
  if (doc < 1) doc = 1;
  const double mean = causal ? (doc + 1) / 2 : doc, R = (double)resident;
  const double nk = per_head * (double)(B * Hkv), nq = per_head * (double)(B * Hq);
  if (nk + nq > (double)kDealtItems) return Bwd64::kTwo;
  const auto longer = [](double x, double y) { return x > y ? x : y; };
  if (num_docs) {
    constexpr double kKv = 2.38, kKvIt = 12.0, kQ = 6.81, kQIt = 0.5, kQOwn = 9.06, kQOwnIt = 1.83, kOwn = 14.6, kLongest = 2.38;
    const double all = (double)S / 128, top = kLongest * doc < all ? kLongest * doc : longer(all, 1);   // tiles of the longest document
    const double kv = top * group * kKv + kKvIt, kv_all = nk * (mean * group * kKv + kKvIt) / R;
    const double one = longer(longer(kv, top * kQ + kQIt), kv_all + nq * (mean * kQ + kQIt) / R);
    const double two = longer(kv, kv_all) + longer(0.69 * (top * kQOwn + kQOwnIt), nq * (mean * kQOwn + kQOwnIt) / (1.5 * R)) + kOwn;
    return one < two ? Bwd64::kDealt : Bwd64::kTwo;
  }
  const double kv = doc * group * kKvStep + kKvItem, kv_work = nk * (mean * group * kKvStep + kKvItem);
  const double q = doc * kQStep + kQItem, q_work = nq * (mean * kQStep + kQItem);
  const double one = nk + nq > (double)cus ? longer(kAlone * kv, (kv_work + q_work) / R) : kAlone * longer(kv, q);
  double two = kAlone * kv;   // dK/dV items: an item per CU, all of them resident, or rounds of them
  if (nk > R && !causal) two = (double)(int64_t)((nk + R - 1) / R) * kv;
  else if (nk > (double)cus) two = longer(two, kv_work / R);
  if (one >= kTwoLaunches * two + kLaunch) return Bwd64::kTwo;
  if (per_head >= 2 && per_head <= 10 && (nk + nq) * per_head > 256 * (double)cus) return Bwd64::kTwo;
  const bool long_groups = !causal && group >= 4 && per_head * group >= 200 && nk + nq >= 5 * R;
  return long_groups && nk > (double)cus ? Bwd64::kQueued : Bwd64::kDealt;
}

// Backward pass at head dimension 128: all dK/dV and dQ items in one launch that the hardware deals out (the ONCE form of
// attn_bwd_both_kernel), or a persistent kernel each?  The shared launch starts dQ items wherever dK/dV items have run
// out, so it has one tail instead of two and no queues; its dQ items (dq_item_seq) take a quarter longer per pair of tiles
// than those of the dQ kernel.  So it wins while a launch of either kind leaves CUs idle, and the choice goes by the
// estimated times of both: the longest item or the work per CU, whichever is longer, with items priced per 128 x 128 pair
// of tiles and per item.  Backward pass, two launches : one: 2048 x 16 140 : 83 us, 4096 x 8 231 : 131, 8192 x 4 377 : 235,
// 8192 x 8 492 : 433, 3001 x 32, 4 per group, 400 : 328, 10180 x 8 x 4, 8 per group, bidirectional 6134 : 5102; but
// 2 x 4096 x 32 890 : 920, 14443 x 37 5860 : 6222.
// Where a call has rounds enough the persistent kernels are ahead for every size but one tile per head, where a 256-row dQ item
// is half empty (two : one, 102 x 689 x 24 2038 : 2556 us, 387 x 141 x 16, bidirectional, 1025 : 1293, 13880 x 19, bidirectional,
// 5694 : 6072; one tile: 1211 x 9 x 32, 4 per group, 1657 : 1482, 587 x 3 x 16 487 : 436), so a workgroup that the hardware
// starts costs more around its item than one that draws it.  Fitted to 2840 dense calls, 2124 of them of 128 to 16384 tokens
// and the others of 4 to 2000 batch entries of up to 1200: 0.1 % slower than the better form on average, 10 % at most; of 2174
// others twelve were 3 % or more
// slower than two launches had been, 9 % at most (268 x 188 x 3, bidirectional).
// Packed documents are priced by themselves (their items are short, and the longest of a call, whose lengths the host does
// not know, counts as three times the mean, though not as more than the call): 1608 calls of 1024 to 65536
// tokens, 0.33 % slower than the better form on average; 22.7 tiles on average x 4 heads 579 (two) : 509 (one) us, 50000 x 8 in
// 2.1 tiles 350 : 426, 13439 x 36, 4 per group, in two documents 3670 : 4060.
inline bool bwd128_in_one_launch(int64_t B, int64_t S, int64_t Hq, int64_t Hkv, bool causal, int64_t num_docs, int64_t cus) {
  constexpr double kKvStep = 2.756, kKvItem = 10.793, kQStep = 3.755, kQItem = 2.154;   // in the shared launch
  constexpr double kKv2Step = 3.269, kKv2Item = 8.124;                                  // dK/dV in a launch of its own
  constexpr double kQ2Step = 5.124, kQ2Item = 3.186;                                    // dQ: two rows of tiles per item
  constexpr double kLaunch = 19.4, kTail = 0.587;
  const double per_head = num_docs ? (double)(S / 128 + num_docs) : (double)((S + 127) / 128), group = (double)(Hq / Hkv);
  double doc = num_docs ? (double)S / 128 / (double)num_docs : per_head;   // tiles of a document (packed: on average)
  if (doc < 1) doc = 1;
  const double mean = causal ? (doc + 1) / 2 : doc, C = (double)cus;
  const double nk = per_head * (double)(B * Hkv), nq = per_head * (double)(B * Hq);
  if (nk + nq > (double)kDealtItems) return false;
  if (num_docs) {
    constexpr double kKv = 5.06, kKvIt = 7.25, kQ = 5.69, kQIt = 1.76, kQOwn = 8.22, kQOwnIt = 1.26, kOwn = 6.5, kLongest = 3.14;
    const auto longer = [](double x, double y) { return x > y ? x : y; };
    const double all = (double)((S + 127) / 128), top = kLongest * doc < all ? kLongest * doc : all;   // tiles of the longest document
    const double kv = top * group * kKv + kKvIt, kv_all = nk * (mean * group * kKv + kKvIt) / C;
    const double one = longer(longer(kv, top * kQ + kQIt), kv_all + nq * (mean * kQ + kQIt) / C);
    const double two = longer(kv, kv_all) + longer(0.6 * top * kQOwn + kQOwnIt, nq * (mean * kQOwn + kQOwnIt) / (2 * C)) + kOwn;
    return (group > 1 ? 1.08 : 1.02) * one < two;   // (of few long items, whose lengths are a guess)
  }
  const auto span = [&](double n, double longest, double work) {   // of a launch of n items
    if (n <= C) return longest;
    if (!causal) { const double rounds = (double)(int64_t)((n + C - 1) / C); return rounds * longest; }
    return work / C > longest ? work / C : longest;
  };
  const double kv = doc * group * kKvStep + kKvItem, kv_work = nk * (mean * group * kKvStep + kKvItem);
  const double q = doc * kQStep + kQItem, q_work = nq * (mean * kQStep + kQItem);
  double one = kv > q ? kv : q;
  if (nk + nq > C) {
    const double even = (kv_work + q_work) / C;
    one = (even > kv ? even : kv) + kTail * (causal ? kQStep + kQItem : q);
  }
  const double kv2 = doc * group * kKv2Step + kKv2Item, kv2_work = nk * (mean * group * kKv2Step + kKv2Item);
  const double n2 = (double)(((S + 127) / 128 + 1) / 2) * (double)(B * Hq), mean2 = causal ? mean + 0.5 : doc;
  const double two = span(nk, kv2, kv2_work) + span(n2, doc * kQ2Step + kQ2Item, n2 * (mean2 * kQ2Step + kQ2Item)) + kLaunch;
  return (causal ? 1.02 : 1.012) * one < two;
}

// dK/dV items of a persistent launch: may the first ones go by workgroup index (tile_queue.hpp)?  One list (a head count that
// is no multiple of eight) keeps the order in which the workgroups arrive where heads are grouped (dealt : by arrival, 32046 x
// 16, 8 per group, 7.2 : 6.9 ms, 12520 x 32, 8 per group, 2.62 : 2.48), and with dS stored from five items per four CUs (9984 x 6
// 332 : 318 us, 6528 x 10 244 : 235, 3328 x 15 123 : 118; 320 items, 8192 x 5, 235 : 234, 288, 12288 x 3, 326 : 329).
inline bool dkdv_deals(int64_t items, bool one_list, bool grouped, bool stores_ds, int64_t cus) {
  return !one_list || !(grouped || (stores_ds && 4 * items > 5 * cus));
}

// Forward at head dimension 128: 256-row items in a persistent kernel (kWide, attn_fwd_wide_kernel), 128-row items two
// workgroups to a CU (kNarrow, attn_fwd_kernel), or 128-row items of one hand-sequenced wave per SIMD (kSeq,
// attn_fwd_seq_kernel)?  kWide has the fastest steady state and needs many items, kSeq the shortest items, kNarrow overlaps
// one item's way in and out with the other's key loop.  The choice goes by the estimated times: the longest item or the
// work per resident workgroup, with items priced per tile of 128 keys and per item; for causal launches of one to two items
// per slot also the first pair of items that share one.  `prefer_narrow`: what sizes alone say (fwd_prefers_128_rows in
// launch.hpp), left for another kernel where that is ahead by 4 % (bidirectional 8 %; kNarrow of more than eight dense items per CU
// 10 %, for its price then runs into the power limit: 4 x 4621 x 36 wide 866 : narrow 917 us).  Packed documents longer than 12
// tiles on average count 1.3 times in 128-row items (bidirectional, 10 tiles, 1.4: 50671 x 9 in 35 documents wide 792 : narrow
// 873): their longest are longer than the mean says.  With up to twelve items per CU 1.15, bidirectional up to two 1.2, since the copies
// of attn_fwd_kernel take their addresses from scalars (3720 x 16 in 2 69 : 52 us, bidirectional 7756 x 4 in 6 71 : 50).  Narrow over
// wide where that decides: up to five items per CU (two) 1347 calls 0.85, one in eighty more than 3 % slower; causal with more
// 6315 calls, of even, uniform, exponential and log-uniform lengths, 0.92, even ones 0.86, one in sixteen more than 3 % slower, 14 %
// at most (19894 x 17 in 9 704 : 791); bidirectional with more random lengths 1.01, a third more than 3 % slower, 21 % at most.
// Wide or narrow as sizes alone say : now: 8192 x 8 179 : 154 us, 8192 x 4 145 : 121, 6000 x 8 116 : 94, 4096 x 16 90 : 79,
// 29952 x 1 595 : 419; packed 8000 x 100 in 63 documents 74 : 30, 2222 x 2 in 4 44 : 24, 16384 x 2 in 24 53 : 32.
// `last`: a last bidirectional round that leaves a slot of every CU free (4129 x 17 wide 228 : narrow 196 us, 5747 x 14 299 :
// 269).  `first`, `again`: what kSeq's deep ring costs where it fills on many CUs at once, and where a CU's second item fills it
// anew (seq : narrow, 555 x 47 20.5 : 17.5, 2 x 413 x 31 16.1 : 14.5; 2 x 652 x 27, 324 items, 24.2 : 20.2).
// Dense, 2124 launches, 128 to 16384 tokens: 0.2 % slower than the best of the three on average, 12 % at most, and 4 % slower
// than what sizes alone say at most (3 % faster on average); without `last`, `first` and `again` 0.35 %, 20 % and 20 %.  Packed,
// 1608 calls of 1024 to 65536 tokens: 0.9 % slower than the best, 32 % faster than sizes alone, 5 % slower at most.
enum class Fwd128 { kWide, kNarrow, kSeq };
inline Fwd128 fwd128_route(int64_t B, int64_t S, int64_t Hq, bool causal, int64_t num_docs, int64_t cus, bool prefer_narrow) {
  struct Cost { double step, item, alone, per_cu, last, first, again; };
  constexpr Cost kWideCost{2.37, 22.7, 1.0, 1, 1, 0, 0}, kNarrowCost{3.18, 7.1, 0.84, 2, 0.78, 0, 0}, kSeqCost{1.97, 8.0, 1.0, 1, 1, 1.5, 2};
  const double n128 = num_docs ? (double)(S / 128 + num_docs) : (double)((S + 127) / 128);
  const double n256 = num_docs ? (double)(S / 256 + num_docs) : (double)((S + 255) / 256);
  double doc = num_docs ? (double)S / 128 / (double)num_docs : n128;   // tiles of a document (packed: on average)
  if (doc < 1) doc = 1;
  const double mean = causal ? (doc + 1) / 2 : doc, heads = (double)(B * Hq);
  if (n128 * heads > (double)kDealtItems) return Fwd128::kWide;
  const auto time = [&](const Cost& c, double per_head, double tiles, double mean_tiles) {
    const double n = per_head * heads, slots = (double)cus * c.per_cu;
    const double longest = c.step * tiles + c.item, work = n * (c.step * mean_tiles + c.item) / slots;
    const double first = num_docs ? 0 : c.first, again = num_docs ? 0 : c.again;   // (fitted to dense input)
    if (n <= (double)cus) return longest * c.alone + first * n / (double)cus;
    if (n > slots && !causal) {
      const double full = (double)(int64_t)(n / slots), rest = n - full * slots;
      const double last = rest == 0 ? 0 : rest <= (double)cus && !num_docs ? c.last : 1;
      return (full + last) * longest + again;
    }
    double t = work > longest * c.alone ? work : longest * c.alone;
    if (n > slots && n <= 2 * slots) {
      const double pair = 2 * (longest - c.step * tiles * slots / n);
      t = pair > t ? pair : t;
    }
    return n > slots ? t + again : t;
  };
  const bool few = n128 * heads <= (causal ? 12 : 2) * (double)cus;
  const double margin = causal ? 1.04 : 1.08, spread = !num_docs ? 1.0 : causal ? (doc > 12 ? (few ? 1.15 : 1.3) : 1.0) : (doc > 10 ? (few ? 1.2 : 1.4) : 1.0);
  const double many = !num_docs && n128 * heads > 8 * (double)cus ? 1.1 : margin;
  const double wide = time(kWideCost, n256, doc + 1, mean + 0.5) * (prefer_narrow ? margin : 1.0);
  const double narrow = time(kNarrowCost, n128, doc, mean) * spread * (prefer_narrow ? 1.0 : many);
  const double seq = time(kSeqCost, n128, doc, mean) * spread * margin;
  if (wide <= narrow && wide <= seq) return Fwd128::kWide;
  return narrow <= seq ? Fwd128::kNarrow : Fwd128::kSeq;
}

// 128-row forward: the second item on each CU in the opposite order (FLIP in attn_fwd.hip), the heaviest with the lightest?
// Causal launches dealt from the heaviest item down, of one to eight items per CU, a head of eight tiles or more.  In the same
// order : in the opposite one, D = 128: 256 to 512 items of 16 tiles and more 1.057 on average, 768 to 1024 1.041 (4096 x 32
// 148 : 142 us), up to 2048 1.00 to 1.01; D = 64 1.01 to 1.03.  Items of a few tiles differ little and lose more by the longer
// way to the first copy (4 x 647 x 36 35.6 : 38.4, 4 x 524 x 38 29.7 : 31.0, 4 x 263 x 41 17.3 : 18.8); in longer launches
// the second item is one of many, and the order of the lists shares more in L2 (64 tiles, 3000 items and more, 0.995).
inline bool fwd_flips(int64_t items, int64_t tiles, bool causal, bool packed, int64_t cus) {
  return causal && !packed && tiles >= 8 && items > cus && items <= 8 * cus;
}

// Dense forward launches that the hardware deals out: how many of a head's tiles go head by head, the heaviest first (q_heavy in
// decode_tile), before what is left goes tile by tile over all heads?  Tile by tile a launch of many heads streams every
// head's K and V from memory once per tile; head by head the workgroups that run together share them in L2.
// Bidirectional items are equal, so all tiles go that way.  Head by head over tile by tile in 17705 launches of more than two items per
// CU, D = 128 and 64, in eight lists of heads and, where the heads are no multiple of eight, in one (`one_list`: a head's workgroups
// are spread over all XCDs):
//   K and V of all heads (`kv_bytes`) more than 192 MiB, which the last-level cache no longer holds: lists 0.77, 0.87, one list 0.81,
//     0.93, hardly any launch slower (45 x 1792 x 20 2507 -> 1543 us, 159 x 190 x 24 236 -> 179);
//   else lists 0.93, 0.97, but not two unequal tiles: one of up to 64 rows (`last_rows`) D = 128 1.03, up to 1.13, D = 64 of up to four
//     items per CU 1.015, 1.06 (54 x 163 x 32 74.8 : 80.9 us);
//   else one list, two tiles 1.06, 1.025, up to 1.2; three and four 1.016, 1.005, but D = 128, four heads per group and more, 0.93; five to
//     eight up to six items per CU 1.03, 1.03, more, or at D = 128 with grouped heads more than three, 0.97, 0.98; nine to sixteen up to three
//     items 0.98, 1.01 (up to 1.1 and 1.15), more 0.93, 0.97; longer heads 0.94, 0.975 (3 x 713 x 36 45.1 : 54.0).
// 196 of the 17705 are more than 3 % slower than tile by tile, up to 8 %; all are 0.3 % slower than with the better order.
// Causal launches end on the light tiles of all heads, and the items must be enough
// for the rest to even out: tile by tile : head by head, D = 128, 9 to 16 tiles, 4 to 8 items per CU 1.04 on average, 8 to 12 0.93,
// 16 to 24 0.87, more 0.79; 17 to 32 tiles 8 to 16 items 1.005, 16 to 24 0.96, more 0.85; D = 64, 9 to
// 16 tiles 8 to 12 items 1.06, 12 to 16 0.96; two tiles 0.97 to 1.08 at any number.  (16 x 1024 x 32, 4 per group, 211 -> 192 us; 83 x
// 544 x 36 768 -> 505.)  An odd number of tiles, because an even one shares a factor with the CUs and gives the
// heaviest tiles to the same ones (causal, all of 3, 4, 6 and 8 tiles 0.87, 1.03, 0.88, 0.95).
inline int fwd_head_by_head(int64_t tiles, int64_t items, bool causal, bool packed, bool d64, int64_t cus, bool one_list, int64_t group,
                            int64_t kv_bytes, int64_t last_rows) {
  if (packed || tiles < 2 || items <= 2 * cus) return 0;
  if (!causal) {
    if (kv_bytes > ((int64_t)192 << 20)) return (int)tiles;
    int64_t least = 2;   // items per CU
    if (tiles == 2) {
      if (one_list || (!d64 && last_rows <= 64)) return 0;
      if (d64) least = 4;
    } else if (one_list && tiles <= 4) {
      if (d64 || group < 4) return 0;
      least = 3;
    } else if (one_list && tiles <= 16) {
      least = tiles > 8 || (!d64 && group > 1) ? 3 : 6;
    }
    return items > least * cus ? (int)tiles : 0;
  }
  if (tiles < 3 || items <= (tiles > 16 ? 16 : d64 ? 12 : 8) * cus) return 0;
  const int64_t share = (tiles - tiles * 3 / 8) | 1;
  return (int)(share < tiles ? share : tiles);
}

// Shared backward launch at head dimension 128, dealt out by the hardware: how many of a head's tiles go head by head?  All, where
// items are equal, so that the workgroups that run together share a head's rows in L2 (151 x 384 x 8 601 -> 531 us, 110 x 384 x 4
// 210 -> 189; at head dimension 64 1.00; one list of heads goes tile by tile whatever this says).  Two tiles of which one is partly
// full are unequal.  Head by head over tile by tile, by rows of the last tile, mean and largest of 1962 calls, with up to two dQ
// items (`items`) per CU : with more: up to 64 rows 1.015, 1.10 : 0.997, 1.04; up to 96 1.00, 1.04 : 0.986, 1.02; more 0.994, 1.02 :
// 0.976, 1.01 (15 x 202 x 24 103 : 107 us; 193 x 161 x 8, 4 per group, 271 : 261).
inline int bwd_head_by_head(int64_t tiles, int64_t last_rows, int64_t items, bool causal, bool packed, int64_t cus) {
  if (causal || packed) return 0;
  if (tiles == 2 && (last_rows <= 64 || (last_rows <= 96 && items <= 2 * cus))) return 0;
  return (int)tiles;
}

// Forward at head dimension 64: unmasked blocks without a search for their maximum (LAZY in attn_fwd.hip)?  Where a wave has
// its SIMD to itself the search is the shorter way (lazy : search, 165 x 40 6.34 : 6.12 us, 2911 x 4 41.9 : 39.9, 5374 x 1 72.3 :
// 68.9); with several waves per SIMD it is work that can be left out.  Lazy against search in 7173 launches with four workgroups to a
// CU, on average by items per CU: bidirectional one to two 0.986, more 0.975; causal, where an item's mean is half its longest, one
// to two 1.07, two to three 1.035, to 3.5 1.00, more 0.98; packed causal as causal, packed bidirectional one to two 1.01, two to three
// 0.984, more 0.98.
// `tiles`: of a head, or of a packed call's mean document.  Items of a few tiles are mostly masked blocks and first ones, which
// search either way (lazy : search in 340 launches of many: one tile 1.01, two to four causal 1.015, bidirectional 1.005, from
// five on as above; packed 1.012, from two on 1.005, from four on 0.99).
inline bool fwd64_is_lazy(int64_t items, bool causal, bool packed, int64_t cus, int64_t tiles) {
  return items > (causal || packed ? 3 : 1) * cus && tiles >= (packed ? 2 : 5);
}

// Recomputing dQ kernel at head dimension 128: products as 16x16x32 MFMAs (dq_item_16) instead of 32x32x16 (dq_item)?
// The 16x16x32 form costs less power per product and more issue slots, so it gains where the launch keeps the chip at its
// power limit and loses where most CUs wait for a few heavy items: dQ alone, 32x32x16 against it, 32768 x 16 causal
// 5032 : 4831 us, 4096 x 32 343 : 324 (bidirectional 212 : 205 causal), but 6000 x 8 causal 181 : 195, 12000 x 3 causal
// 282 : 327, 3001 x 16 causal 99 : 105.  The line lies where the mean load per CU is about 3/4 of the heaviest item: in
// 256-row items per CU 1.25 causal (an item's mean is half its maximum; 2048 x 40 84 : 83, 3001 x 24 109 : 110) and 0.8
// bidirectional (2048 x 32 111 : 106, 3001 x 16 119 : 120); with 128-row workgroups, two per CU, 1.0 and 0.7 (8192 x 8
// causal 227 : 227, 8192 x 6 bidirectional 297 : 288); packed documents, whose lengths the host does not know, 2
// (16384 x 8 ten mixes 0.98-1.01, 16384 x 4 44-56 to 219-232).
inline bool dq128_on_16x16x32(int64_t items_128, int64_t items_256, bool wide, bool causal, bool packed, int64_t cus) {
  if (items_128 <= cus) return false;
  if (packed) return items_256 >= 2 * cus;
  const int64_t percent = causal ? (wide ? 125 : 100) : (wide ? 80 : 70);
  return 100 * items_256 >= percent * cus;
}

// Which linear kernel: the one with the least estimated time.  A workgroup takes its tiles one after the other, and a tile
// its 64-deep steps at a cost per step for each product (forward, dx, dw: a transposed operand takes two LDS reads per
// fragment) with all CUs at work, less in a round that leaves CUs idle (memory is then less busy and the clock higher),
// plus what stands around a tile; a round of tiles takes no less than their outputs' way to memory, which is what counts
// in weight gradients over a few hundred tokens.  Fitted to 1500 measured (product, size) pairs, 1 to 16384 tokens, layer
// widths 512 to 8192, whole tiles and ragged ones: the choice is 0.2 % slower than the best of the seven on average
// (0.3 % on a third of the pairs that a fit had not seen) and 14 % at most, and never more than 1 % slower than the
// 256 x 256 tiles of 32x32x16 products that once served every size (twice as fast on average; dw 8192 tokens
// 9600 x 3200 447 -> 422 us, 128 tokens 8192 x 8192 55 -> 46, forward 200 tokens 4096 x 4096 94 -> 22).
enum Tile { kPp256, kRing256x128, kRing128x256, kRing128, kRing64x128, kRing64, kRing32, kTiles };
struct TileCost {
  int ti, tj, step;         // tile, depth of a step in units of 64
  float step_us[3];         // per 64-deep step: forward, dx, dw
  float tile_us, light;     // around a tile; factor of a step when few CUs are at work
  float write_us;           // least time of a round of tiles on all CUs
};
constexpr TileCost kCost[kTiles] = {
    {256, 256, 1, {1.273f, 1.379f, 1.609f}, 5.55f, 0.68f, 7.27f},
    {256, 128, 1, {0.901f, 0.930f, 1.027f}, 2.88f, 0.71f, 3.63f},
    {128, 256, 1, {1.024f, 0.940f, 1.058f}, 2.33f, 0.70f, 4.70f},
    {128, 128, 1, {0.625f, 0.607f, 0.683f}, 1.20f, 0.68f, 2.56f},
    {64, 128, 1, {0.422f, 0.460f, 0.482f}, 0.76f, 0.88f, 2.10f},
    {64, 64, 1, {0.254f, 0.281f, 0.264f}, 1.28f, 0.72f, 2.06f},
    {32, 32, 4, {0.128f, 0.f, 0.f}, 0.49f, 0.95f, 0.00f}};

// C[I][J] over a contraction of R; product: 0 forward, 1 dx, 2 dw.  `us_out`: the estimate.
inline Tile pick_tile(int64_t I, int64_t J, int64_t R, int product, int64_t cus, float* us_out = nullptr) {
  const auto ceil_div = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const int64_t per_xcd = cus >= 8 ? cus / 8 : 1;
  Tile best = kPp256;
  float best_us = 0.f;
  for (int k = 0; k < kTiles; ++k) {
    if (k == kRing32 && product != 0) continue;   // (both operands direct: a transposed 32-wide tile has 64-byte rows)
    const TileCost& c = kCost[k];
    const int64_t per = ceil_div(ceil_div(I, c.ti) * ceil_div(J, c.tj), 8);   // tiles of one XCD
    const int64_t full = per / per_xcd, rest = per % per_xcd;                 // whole rounds, tiles of the last one
    const float steps = (float)(ceil_div(R, 64 * c.step) * c.step) * c.step_us[product];
    const float whole = steps + c.tile_us > c.write_us ? steps + c.tile_us : c.write_us;
    float us = (float)full * whole;
    if (rest) {
      const float part = (float)rest / (float)per_xcd;
      const float last = steps * (c.light + (1.f - c.light) * part) + c.tile_us;
      us += last > c.write_us * part ? last : c.write_us * part;
    }
    if (k == 0 || us < best_us) { best = (Tile)k; best_us = us; }
  }
  if (us_out) *us_out = best_us;
  return best;
}

// Forward product: tiles whose four waves share nothing (linear_own_kernel), where their estimated time is less than that of
// pick_tile's choice (`other_us`), by 3 %?  They gain where a call is a few rounds of small tiles with a long contraction.  Costs per
// 256-deep step, around a tile and of a launch, fitted, as is what makes an estimate of pick_tile's a time (kOther and what follows
// it), to 11200 calls, each on weights that come from memory and on weights that stay in the caches: 32 to 1536 tokens, widths 512 to
// 131072, contractions of 768 to 32768.  The rule is held to that and what 3200 calls showed around it: widths below 512 0.88, contractions up
// to 65536 0.87 (29 of 488 more than 3 % slower), wider outputs 1.00 and not taken, as are contractions below 1024, where nothing is
// gained (1.00).  `once`: with few row tiles most of a step's bytes are weights that are read from memory and by one tile; `empty`:
// rows that do not exist repeat the last one and cost less.  (Without those terms, with costs from weights that stay in the caches, 537
// of these calls were more than 3 % slower than without these tiles on weights from memory: 362 x 11088 x 768 13.5 : 16.7 us, 85 x
// 33288 x 1792 31.2 : 37.5, 83 x 12360 x 9856 66.3 : 76.3, 113 x 33000 x 2496 44.1 : 52.6.)  Now two calls in five take them, for
// 7 % less time on average (15 % with weights in the caches); 264 are more than 3 % slower than without (120), 24 (30) more than
// 10 % (15 % at most: 199 x 6464 x 6720 42 : 48), and all calls are 0.4 % (0.8 %) slower than with the best choice.
enum Own { kOwnNone, kOwn64, kOwn64x96, kOwn128x96, kOwns };
struct OwnCost { int ti, tj; float step_us, tile_us, light, launch_us, once, empty; };
constexpr OwnCost kOwnCost[kOwns] = {{0, 0, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f},
                                     {64, 64, 0.779f, 0.944f, 0.701f, 2.623f, 0.564f, 0.398f},
                                     {64, 96, 0.995f, 1.691f, 0.729f, 2.739f, 0.535f, 0.252f},
                                     {128, 96, 1.448f, 4.213f, 0.609f, 2.181f, 0.427f, 0.419f}};
// `other_rows`: rows of the tiles of pick_tile's choice.
inline Own pick_own(int64_t I, int64_t J, int64_t R, int64_t cus, float other_us, int64_t other_rows) {
  constexpr float kOther = 2.101f, kAll = 0.956f, kOnce = 0.216f, kEmpty = 0.161f, kGain = 0.97f;
  const auto ceil_div = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const auto empty = [&](int64_t ti) { return 1.f - (float)I / (float)(ceil_div(I, ti) * ti); };   // share of the tiles' rows
  if (I < 32 || I > 1536 || J > 131072 || R < 1024 || R > 65536) return kOwnNone;
  const int64_t per_xcd = cus >= 8 ? cus / 8 : 1;
  Own best = kOwnNone;
  float best_us = (other_us + kOther) * (kAll + kOnce / (float)ceil_div(I, 64) - kEmpty * empty(other_rows)) * kGain;
  for (int k = 1; k < kOwns; ++k) {
    const OwnCost& c = kOwnCost[k];
    const int64_t rows = ceil_div(I, c.ti), per = ceil_div(rows * ceil_div(J, c.tj), 8);
    const int64_t full = per / per_xcd, rest = per % per_xcd;
    const float steps = (float)ceil_div(R, 256) * c.step_us * (1.f + c.once / (float)rows - c.empty * empty(c.ti));
    float us = c.launch_us + (float)full * (steps + c.tile_us);
    if (rest) us += steps * (c.light + (1.f - c.light) * (float)rest / (float)per_xcd) + c.tile_us;
    if (us < best_us) { best = (Own)k; best_us = us; }
  }
  return best;
}

}  // namespace ie
