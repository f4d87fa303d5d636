// How the grouped GEMMs split an expert's dispatched rows into items and the
// items over workgroups.  Plain constexpr arithmetic, used by the dispatch, the
// kernels and the host code that sizes their grids.
#pragma once

namespace amoe {

// M-tiles per wave, in one M group and in each of two (see grouped.hip)
constexpr int grouped_tile_m(int elem_bytes) { return elem_bytes == 2 ? 8 : 2; }
constexpr int grouped_tile_m2(int elem_bytes) { return elem_bytes == 2 ? 6 : 2; }
// most rows of an item; items above grouped_big_rows take two M groups and half runs
constexpr int grouped_item_rows(int elem_bytes) { return 2 * 16 * grouped_tile_m2(elem_bytes); }
constexpr int grouped_big_rows(int elem_bytes) { return 16 * grouped_tile_m(elem_bytes); }

// An expert's `count` rows in items m = 0 .. items - 1 of min(rows, count - rows m)
// rows, the first `big` of which are big.  bf16: equal runs of whole M-tiles, at
// most item_rows each, all big or none, whatever the last one holds.  fp32, whose
// time is the M-tiles multiplied (a big item's four, also for fewer rows): full
// items and the rest, 65 rows in 64 + 1 rather than 48 + 17 (16 experts, top-1,
// 1075 tokens, H = 1088, I = 1760: 323 -> 221 us a step).
struct ItemSplit {
  int rows, items, big;
};
constexpr ItemSplit split_rows(int count, int elem_bytes) {
  const int item_rows = grouped_item_rows(elem_bytes), big_rows = grouped_big_rows(elem_bytes);
  const int most = (count + item_rows - 1) / item_rows;
  if (elem_bytes == 4) return {item_rows, most, count / item_rows + (count % item_rows > big_rows ? 1 : 0)};
  const int tiles = (count + 15) / 16;
  const int rows = most > 0 ? 16 * ((tiles + most - 1) / most) : 16;
  const int items = (count + rows - 1) / rows;
  return {rows, items, (rows < count ? rows : count) > big_rows ? items : 0};
}

// most items of a block of `slots` routing entries: one per active expert and
// one more per full item
constexpr int grouped_max_items(int slots, int E, int item_rows) {
  return (E < slots ? E : slots) + slots / item_rows;
}

// The last items take half runs, as many of them as make one round of the
// resident workgroups, two per CU (half as many measured 1-3 % slower at 4 x 60
// nodes, twice as many 2-4 % at 4 x 60 and 32 x 60: a half run stages the item's
// rows again).
constexpr int grouped_split_items(int nblocks) {
  constexpr int kHalfRuns = 512;
  return (kHalfRuns / 2 + nblocks - 1) / nblocks;
}

// fp32: all items take quarter runs, whose waves share the K chunks, while their
// half runs are no more than this, one per CU: fp32 products take a wave so long
// that the idle CUs cost more than the rows staged twice as often.  Drawn blocks of
// 193 to 1600 tokens, top-1 and top-2 mostly: 8 % faster than without (twice as
// many 6 %, half as many 7 %), 360 tokens, 32 experts, top-2 (H = 3424, I = 224)
// 210 -> 150 us a step.
constexpr int kQuarterHalves = 256;
constexpr bool grouped_quarters(int n_items, int nblocks, int elem_bytes) {
  return elem_bytes == 4 && n_items <= kQuarterHalves / (2 * nblocks);
}

// Workgroup `block`'s share: output run `run` of the `parts` x nblocks that an
// item's runs are cut into; nothing if item >= n_items.  The n_big big items come first and take half runs, as do
// the last ones.  The items go round-robin over the XCDs (workgroup b
// runs on XCD b % 8), all runs of one on the same XCD.
struct GroupedShare {
  int item, run, parts;
};
constexpr GroupedShare grouped_share(int block, int n_items, int n_big, int n_split, int nblocks, int elem_bytes) {
  const int xcd = block % 8;
  const int n_whole = n_big > n_items - n_split ? n_big : n_items - n_split;  // items [n_big, n_whole) take whole runs
  const int big = (n_big + 7 - xcd) / 8, whole = (n_whole + 7 - xcd) / 8;      // of the first n items on this XCD
  int slot = block / 8, first = 0, parts = 2;  // item `first` of the XCD starts at slot 0
  if (grouped_quarters(n_items, nblocks, elem_bytes)) {
    parts = 4;
  } else if (slot >= 2 * nblocks * big) {
    slot -= 2 * nblocks * big;
    first = big;
    parts = 1;
    if (slot >= nblocks * (whole - big)) {
      slot -= nblocks * (whole - big);
      first = whole;
      parts = 2;
    }
  }
  const int item = slot / (parts * nblocks);  // one division for all: a branch each cost every workgroup three
  return {(first + item) * 8 + xcd, slot - item * parts * nblocks, parts};
}

// Workgroups that cover every item's nblocks runs for any routing of `slots`
// entries: per XCD one whole run's workgroups for each item and as many again
// for the big items and for the last ones.  There are at most slots / big_rows
// big items.  fp32: each holds more than big_rows rows.  bf16: runs of
// big_rows / 16 + 1 M-tiles or more in each of n items make more than
// n big_rows / 16 M-tiles, so the expert has at least n big_rows rows although its
// last item may hold fewer (257 rows: 144 + 113).
constexpr long long grouped_workgroups(int slots, int max_items, int nblocks, int elem_bytes) {
  const int n_split = grouped_split_items(nblocks);
  const int max_big = slots / grouped_big_rows(elem_bytes);
  const long long groups = (max_items + 7) / 8 + (max_big + 7) / 8 + ((n_split < max_items ? n_split : max_items) + 7) / 8;
  const int most_q = kQuarterHalves / (2 * nblocks);  // items in quarter runs
  const long long quarters = grouped_quarters(1, nblocks, elem_bytes) ? 4 * (((most_q < max_items ? most_q : max_items) + 7) / 8) : 0;
  return 8 * (groups > quarters ? groups : quarters) * nblocks;
}

}  // namespace amoe
