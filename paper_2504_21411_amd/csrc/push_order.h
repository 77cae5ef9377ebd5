// Numbering of the push kernel's workgroups and the rows a wave takes: plain functions of integers, for
// host and device alike.
#pragma once

namespace gs {

// A work item is a (row block, instance) pair; its jsplit slices of the targets are one workgroup
// each.  The hardware deals consecutive workgroups round-robin to the eight XCDs, each with its own
// L2 and 32 compute units, and the slices of an item read the same source rows: they are numbered so
// that they land on one XCD and the rows are fetched into one L2 only,
//   workgroup = (item of the XCD * jsplit + slice) * 8 + XCD.
//
// run = 0: items by row block, then instance, dealt round-robin.
// run > 0: an XCD takes the row blocks of one instance one after the other, so that the parts of a
// cache line that two tiles store (the shifts are not aligned) meet in its L2.  Counted, 2048 instances,
// 24 strategies, 2048 bins, a front: writes of less than 64 bytes 637 -> 240 thousand of 6.3 million with
// backpointers, 85 -> 53 of 4.7 million min-only; HBM bytes 687 -> 676 MB.  Two things keep the
// XCDs and their compute units evenly loaded however the work is spread:
//   - round r gives instance 8 r + (XCD + r) % 8 to an XCD: budgets that repeat every eight
//     instances would otherwise fill one XCD with the large ones (512 instances, 24 strategies, 4096
//     bins, budgets of 1/8 to 8/8: 706 -> 543 us over 9 fronts, min-only 620 -> 500; equal budgets 975
//     both);
//   - run is odd: with 8 or 16 row blocks the k-th of every instance would go to the same few of an
//     XCD's 32 compute units, and most of the work is in the middle ones or, under a small budget, in
//     the first (1024 instances, 16 strategies, 2047 bins: 639 -> 594 us, min-only 576 -> 550).
struct PushItem {
  int b, row_block, slice; // (b or row_block may lie beyond the last: nothing to do)
};

constexpr PushItem push_item(unsigned workgroup, int jsplit, int B, int run) {
  const int q = (int)(workgroup >> 3), xcd = (int)(workgroup & 7u);
  const int item = q / jsplit, slice = q - item * jsplit;
  if (run > 0) {
    const int round = item / run;
    return {round * 8 + ((xcd + round) & 7), item - round * run, slice};
  }
  const unsigned at = (unsigned)item * 8u + (unsigned)xcd, row_block = at / (unsigned)B;
  return {(int)(at - row_block * (unsigned)B), (int)row_block, slice};
}

constexpr int push_run(long long row_blocks, bool by_instance) {
  return by_instance ? (int)(row_blocks | 1) : 0;
}

constexpr long long push_workgroups(long long row_blocks, long long B, int jsplit, int run) {
  return (run > 0 ? (B + 7) / 8 * run : (row_blocks * B + 7) / 8) * 8 * jsplit;
}

// By instance, where the planes are too large for the 256 MB memory-side cache to put the parts of a
// line together (a plane is read, one written, backpointers beside it) and XCDs that get one instance
// less do not idle for more than a tenth.  (A batch of a multiple of 8 has its instances bound to XCDs
// in either order.)  7 to 9 fronts, us, plain / by instance, plane of the whole batch: 25 MB (64
// instances, 12 strategies) 118 / 126, 34 MB (256, 8) 136 / 153, 58 MB (1000, 12) 261 / 275, 61 MB (256,
// 24) 239 / 248; 77 MB (300, 8) 230 / 224, min-only 233 / 209; 98 MB (512, 12) 334 / 330, 350 / 329; 115
// MB (150, 16) 396 / 361, 404 / 386; 346 MB (300, 24) 1492 / 1227, 1182 / 985; 403 MB (2048, 24, 11
// fronts) 2884 / 2328, 2270 / 1787; two groups of 15 instances (44), budgets of 1/8 to 8/8 of 40000
// bins, min-only 482 / 513.
constexpr bool push_by_instance(long long plane_bytes, int B) {
  return plane_bytes >= (64ll << 20) && (B % 8 == 0 || (B >= 32 && 10 * (8 - B % 8) <= B));
}

// Groups of 64 rows per wave: they share a column's scalar loads, its T and O and the loop; they cost
// registers.  Measured, 7 fronts, us at one / two groups, the order as push_by_instance says: S = 8
// 8064 tiles 85 / 76, 12600 tiles 100 / 85, 16384 143 / 131, 37888 262 / 220 (min-only 250 / 208); S = 16
// 11280 tiles 178 / 181, 16384 238 / 227, 16884 235 / 231 (min-only 244 / 229); beyond, by instance: S
// = 16 42210 652 / 681 (534 / 560), 65536 747 / 814, S = 24 24101 578 / 599 (500 / 523), 65536 1485 /
// 1542, S = 32 23475 799 / 822 (625 / 656); plain: S = 16 31300 471 / 461 (442 / 439), S = 24 31300 851 /
// 807 (683 / 654), 18760 421 / 416 (413 / 414), S = 32 15640 522 / 541 (461 / 479); S = 44 16380 968 /
// 1025.
// With a few strategies a column is so short that four groups pay.  Whole searches, two / four: S = 1 14
// K tiles 66 / 60, 79 K 308 / 233; S = 2 57 K 108 / 92, min-only 319 K (15 fronts) 1219 / 818; S = 3 8.8 K 88 /
// 86, 54 K 311 / 261, min-only 106 K 290 / 228; S = 4 10 K 107 / 112, 15.5 K 160 / 154, 43 K 236 / 197, by
// instance 255 K min-only 1150 / 1196; S = 6 22 K 318 / 324, min-only 16 K 180 / 176, 28 K 283 / 260.  Over
// 164 random shapes of up to 8 strategies the groups picked take 1.010 times the best ones' time, two at
// most 1.055.
constexpr int push_row_groups(int S, bool with_bp, long long tiles, bool by_instance) {
  if (S <= 3 && tiles >= 8192) return 4;
  if (S == 4 && tiles >= 12288 && !by_instance) return 4;
  if (S <= 6 && !with_bp && tiles >= 16384 && !by_instance) return 4;
  const bool two = S <= 8    ? tiles >= 4096
                   : S <= 16 ? tiles >= 12288 && (tiles < 24576 || !by_instance)
                             : S <= 32 && tiles >= 24576 && !by_instance;
  return two ? 2 : 1;
}

} // namespace gs
