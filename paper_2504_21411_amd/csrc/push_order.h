// Numbering of the push kernel's workgroups: plain functions of integers, for host and device alike.
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
// cache line that two tiles store (the shifts are not aligned) meet in its L2.  Two things keep the
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

} // namespace gs
