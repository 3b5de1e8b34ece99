// Which form of the two backward kernels serves a problem: how many rows a work-group owns and how many wave groups share
// them (the groups take alternate 32-row blocks of the other side and add their sums at the end).
//
//   form      dQ: queries per work-group                dK/dV: keys per work-group
//   1         128, one group of four waves              the same
//   kDense    -                                         the same, three waves per SIMD (d <= 64)
//   2         64, two groups of two waves               128, two groups of four waves
//   kHalf     -                                         64, two groups of two waves (d <= 96)
//   4         64, four groups of two waves              the same
//   8         32, eight groups of one wave (d <= 64)    the same
//   kNarrow   32, four groups of one wave (d 96, 128)   the same (eight groups' tiles would not fit the LDS)
//
// What decides.  Without a mask all blocks are equal and the number of rounds counts.  Under the mask the work-group of the
// longest block decides, as long as the others fit beside it: more groups walk it faster, but each of them has eight waves
// to itself (one work-group per CU) and pays for the exchange at the end, which short sequences do not earn back.  So
// with growing grids the best form goes from many groups on few rows to one group on 128.  "Block" below is one of
// 128 rows, "ordered" says that the head count is a multiple of eight: only then the order table (block_order.hpp)
// balances a causal grid; dK/dV runs the others as pairs of mirrored blocks, half as many work-groups.
// The forms differ in the order of float32 sums only.  The rules look at sizes alone, never at strides, and those of dK/dV at the
// keys only, so that a chunk of queries gets the sums of the square problem.
// Figures: us per kernel, launched back to back, at the sizes named; B H is written as one number of heads.
//
// Plain C++ (no HIP): used by the launchers and by a host test.
#pragma once
#include "block_order.hpp"

constexpr int kNarrow = 5, kHalf = 6, kDense = 7;
constexpr int kNoGroupsBelow = 512;          // keys; shorter sequences do not pay for the exchange

// forms that exist (are compiled) for a kernel
constexpr bool dkdv_has_form(int d, bool causal, bool grouped, int form) {
  return form == 1 || (form == kDense && d <= 64 && !grouped) || (form == 2 && d <= 128 && !(causal && d <= 64)) ||
         (form == kHalf && d <= 96 && !grouped) || (form == 4 && d <= 128) || (form == 8 && d <= 64) ||
         (form == kNarrow && d > 64 && d <= 128);
}
constexpr bool dq_has_form(int d, int form) {
  return form == 1 || form == 2 || (form == 4 && d <= 128) || (form == 8 && d <= 64) || (form == kNarrow && d > 64 && d <= 128);
}

// kHalf.  Resident at once: three work-groups per CU at d <= 64, two at d = 96 (222 to 237 registers).
constexpr bool dkdv_takes_half(int d, bool causal, bool grouped, long long heads, int nk) {
  if (!dkdv_has_form(d, causal, grouped, kHalf)) return false;
  const long long blocks = heads * ((nk + 127) / 128), halves = heads * ((nk + 63) / 64);
  const bool ordered = heads % 8 == 0;
  if (blocks > 3 * kNumCUs / 2) return false;
  if (!causal) {
    // against one group.  d64 H18 N2048 52.7 -> 45.2; beyond the limit H77 N640 23.2 -> 28.4.  d = 96: as long as all are
    // resident (H54 N576 29.0 -> 22.6, but H58 21.1 -> 22.7), and beyond that where both kernels are the aligned ones (H17 N2048 71.1 ->
    // 65.8; with bounds checks H11 N3000 97.6 -> 106.3) and, on short sequences, the XCDs share the heads out (work-groups in
    // eights: H64 N640 29.7 -> 27.4, but H70 30.8 -> 34.7).
    if (blocks <= kNumCUs) return false;
    return d <= 64 || halves <= 2 * kNumCUs || (nk % 128 == 0 && (halves % 8 == 0 || nk >= 768));
  }
  // Above one block per CU, against one group (d = 96: two on 128 keys): d64 H24 N1536 29.5 -> 24.0, d96 35.1 -> 28.9.  In pairs even
  // or worse (d96 H18 N2688 61.2 -> 66.1), but for short sequences at d = 96 (H43 N768 28.4 -> 27.8).
  if (blocks > kNumCUs) return ordered || (d == 96 && nk <= 1024);
  // Below, against four groups, whose work-groups then take two rounds; longer sequences are decided by the longest block.
  // d64 H24 N1000 18.5 -> 17.3; d32 at the lower limit H24 N768 9.87 -> 10.22; in pairs d64 H17 N1000 19.0 -> 19.8, d96 21.5 -> 20.5.
  if (nk > 1024) return false;
  return d == 96 ? blocks > kNumCUs / 2 : ordered && blocks > 9 * kNumCUs / 16;
}

// heads: key/value heads of all batches; grouped: several query heads to each
constexpr int dkdv_form(int d, bool causal, bool grouped, long long heads, int nk) {
  const long long blocks = heads * ((nk + 127) / 128);
  const bool pairs = causal && heads % 8 != 0;
  if (nk >= kNoGroupsBelow && d <= 128) {
    // 32 keys, as long as every work-group gets a CU of its own.  Four groups on 64 keys -> this: d64 H8 N1024 causal 13.8 -> 11.3, H1
    // N1024 17.8 -> 15.8, d128 H1 N5120 69.3 -> 48.5; beyond the limit d64 H24 N1000 18.5 -> 31.1.
    // d = 64 in pairs: up to two tiles of 256 queries eight groups are slower than four, and two on 64 keys faster than either
    // (four, eight, two: H10 N640 15.7, 16.4, 14.4; H22 16.4, 17.4, 15.2; from three tiles on H11 N768 16.7, 15.6, 16.0).
    if (blocks <= (pairs ? 2 : 1) * kNumCUs / 4)
      return d > 64 ? kNarrow : d == 64 && pairs && !grouped && nk < 768 ? kHalf : 8;
    if (dkdv_takes_half(d, causal, grouped, heads, nk)) return kHalf;
    // 64 keys, four groups: two groups on 128 keys -> this: H64/16 N2048 d128 causal 200 -> 149, H16 N2048 d64 35.3 -> 28.5, H8 N2048
    // d128 full 50.4 -> 39.1; beyond the limits H24 N2048 d128 causal 62 -> 89, H48 N1024 d64 26.0 -> 37.5.
    if (blocks <= (causal ? kNumCUs : kNumCUs / 2)) return 4;
    // 128 keys, two groups (under the mask at d >= 96 only: at d <= 64 two work-groups of one group fit a CU and do as well): one
    // group -> this: H24 N2048 d128 causal 70.8 -> 62.6, H16 N2048 d128 full 74.4 -> 66.5; beyond the limits H40 N2048 d128 causal 93 -> 129,
    // H24 N2048 d128 full 108 -> 114, H48 N1024 d64 causal 24.5 -> 26.0.
    if (dkdv_has_form(d, causal, grouped, 2) && blocks <= (causal ? 2 : 1) * kNumCUs) return 2;
  }
  // Three waves per SIMD where the grid has them: two -> three: H96 N1024 d64 causal 39.1 -> 35.7, H384 N512 full 62.5 -> 58.6, H96 N1024 d32
  // causal 28.2 -> 23.4; just above the limit H400 N200 d64 causal 19.0 -> 19.2; below it H48 N1024 24.5 -> 25.4.
  if (dkdv_has_form(d, causal, grouped, kDense) && blocks > (pairs ? 4 : 2) * kNumCUs) return kDense;
  return 1;
}

// Two groups on 64 queries.  Resident at once: four work-groups per CU at d = 32, three at d = 64, two at d = 96 and 128.
constexpr bool dq_takes_two(int d, bool causal, long long heads, int nq, int nk) {
  const long long blocks = heads * ((nq + 127) / 128), halves = heads * ((nq + 63) / 64);
  const bool ordered = heads % 8 == 0;
  if (!causal) {
    // d = 128: against four groups, up to half a block per CU (H8 N1024 16.8 -> 15.6, H8 N2048 27.1 -> 26.1; H17 N1024 with one group
    // 21.4 -> 23.7); four groups walk the longer sequences faster (H3 N3000 35.1 -> 36.5).
    if (d == 128) return blocks <= kNumCUs / 2 && nk <= 2048;
    // Otherwise against one group, above one block per CU: d64 H18 N2048 40.7 -> 34.8, d96 53.2 -> 50.0.  Past two work-groups per CU
    // K and V are read from L2 for 64 queries at a time, which short sequences pay for where the XCDs do not share the heads out
    // (work-groups in eights): d96 H58 N640 23.6 -> 28.3, H53 N768 27.4 -> 30.8, d64 H58 N640 17.5 -> 18.4.
    if (blocks <= kNumCUs || blocks > 3 * kNumCUs / 2) return false;
    return d == 32 || halves <= 2 * kNumCUs || halves % 8 == 0 || nk >= (d == 64 ? 768 : 1024);
  }
  // Under the mask, lower limit, against four groups: the longest block decides up to there, and four groups walk it faster, the longer
  // the sequence the further: from half a block per CU (d = 128: a quarter) at 1024 keys to one block at 2816.  H24 N1024 d64 15.2 ->
  // 12.9, H14 N2048 26.6 -> 24.3, H32 N1024 d128 26.2 -> 19.9; below the limit H16 N1280 d64 14.3 -> 14.6, H12 N2048 21.5 -> 24.1.  At d = 32,
  // where a tile has the least work, one block from 640 keys (unordered grids: 1024) on: H24 N1000 9.4 -> 10.1, H16 N2048 13.1 -> 15.1, but
  // H26 N1000 11.7 -> 11.2.
  const int line = 80 + nk / 16 < kNumCUs ? 80 + nk / 16 : kNumCUs;
  const int above = d == 32 ? (nk <= (ordered ? 640 : 1024) ? kNumCUs / 2 : kNumCUs)
                            : nk > 1024 ? line : d == 128 ? kNumCUs / 4 : kNumCUs / 2;
  // Upper limit, against one group: d32 H17 N2048 27.7 -> 21.6, d64 H9 N4096 69.2 -> 50.8, H48 N1024 18.2 -> 15.5, d96 H20 N2048 46.0 -> 38.1,
  // d128 56.8 -> 47.5.  Short sequences past the two resident work-groups per CU of d = 96 and 128: d96 H59 N768 24.5 -> 26.5 (ordered:
  // H48 18.5 -> 16.1), d128 H80 N512 18.6 -> 19.6.
  const int short128 = kNumCUs + (nk - kNoGroupsBelow) / 2;
  const int upto = d == 32 ? 2 * kNumCUs
                 : d == 64 || (d == 96 && (nk > 1024 || ordered)) ? 3 * kNumCUs / 2
                 : d == 96 || short128 > 5 * kNumCUs / 4 ? 5 * kNumCUs / 4 : short128;
  return blocks > above && blocks <= upto;
}

// heads: query heads of all batches
constexpr int dq_form(int d, bool causal, long long heads, int nq, int nk) {
  const long long blocks = heads * ((nq + 127) / 128);
  if (nk < kNoGroupsBelow) return 1;
  if (d > 128) {
    // One wave per SIMD: two groups on 64 queries are what fits.  H8 N2048 full 73 -> 57, beyond half a block per CU H16 95 -> 109.
    // The causal mask takes the limit to one block per CU only where the order table balances the halved blocks, in square problems
    // (with more keys than queries the blocks differ less) and from 1500 keys on: H16 N2048 85 -> 79, H8 N4000 145 -> 124; not taken:
    // H15 N2048 82 -> 98, H24 N1280 57 -> 60, H32 N1024 51 -> 53.
    const bool balanced = causal && heads % 8 == 0 && nk == nq && nq >= 1500;
    return blocks <= (balanced ? kNumCUs : kNumCUs / 2) ? 2 : 1;
  }
  // 32 queries, up to one work-group per CU.  Four groups on 64 queries -> this: d64 H8 N1024 causal 11.5 -> 9.9, H1 N5120 30.4 -> 20.1, d128
  // H8 N1024 17.3 -> 12.9; beyond the limit d64 H12 N1024 11.4 -> 15.6.
  if (blocks <= kNumCUs / 4) return d <= 64 ? 8 : kNarrow;
  if (dq_takes_two(d, causal, heads, nq, nk)) return 2;
  // 64 queries, four groups: one group on 128 -> this: H16 N2048 d128 causal 50 -> 45, H8 N2048 d64 30 -> 18, H8 N2048 d128 full 44 -> 32;
  // beyond the limits H24 N2048 d128 causal 52 -> 66, H16 N2048 d128 full 57 -> 64.
  return blocks <= (causal ? kNumCUs : kNumCUs / 2) ? 4 : 1;
}
