// Byte offsets inside a tile of rows that may lie far apart (the strided entry points).
//
// The tile loader adds an unsigned 32-bit per-lane offset to a scalar tile address, so the distance
// between a tile's first and last row has to fit 32 bits: rows of a tile times the largest row stride.
//
// Plain C++ (no HIP): used by the kernels, by the argument checks and by a host test.
#pragma once

constexpr int kMaxTileRows = 128;                    // rows of the largest streamed tile
constexpr long long kRowStrideLimit = 1ll << 24;     // row strides (in elements, multiples of 8) stay below

// byte offset of 16-byte chunk `chunk_bytes` of row `row`, in unsigned arithmetic: from a stride of
// 8.4 million elements on the last rows of a 128-row tile lie beyond 2^31
constexpr unsigned row_offset(int row, int row_stride, int chunk_bytes) {
  return (unsigned)row * (2u * (unsigned)row_stride) + (unsigned)chunk_bytes;
}
static_assert((kMaxTileRows - 1) * 2ll * (kRowStrideLimit - 8) + 64 <= 1ll << 32, "a tile spans less than 4 GiB");
