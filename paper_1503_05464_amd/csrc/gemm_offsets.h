// How the batched GEMM addresses A: 32-bit byte offsets within a chunk of the
// inner dimension, and the test that says whether a product's A allows them.
// Plain C++, so that the arithmetic can be checked on the host.
#pragma once

namespace hss {

constexpr int kGemmSlice = 16;     // k of one slice
constexpr int kGemmChunk = 512;    // k of one chunk: offsets start anew at each
constexpr int kGemmMaxRows = 128;  // rows of the tallest tile

// Offset from the tile's first entry of a chunk to row `row`, entry `k` of its
// first slice (A is M x K, or K x M if transposed), and from one slice to the
// next.  Taken modulo 2^32.
constexpr unsigned gemm_entry_offset(bool trans, long long lda, int row, int k) {
  return 8u * (unsigned)(trans ? (long long)k * lda + row : (long long)row * lda + k);
}
constexpr unsigned gemm_slice_step(bool trans, long long lda) {
  return 8u * (unsigned)(trans ? kGemmSlice * lda : kGemmSlice);
}

// Whether no offset of a tile wraps: the entries of a whole number of slices
// lie within 2^32 - 1 bytes, the most that a buffer resource spans.
constexpr bool gemm_offsets_fit(bool trans, int M, int K, long long lda) {
  const long long rows = M < kGemmMaxRows ? M : kGemmMaxRows;
  const long long ks = K < kGemmChunk ? (K + kGemmSlice - 1) / kGemmSlice * kGemmSlice : kGemmChunk;
  const long long most = 0xffffffffll / 8;
  return trans ? lda <= (most - rows) / (ks > 0 ? ks : 1) : lda <= (most - ks) / (rows > 0 ? rows : 1);
}

}  // namespace hss
