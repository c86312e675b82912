// Token rows of one head on their way into LDS, for the any-length attention kernels: rows of 64 bf16 = 128 bytes, without
// a pass through registers, eight rows per load and wave.
#pragma once
#include "common.h"
#include "mfma_util.h"

namespace mb {

// A staged row is 8 pieces of 16 bytes; piece x of row r sits at position x ^ stage_swizzle(r).  Both ways of reading are
// free of bank conflicts so: a fragment read takes one piece of 16 consecutive rows per quarter wave (pairs of rows fill
// the 64 banks, and the 8 pairs lie at 8 different positions), a transposing read takes half of 4 consecutive rows per half
// wave (rows 0, 1 and rows 2, 3 lie in different halves: bit 1 of the row moves the piece by four).
__device__ __forceinline__ int stage_swizzle(int row) {
  return 4 * ((row >> 1) & 1) + 2 * ((row >> 2) & 1) + ((row >> 3) & 1);
}

// What a lane reads of eight rows whose first is a multiple of 8 and has `odd` = (first / 8) % 2.
__device__ __forceinline__ int stage_piece(int lane, int odd) { return (lane & 7) ^ stage_swizzle(lane >> 3) ^ odd; }
// Its byte offset inside them; `stride` elements from row to row.
__device__ __forceinline__ uint32_t stage_lane_off(int lane, int odd, int64_t stride) {
  return ((uint32_t)(lane >> 3) * (uint32_t)stride + (uint32_t)stage_piece(lane, odd) * 8u) * 2u;
}

// One head of `count` consecutive rows (fewer than 2^31 bytes) as a descriptor: a lane's offset past the last row is out of
// its range and deposits zeros.
__device__ __forceinline__ u32x4 stage_rsrc_bytes(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  u32x4 r;
  r[0] = (uint32_t)a;
  r[1] = (uint32_t)(a >> 32) & 0xffffu;
  r[2] = bytes;
  r[3] = 0x00020000u;   // raw buffer, 32-bit data format (gfx9 family)
  return r;
}
__device__ __forceinline__ u32x4 stage_rsrc(const uint16_t* first_row, int64_t stride, int count) {
  return stage_rsrc_bytes(first_row, count > 0 ? ((uint32_t)(count - 1) * (uint32_t)stride + 64u) * 2u : 0u);
}

// 64 pieces of 16 bytes, or of 4 (lse, Delta), from `lane_off` bytes into a descriptor to byte `lds` and behind it.
__device__ __forceinline__ void stage_rows(uint32_t lds, uint32_t lane_off, u32x4 rsrc) { load_to_lds(lds, lane_off, rsrc, 0u); }
__device__ __forceinline__ void stage_words(uint32_t lds, uint32_t lane_off, u32x4 rsrc) { load_word_to_lds(lds, lane_off, rsrc); }
// 64 pieces of 16 bytes, each lane from its own address.
__device__ __forceinline__ void stage_each(uint32_t lds, const void* lane_ptr) { load_to_lds_each(lds, lane_ptr); }

// Rows that are not consecutive, or too far apart for a descriptor: every lane's own address (`head`: the head's columns in
// buffer row 0).  Lanes whose row is at or beyond `count` read zeros here.
static __device__ const uint32_t kZeroPiece[4] = {0u, 0u, 0u, 0u};
__device__ __forceinline__ const void* stage_address(const uint16_t* head, int64_t stride, const int32_t* __restrict__ rows,
                                                     int start, int first, int count, int lane, int odd) {
  const int i = first + (lane >> 3);
  const void* p = kZeroPiece;
  if (i < count) p = head + tok_row(rows, start + i) * stride + stage_piece(lane, odd) * 8;
  return p;
}

// Byte offsets of what a lane reads of a staged tile as matrix operands.  Rows (lds_read8): k-step s takes columns
// 16 s + 8 g .. + 7 of row lane % 32, the next 32 rows lie 4096 bytes on.
__device__ __forceinline__ void stage_row_places(int lane, uint32_t (&at)[4]) {
  const int c = lane & 31, g = lane >> 5;
#pragma unroll
  for (int s = 0; s < 4; ++s) at[s] = (uint32_t)(c * 64 + ((2 * s + g) ^ stage_swizzle(c)) * 8) * 2;
}
// Transposed patches (lds_read_tr4, two halves joined): columns 32 db .. + 31 of 16 rows, the next 16 rows 2048 bytes on.
__device__ __forceinline__ void stage_tr_places(int lane, uint32_t (&at)[2][2]) {
  const int i = lane & 15, q = lane >> 4;
  const int row = (i >> 2) + 4 * (q >> 1), piece = 2 * (q & 1) + ((i & 3) >> 1);
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int r = row + 8 * half;
      at[db][half] = (uint32_t)(r * 64 + ((4 * db + piece) ^ stage_swizzle(r)) * 8 + 4 * (i & 1)) * 2;
    }
}

// All but the newest `kNewer` loads of this wave have arrived and its LDS operations are done; then the workgroup's barrier.
template <int kNewer>
__device__ __forceinline__ void staged_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(kNewer) : "memory");
}

}  // namespace mb
