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
// its range and deposits zeros.  (From 129 rows on the last row of a tile that holds any stays below 2^32 bytes, so what has to
// be zeros is.  In the tiles that are requested beyond it an offset may wrap round: those loads stay inside the descriptor and
// nobody reads what they bring.)
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
// buffer row 0, `row`: the buffer row of the lane's token).  Lanes without a token read zeros here.
static __device__ const uint32_t kZeroPiece[4] = {0u, 0u, 0u, 0u};
__device__ __forceinline__ const void* stage_address(const uint16_t* head, int64_t stride, int row, bool there, uint32_t piece_bytes) {
  const void* p = kZeroPiece;
  if (there) p = reinterpret_cast<const char*>(head + (int64_t)row * stride) + piece_bytes;
  return p;
}
// The buffer row of token i of a sequence that has `count` (past the end: of its last token).
__device__ __forceinline__ int stage_row_of(const int32_t* __restrict__ rows, int start, int i, int count) {
  const int t = start + min(i, count - 1);
  return rows ? rows[t] : t;
}

// (waited for here: among the loads into LDS, of which the compiler knows nothing, it would wait for all of those as well)
template <int kN>
__device__ __forceinline__ void rows_known(int (&row)[kN]) {
#pragma unroll
  for (int j = 0; j < kN; ++j) asm volatile("" : "+v"(row[j]));
}

// Where token_rows says where the rows are, a wave brings the row numbers of its 16 rows of a tile (8 w .. + 7 and 32 behind
// them) to LDS a step before it requests the rows.  A number that a lane waits for in a register is waited for behind
// every tile requested before it, which puts each step's loads a memory round trip behind the last ones.  So and now, masks with
// holes: 64 sequences of up to 512 tokens, 12 heads, forward 62 and 48 us, dQ + dK/dV 177 and 131; 16 of up to 1815, 16 heads, 150
// and 116, 382 and 303.
struct StageRows {
  static constexpr int kWords = 2 * 4 * 64;   // LDS: two tiles, four waves
  const int32_t* rows;   // the sequence's row numbers, nullptr: token t sits in row t
  int start, count, wave;
  int32_t* part;         // this wave's words
  __device__ __forceinline__ StageRows(const int32_t* all, int start_, int count_, int32_t* words, int wave_)
      : rows(all ? all + start_ : nullptr), start(start_), count(count_), wave(wave_), part(words + wave_ * 64) {}
  // byte offset of the number that a lane brings of the first tile
  static __device__ __forceinline__ uint32_t lane_off(int wave, int lane) {
    return (uint32_t)(8 * wave + (lane & 7) + 4 * (lane & 8)) * 4u;
  }
  __device__ __forceinline__ void request(int t, uint32_t lane_off) const {   // of tile t (past the end: zeros)
    if (!rows) return;
    const uint64_t a = reinterpret_cast<uint64_t>(rows);
    const u32x4 rsrc = {(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a),
                        (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu),
                        (uint32_t)__builtin_amdgcn_readfirstlane(count * 4), 0x00020000u};
    const uint32_t lds = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) int32_t*)part);
    stage_words(__builtin_amdgcn_readfirstlane(lds + (t & 1) * 1024), lane_off + (uint32_t)t * 256u, rsrc);
  }
  // the row of the lane's token in the wave's first (half 0) or second eight rows of tile t
  __device__ __forceinline__ int get(int t, int half, int lane) const {
    return rows ? part[(t & 1) * 256 + half * 8 + (lane >> 3)] : start + t * 64 + 8 * (wave + 4 * half) + (lane >> 3);
  }
};

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
