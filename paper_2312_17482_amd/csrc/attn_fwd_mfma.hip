// Forward ALiBi attention on the matrix cores: bf16, head_dim 64, variable-length packed sequences.
//
// Computes the attention weights of the paper's Eq. 1, softmax_j(scale * q_i.k_j - m_h*|i-j|), and
// O = P V tile by tile with a running (online) softmax, so the score matrix never leaves the chip
// ("FlashAttention" paragraph).  The bias is evaluated in registers from the token distance.
//
// Work split: one workgroup (4 waves) per (sequence, head, tile of 128 queries); wave w owns queries
// 32w..32w+31 of the tile.  K and V tiles of 128 keys are staged in LDS and shared by the 4 waves.
// Global memory is always touched as full 128-byte rows of one head (8 lanes x 16 bytes).
// Scores are produced TRANSPOSED, S^T = K Q^T (keys along accumulator rows, queries along lanes), so
//   * a query's row statistics (max, sum) are reductions over a lane's own registers plus one
//     exchange with the partner lane l^32, and
//   * the accumulator tile, rounded to bf16, is already the B operand of O^T += V^T P^T.
#include "attn_plan.h"
#include "attn_stage.h"
#include "common.h"
#include "mfma_util.h"

namespace mb {
namespace {

constexpr int kBlockQ = 128;   // queries per workgroup
constexpr int kBlockK = 128;   // keys per LDS tile
constexpr int kD = 64;
constexpr int kKStride = 72;   // LDS row pitch of K in bf16 (144 B): 16-byte row reads spread over banks
constexpr int kVStride = 80;   // LDS row pitch of V in bf16 (160 B): 4-row transposing reads spread over banks

// Any sequence length: tiles of 64 keys with a running (online) softmax.  The tiles go straight to LDS, two steps ahead,
// through a ring of three regions (attn_stage.h): no registers and no vector instructions on the way, no bank conflicts,
// one barrier per tile.  At most 168 registers and 50 KB of LDS, so that three workgroups share a compute unit.
// Same arithmetic as the single-tile kernel below (bias in the accumulator's start value, scale folded into the exponent);
// the running output is rescaled only when some query's maximum actually moved.
// What bounds it at full length: the vector unit.  A tile costs a wave about 155 vector instructions of 4 cycles, 32
// exponentials of 8 and 10 for each of 16 matrix instructions to be issued, 1030 cycles; it takes 1340.
// With tiles through registers and padded rows (a quarter of the LDS cycles were conflicts), before and after: 16 x 2048 tokens,
// 16 heads 340 and 328 us; 64 x 64 .. 512 tokens, 12 heads 53 and 48 us; 64 x 512 with a key mask 86 and 79 us.
// Tried: the tile with the diagonal first and outwards from there, so that the maximum hardly moves: 328 -> 339 us.
constexpr int kTileK = 64;                                        // keys per LDS tile
constexpr int kRegion = 2 * kTileK * kD;                          // one K tile + one V tile, as attn_stage.h stages them
constexpr int kRing = 3;                                          // regions

// A sequence longer than the max_seqlen the launch was sized for: the sticky flag is raised and the
// sequence's log-sum-exp rows (n of them, from `row`) become NaN, so the misuse shows in the result too.
__device__ __forceinline__ void poison_lse(float* __restrict__ row, int n, int32_t* __restrict__ misuse) {
  raise_misuse(misuse);
  for (int i = threadIdx.x; i < n; i += blockDim.x) row[i] = __builtin_nanf("");
}

// The forward's own plan launch: workgroup c builds list c (see attn_plan.h); workgroup 0 then marks the
// sequences the plan skipped (longer than max_seqlen) by setting their log-sum-exp rows to NaN.
__global__ __launch_bounds__(kPlanThreads) void attn_plan_kernel(const int32_t* __restrict__ cu,
                                                                 const int32_t* __restrict__ key_lens, int B, int H,
                                                                 int max_seqlen, int64_t cap, int32_t* __restrict__ plan,
                                                                 int32_t* __restrict__ misuse, float* __restrict__ lse,
                                                                 int T) {
  __shared__ __attribute__((aligned(16))) PlanLds lds;
  build_plan_list(cu, key_lens, B, H, max_seqlen, cap, plan, blockIdx.x, misuse, lds);
  if (blockIdx.x != 0 || lse == nullptr) return;
  // is there one at all?  (a thread per sequence: looked at one after the other, 64 sequences took as long as the plan)
  bool skipped = false;
  for (int b = threadIdx.x; b < B; b += kPlanThreads) skipped = skipped || cu[b + 1] - cu[b] > max_seqlen;
  if (!__syncthreads_or(skipped)) return;
  for (int b = 0; b < B; ++b) {
    const int s0 = cu[b], len = cu[b + 1] - s0;
    if (len > max_seqlen)
      for (int h = 0; h < H; ++h) poison_lse(lse + (int64_t)h * T + s0, len, misuse);
  }
}

// kMode (see kRowsIdentity .. in common.h): the rows of a sequence whose tokens sit in consecutive rows of the activation
// buffers, spanning fewer than 2^31 bytes, are loaded through descriptors that start at its first row and end at its last
// one: a lane's offset grows by a constant from tile to tile, and rows past the end arrive as zeros without a compare.
// Otherwise every lane forms its own address (row numbers out of token_rows, if given: StageRows).
template <int kMode>
__global__ __launch_bounds__(256, 3) void attn_fwd_tiled_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v, int64_t qs,
    int64_t ks, int64_t vs, const float* __restrict__ slopes, float scale, uint16_t* __restrict__ o, int64_t os,
    float* __restrict__ lse, int T, const int32_t* __restrict__ token_rows, const int32_t* __restrict__ plan,
    int64_t plan_cap) {
  const int32_t* rows = kMode == kRowsIdentity ? nullptr : token_rows;
  __shared__ __attribute__((aligned(1024))) uint16_t smem[kRing * kRegion];   // 48 KB; also stages Q and O rows
  __shared__ __attribute__((aligned(16))) int32_t sRows[kMode == kRowsIdentity ? 4 : StageRows::kWords];

  int start, n, nk, qtile, h;   // nk <= n: the sequence's first nk tokens are its keys
  if (!plan_fetch(plan, plan_cap, &start, &n, &nk, &qtile, &h)) return;   // this XCD's list is shorter
  const int q0 = qtile * kBlockQ;   // < n by construction of the plan
  // first buffer row of the sequence, and whether its tokens sit in consecutive rows
  const int row0 = kMode == kRowsMaybeContiguous ? __builtin_amdgcn_readfirstlane(rows[start]) : start;
  const bool contig =
      kMode == kRowsIdentity ||
      (kMode == kRowsMaybeContiguous && __builtin_amdgcn_readfirstlane(rows[start + n - 1]) - row0 == n - 1);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps per-wave branches scalar
  const int c = lane & 31, g = lane >> 5;
  const int qw = q0 + 32 * wave;          // first query of this wave
  const bool wave_active = qw < n;
  const int qi = qw + c;                  // this lane's query (position inside the sequence)
  const int qblk = (q0 >> 5) + wave;      // index of this wave's block of 32 queries
  const int ntiles = (nk + kTileK - 1) / kTileK;

  // ---- loads: this wave's Q rows, then its share of the K / V tiles
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint16_t*)smem);
  const StageRows where(rows, start, nk, sRows, wave);
  int own_row[4], first_row[4];   // without descriptors: rows of the wave's queries and of its share of two tiles
  if (!contig) {
#pragma unroll
    for (int j = 0; j < 4; ++j) own_row[j] = stage_row_of(rows, start, qw + 8 * j + (lane >> 3), n);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      first_row[j] = stage_row_of(rows, start, (j >> 1) * kTileK + 8 * (wave + 4 * (j & 1)) + (lane >> 3), nk);
    rows_known(own_row);
    rows_known(first_row);
  }
  {
    const u32x4 q_rsrc = stage_rsrc(q + row0 * qs + h * kD, qs, n);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t at = lds0 + (2 * kRegion + (32 * wave + 8 * j) * kD) * 2;
      if (contig) stage_rows(at, stage_lane_off(lane, j & 1, qs) + (uint32_t)(qw + 8 * j) * (uint32_t)qs * 2u, q_rsrc);
      else stage_each(at, stage_address(q + h * kD, qs, own_row[j], qw + 8 * j + (lane >> 3) < n, stage_piece(lane, j & 1) * 16));
    }
  }
  const u32x4 k_rsrc = stage_rsrc(k + row0 * ks + h * kD, ks, nk), v_rsrc = stage_rsrc(v + row0 * vs + h * kD, vs, nk);
  // the wave's first 8 rows of the tile to load next; its second 8 rows lie 32 behind them (without descriptors: the lane's
  // place among the row numbers, and inside a row)
  uint32_t k_off = stage_lane_off(lane, wave & 1, ks) + 8u * wave * (uint32_t)ks * 2u;
  uint32_t v_off = stage_lane_off(lane, wave & 1, vs) + 8u * wave * (uint32_t)vs * 2u;
  if (!contig) {
    k_off = StageRows::lane_off(wave, lane);
    v_off = stage_piece(lane, wave & 1) * 16;
  }
  constexpr int kRowLoads = 4;   // loads per wave and tile
  auto place = [&](int region, int j) {   // of the j-th of them: K and V rows by turns
    return lds0 + (uint32_t)(region * kRegion + ((j & 1) == 0 ? 0 : kTileK * kD) + 8 * (wave + 4 * (j >> 1)) * kD) * 2;
  };
  auto issue_row = [&](int region, int j) {   // with descriptors; the tiles are taken in order
    const bool is_k = (j & 1) == 0;
    uint32_t& off = is_k ? k_off : v_off;
    stage_rows(place(region, j), off, is_k ? k_rsrc : v_rsrc);
    off += 64u * (uint32_t)(is_k ? ks : vs);
  };
  auto issue_each = [&](int t, int region, const int* row) {   // without: tile t, whose rows are `row`
#pragma unroll
    for (int j = 0; j < kRowLoads; ++j) {
      const bool is_k = (j & 1) == 0;
      stage_each(place(region, j), stage_address((is_k ? k : v) + h * kD, is_k ? ks : vs, row[j >> 1],
                                                 t * kTileK + 8 * (wave + 4 * (j >> 1)) + (lane >> 3) < nk, v_off));
    }
  };
  // Requests tile t, two steps behind the newest that has arrived, and before it the row numbers of the tile behind it.
  auto issue_tile = [&](int t, int region) {
    if (contig) {
#pragma unroll
      for (int j = 0; j < kRowLoads; ++j) issue_row(region, j);
    } else {
      const int row[2] = {where.get(t, 0, lane), where.get(t, 1, lane)};
      where.request(t + 1, k_off);
      issue_each(t, region, row);
    }
  };
  if (contig) {
    issue_tile(0, 0);
    issue_tile(1, 1);
  } else {
    issue_each(0, 0, first_row);
    where.request(2, k_off);
    issue_each(1, 1, first_row + 2);
  }

  // ---- places in a region (bytes): K rows, transposed patches of V
  const char* const lds = reinterpret_cast<const char*>(smem);
  uint32_t row_at[4], tr_at[2][2];
  stage_row_places(lane, row_at);
  stage_tr_places(lane, tr_at);
  bf16x8 bq[4];   // Q^T fragments of the wave's own rows
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(2 * kRowLoads) : "memory");
#pragma unroll
  for (int s = 0; s < 4; ++s)
    bq[s] = lds_read8(reinterpret_cast<const uint16_t*>(lds + row_at[s] + (2 * kRegion + 32 * wave * kD) * 2));

  const float cs = scale * kLog2e;
  const float k1 = slopes[h] / scale;

  f32x16 oacc[2];
#pragma unroll
  for (int i = 0; i < 16; ++i) { oacc[0][i] = 0.f; oacc[1][i] = 0.f; }
  float m_run = -INFINITY;   // running maximum of the raw accumulator (dot product + bias/scale)
  float l_run = 0.f;         // running row sum, this half-wave's share

  f32x16 row_bias;           // (m_h / scale) * (accumulator row) left of the diagonal, its negative right of it
#pragma unroll
  for (int i = 0; i < 16; ++i) row_bias[i] = k1 * (float)(8 * (i >> 2) + (i & 3));
  asm volatile("" : "+v"(row_bias));   // in vector registers: the compiler would keep it in scalar ones and copy it each time

  // One tile of 64 keys.  The code that touches the running output exists once, with no branch
  // around it: a ragged last tile is handled by setting the scores of the keys that do not exist to -inf (their
  // K rows are staged as zeros), and only the first product has variants.
  auto tile = [&](int jt, uint32_t region, auto load) {
    const int j0 = jt * kTileK;
    const int rem = nk - j0;
    uint32_t ka[4], va[2][2];
#pragma unroll
    for (int s = 0; s < 4; ++s) ka[s] = row_at[s] + region;
#pragma unroll
    for (int s = 0; s < 4; ++s) va[s >> 1][s & 1] = tr_at[s >> 1][s & 1] + region;
    auto read_k = [&](int jb, int s) {
      return lds_read8(reinterpret_cast<const uint16_t*>(lds + ka[s] + jb * (32 * kD * 2)));
    };
    auto read_v = [&](int jb, int kk, int db) {
      const uint32_t at = (kTileK + 32 * jb + 16 * kk) * kD * 2;
      return join_tr(lds_read_tr4(reinterpret_cast<const uint16_t*>(lds + va[db][0] + at)),
                     lds_read_tr4(reinterpret_cast<const uint16_t*>(lds + va[db][1] + at)));
    };
    float fi = (float)(qi - j0 - 4 * g);   // i - j = fi - cj with cj = 32jb + 8*(v/4) + v%4
    asm volatile("" : "+v"(fi));
    // Off the diagonal block |i-j| = +-(fi - cj) is linear: its part per accumulator row is the same in every block (up
    // to the sign) and enters as the first product's C operand, straight from the registers that hold it; its part per
    // lane, off[jb], is added to the block's maximum and to the exponent's constant.  No instruction per score.
    f32x16 sacc[2];
    float off[2];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
      const int kblk = 2 * jt + jb;
      const bf16x8 ak = read_k(jb, 0);
      if (kblk == qblk) {   // the block that holds the diagonal; the ones behind it lie on its other side
        f32x16 diag;
#pragma unroll
        for (int i = 0; i < 16; ++i) diag[i] = -k1 * fabsf(fi - (float)(jb * 32 + 8 * (i >> 2) + (i & 3)));
        sacc[jb] = mfma32(ak, bq[0], diag);
        off[jb] = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) row_bias[i] = -row_bias[i];
      } else {
        sacc[jb] = mfma32(ak, bq[0], row_bias);
        off[jb] = (kblk < qblk ? -k1 : k1) * (fi - (float)(32 * jb));
      }
    }
#pragma unroll
    for (int s = 1; s < 4; ++s) {
      sacc[0] = mfma32(read_k(0, s), bq[s], sacc[0]);
      sacc[1] = mfma32(read_k(1, s), bq[s], sacc[1]);
    }
    load(0);
    load(1);
    if (rem < kTileK) {   // ragged end: keys that do not exist (or are masked out) get -inf
      const int lim = rem - 4 * g;
#pragma unroll
      for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          sacc[jb][i] = (jb * 32 + 8 * (i >> 2) + (i & 3)) >= lim ? -INFINITY : sacc[jb][i];
    }
    float mt = -INFINITY;
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
      float mb = -INFINITY;
#pragma unroll
      for (int i = 0; i < 16; ++i) mb = fmaxf(mb, sacc[jb][i]);
      mt = fmaxf(mt, mb + off[jb]);
    }
    mt = max_both_halves(mt);
    const float m_new = fmaxf(m_run, mt);
    if (jt > 0 && __any(m_new > m_run)) {   // some query's maximum moved: rescale the running sums
      const float alpha = fast_exp2((m_run - m_new) * cs);
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < 16; ++i) { oacc[0][i] *= alpha; oacc[1][i] *= alpha; }
    }
    m_run = m_new;
    float lsum[4] = {0.f, 0.f, 0.f, 0.f};   // four short chains of additions instead of one long one
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
      const float e0 = (off[jb] - m_new) * cs;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float p = fast_exp2(fmaf(sacc[jb][i], cs, e0));
        sacc[jb][i] = p;
        lsum[i & 3] += p;
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 bp = pack8(sacc[jb][8 * kk + 0], sacc[jb][8 * kk + 1], sacc[jb][8 * kk + 2],
                                sacc[jb][8 * kk + 3], sacc[jb][8 * kk + 4], sacc[jb][8 * kk + 5],
                                sacc[jb][8 * kk + 6], sacc[jb][8 * kk + 7]);
#pragma unroll
        for (int db = 0; db < 2; ++db) oacc[db] = mfma32(read_v(jb, kk, db), bp, oacc[db]);
      }
      if (jb == 0) {
        load(2);
        load(3);
      }
    }
    l_run += (lsum[0] + lsum[1]) + (lsum[2] + lsum[3]);
  };

  // Step jt: tile jt has arrived, the next one is on its way and the one behind that is requested.  Loads past the end are
  // issued too: their number stays the same.
  int region = 0;
  if (!wave_active) {   // (a loop of its own: inside the other one the accumulators would be copied in every step)
    for (int jt = 0; jt < ntiles; ++jt) {
      staged_barrier<kRowLoads>();
      issue_tile(jt + 2, region == 0 ? kRing - 1 : region - 1);
      region = region == kRing - 1 ? 0 : region + 1;
    }
    staged_barrier<0>();
    return;
  }
#pragma unroll 1
  for (int jt = 0; jt < ntiles; ++jt) {
    const int to = region == 0 ? kRing - 1 : region - 1;   // of tile jt + 2: the region of tile jt - 1
    staged_barrier<kRowLoads>();
    if (!contig) issue_tile(jt + 2, to);
    tile(jt, (uint32_t)region * (kRegion * 2), [&](int j) {
      if (contig) issue_row(to, j);
    });
    region = region == kRing - 1 ? 0 : region + 1;
  }
  staged_barrier<0>();   // everyone is done with the K/V regions: they now carry the output rows

  const float l = sum_both_halves(l_run);
  const float inv = 1.f / l;
  if (g == 0 && qi < n) lse[(int64_t)h * T + start + qi] = (m_run * cs + __log2f(l)) * kLn2;
  // O^T accumulators -> 32 LDS rows private to this wave -> full 128-byte rows
  uint16_t* slab = &smem[(32 * wave) * kKStride];
#pragma unroll
  for (int db = 0; db < 2; ++db) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      u32x2 w;
      w[0] = pack_bf16(oacc[db][4 * r + 0] * inv, oacc[db][4 * r + 1] * inv);
      w[1] = pack_bf16(oacc[db][4 * r + 2] * inv, oacc[db][4 * r + 3] * inv);
      *reinterpret_cast<u32x2*>(&slab[c * kKStride + 32 * db + 8 * r + 4 * g]) = w;
    }
  }
  const int orow = lane >> 3, ocol = (lane & 7) * 8;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int row = 8 * it + orow;
    const u32x4 w = *reinterpret_cast<const u32x4*>(&slab[row * kKStride + ocol]);
    if (qw + row < n) *reinterpret_cast<u32x4*>(o + tok_row(rows, start + qw + row) * os + h * kD + ocol) = w;
  }
}

// ------------------------------------------------------------------------------------------------ n <= 128
// Sequences of at most 128 tokens (the pretraining length of the paper): one K/V tile per
// (sequence, head), so the softmax is a single pass with no running rescale.  Such a unit is tiny
// (48 KB in, 16 KB out), so the kernel is built for occupancy: one workgroup per (sequence, head),
// <= 128 registers and 39 KB of LDS, i.e. four workgroups per compute unit whose load, compute and
// store phases overlap each other.
//
// Arithmetic per score is kept to a handful of vector instructions:
//   * the accumulator of S^T = K Q^T is not zeroed but pre-loaded with bias/scale = -(m_h/scale)|i-j|,
//     so the matrix core adds the bias; off the diagonal block |i-j| is linear in i and j, which makes
//     the pre-load one fused multiply-add per score;
//   * the row maximum is taken on the raw accumulator and the scale is folded into the exponent:
//     p = exp2(acc * c - max * c), c = scale * log2(e)   (requires scale > 0).
// kRows: the activation buffers are a padded batch and token t sits at row rows[t] (the gather and the
// scatter of the unpadding step happen in this kernel's own row loads and stores).
template <bool kRows>
__global__ __launch_bounds__(256, 4) void attn_fwd_short_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v, int64_t qs,
    int64_t ks, int64_t vs, const int32_t* __restrict__ cu, const float* __restrict__ slopes, float scale,
    uint16_t* __restrict__ o, int64_t os, float* __restrict__ lse, int T, const int32_t* __restrict__ rows,
    int32_t* __restrict__ misuse, const int32_t* __restrict__ key_lens) {
  // Every global access is a full 128-byte row of one head shared by 8 lanes (16 bytes each); the
  // fragment layouts the matrix cores need are produced by passing through LDS:
  //   sV first carries the Q tile (rows -> Q^T fragments), then V;  after the S phase each wave reuses
  //   its own 32 rows of sK to turn its O^T accumulators back into rows.
  __shared__ __attribute__((aligned(16))) uint16_t sK[kBlockK * kKStride];
  __shared__ __attribute__((aligned(16))) uint16_t sV[kBlockK * kVStride];

  const int h = blockIdx.x, b = blockIdx.y;
  const int start = cu[b];
  const int n = cu[b + 1] - start;
  if (n <= 0) return;
  if (n > kBlockK) {   // the caller promised max_seqlen <= 128: skipped, never truncated
    poison_lse(lse + (int64_t)h * T + start, n, misuse);
    return;
  }
  const int nk = key_lens ? min(key_lens[b], n) : n;   // the sequence's first nk tokens are its keys
  if (nk <= 0) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 31, g = lane >> 5;
  const int qi = 32 * wave + c;
  const int nblk = (n + 31) >> 5;       // blocks of 32 queries
  const int nblk_k = (nk + 31) >> 5;    // blocks of 32 keys
  const bool wave_active = wave < nblk;

  // ---- coalesced row loads: thread (st_row, st_col) moves 16 bytes of rows st_row, +32, +64, +96
  const int st_row = tid >> 3, st_col = (tid & 7) * 8;
  u32x4 tq[4], tk[4], tv[4];
  // Rows listed in ascending order whose first and last differ by n - 1 are consecutive (the usual
  // case: padding is a suffix of each batch row); then no per-token index load is needed.
  int row0 = start;
  bool contig = true;
  if (kRows) {
    row0 = __builtin_amdgcn_readfirstlane(rows[start]);
    contig = __builtin_amdgcn_readfirstlane(rows[start + n - 1]) - row0 == n - 1;
  }
  // Consecutive rows move with buffer instructions (256 x 128 positions, 16 heads, padded rows: 51 us with an address and a
  // compare per lane, 48 so; packed rows the same either way): a descriptor per tensor from the unit's first row to its last, 32-bit
  // offsets (127 rows of 2^24 elements stay below 2^32 bytes), zeros and dropped stores past the end without a compare.
  auto rsrc = [&](const uint16_t* base, int64_t stride, int cnt) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base) + ((int64_t)row0 * stride + h * kD), 0,
                                             (int)(((uint32_t)(cnt - 1) * (uint32_t)stride + kD) * 2u), 0x00020000);
  };
  auto piece = [&](int64_t stride, int row) { return ((uint32_t)row * (uint32_t)stride + (uint32_t)st_col) * 2u; };
  if (contig) {
    const __amdgpu_buffer_rsrc_t qr = rsrc(q, qs, n), kr = rsrc(k, ks, nk), vr = rsrc(v, vs, nk);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      if (it >= nblk) break;   // (loads of nothing take their turn too: 231 sequences of up to 31 tokens, 12 heads, 9.9 us
                               // with them, 8.6 without; 256 x 128 positions 22.1 and 20.9)
      tq[it] = __builtin_amdgcn_raw_buffer_load_b128(qr, piece(qs, 32 * it + st_row), 0, 0);
      tk[it] = __builtin_amdgcn_raw_buffer_load_b128(kr, piece(ks, 32 * it + st_row), 0, 0);
      tv[it] = __builtin_amdgcn_raw_buffer_load_b128(vr, piece(vs, 32 * it + st_row), 0, 0);
    }
  } else {
    int64_t gr[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) gr[it] = 32 * it + st_row < n ? rows[start + 32 * it + st_row] : 0;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      tq[it] = tk[it] = tv[it] = u32x4{0u, 0u, 0u, 0u};
      if (32 * it + st_row < n) tq[it] = *reinterpret_cast<const u32x4*>(q + gr[it] * qs + h * kD + st_col);
      if (32 * it + st_row < nk) {
        tk[it] = *reinterpret_cast<const u32x4*>(k + gr[it] * ks + h * kD + st_col);
        tv[it] = *reinterpret_cast<const u32x4*>(v + gr[it] * vs + h * kD + st_col);
      }
    }
  }
  // rows n..32*nblk-1 are staged as zeros; rows >= 32*nblk are never read
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    if (it < nblk) {
      *reinterpret_cast<u32x4*>(&sV[(32 * it + st_row) * kKStride + st_col]) = tq[it];   // Q, pitch kKStride
      *reinterpret_cast<u32x4*>(&sK[(32 * it + st_row) * kKStride + st_col]) = tk[it];
    }
  }
  __syncthreads();
  bf16x8 bq[4];   // Q^T fragments: lane = query column, 8 consecutive d per k-step
#pragma unroll
  for (int s = 0; s < 4; ++s) bq[s] = lds_read8(&sV[qi * kKStride + 16 * s + 8 * g]);
  __syncthreads();   // Q has been read by everyone: sV may now take V
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    if (it < nblk) *reinterpret_cast<u32x4*>(&sV[(32 * it + st_row) * kVStride + st_col]) = tv[it];
  }

  const float cs = scale * kLog2e;
  const float k1 = slopes[h] / scale;   // bias in units of the raw dot product
  float fi = (float)(qi - 4 * g);       // i - j = fi - cj with cj = 32jb + 8*(v/4) + v%4
  asm volatile("" : "+v"(fi));          // keep the distance arithmetic in floating point
  const int lim = nk - 4 * g;           // key of (jb, v) is real iff cj < lim

  // ---- accumulators pre-loaded with the bias, then S^T = K Q^T on top
  f32x16 sacc[4];
  float m = -INFINITY;
  if (wave_active) {
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      if (jb < nblk_k) {
        if (jb == wave) {   // the block that holds the diagonal
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const float cj = (float)(jb * 32 + 8 * (i >> 2) + (i & 3));
            sacc[jb][i] = -k1 * fabsf(fi - cj);
          }
        } else {            // entirely left (j < i) or right (j > i) of the diagonal: |i-j| = +-(fi - cj)
          const float sk = jb < wave ? k1 : -k1;
          const float a = -sk * fi;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const float cj = (float)(jb * 32 + 8 * (i >> 2) + (i & 3));
            sacc[jb][i] = fmaf(cj, sk, a);
          }
        }
        if (jb == nblk_k - 1 && (nk & 31)) {   // ragged end: keys >= nk get -inf
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int cj = jb * 32 + 8 * (i >> 2) + (i & 3);
            sacc[jb][i] = cj >= lim ? -INFINITY : sacc[jb][i];
          }
        }
        const uint16_t* krow = &sK[(jb * 32 + c) * kKStride + 8 * g];
#pragma unroll
        for (int s = 0; s < 4; ++s) sacc[jb] = mfma32(lds_read8(krow + 16 * s), bq[s], sacc[jb]);
      }
    }
    // ---- row maximum of the raw accumulators
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      if (jb < nblk_k) {
#pragma unroll
        for (int i = 0; i < 16; ++i) m = fmaxf(m, sacc[jb][i]);
      }
    }
    m = max_both_halves(m);
  }
  __syncthreads();   // V is in LDS; nobody reads sK any more
  if (!wave_active) return;
  const float mc = m * cs;

  // ---- P^T = exp2(acc*cs - m*cs), row sum, O^T = V^T P^T
  const int tr_i = lane & 15, tr_q = lane >> 4;
  const int tr_row = (tr_i >> 2) + 4 * (tr_q >> 1);
  const int tr_col = 16 * (tr_q & 1) + 4 * (tr_i & 3);
  f32x16 oacc[2];
  float l = 0.f;
#pragma unroll
  for (int jb = 0; jb < 4; ++jb) {
    if (jb < nblk_k) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float p = fast_exp2(fmaf(sacc[jb][i], cs, -mc));
        sacc[jb][i] = p;
        l += p;
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 bp = pack8(sacc[jb][8 * kk + 0], sacc[jb][8 * kk + 1], sacc[jb][8 * kk + 2],
                                sacc[jb][8 * kk + 3], sacc[jb][8 * kk + 4], sacc[jb][8 * kk + 5],
                                sacc[jb][8 * kk + 6], sacc[jb][8 * kk + 7]);
        const uint16_t* vb = &sV[(jb * 32 + 16 * kk + tr_row) * kVStride + tr_col];
#pragma unroll
        for (int db = 0; db < 2; ++db) {
          const s16x4 lo = lds_read_tr4(vb + 32 * db);
          const s16x4 hi = lds_read_tr4(vb + 32 * db + 8 * kVStride);
          if (jb == 0 && kk == 0) {
            const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            oacc[db] = mfma32(join_tr(lo, hi), bp, zero);
          } else {
            oacc[db] = mfma32(join_tr(lo, hi), bp, oacc[db]);
          }
        }
      }
    }
  }
  l = sum_both_halves(l);
  const float inv = 1.f / l;
  if (g == 0 && qi < n) lse[(int64_t)h * T + start + qi] = (mc + __log2f(l)) * kLn2;

  // ---- O^T accumulators (lane = query, 4 consecutive d per register group) -> this wave's 32 rows of
  //      sK -> full rows of 128 bytes, 8 lanes each
  uint16_t* slab = &sK[(32 * wave) * kKStride];
#pragma unroll
  for (int db = 0; db < 2; ++db) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      u32x2 w;
      w[0] = pack_bf16(oacc[db][4 * r + 0] * inv, oacc[db][4 * r + 1] * inv);
      w[1] = pack_bf16(oacc[db][4 * r + 2] * inv, oacc[db][4 * r + 3] * inv);
      *reinterpret_cast<u32x2*>(&slab[c * kKStride + 32 * db + 8 * r + 4 * g]) = w;
    }
  }
  // (same wave wrote and reads the slab: LDS operations of one wave complete in order)
  const int orow = lane >> 3, ocol = (lane & 7) * 8;
  const __amdgpu_buffer_rsrc_t orr = rsrc(o, os, n);
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int row = 8 * it + orow;
    const u32x4 w = *reinterpret_cast<const u32x4*>(&slab[row * kKStride + ocol]);
    if (contig) {
      __builtin_amdgcn_raw_buffer_store_b128(
          w, orr, ((uint32_t)(32 * wave + row) * (uint32_t)os + (uint32_t)ocol) * 2u, 0, 0);
    } else if (32 * wave + row < n) {
      *reinterpret_cast<u32x4*>(o + (int64_t)rows[start + 32 * wave + row] * os + h * kD + ocol) = w;
    }
  }
}

}  // namespace

mb_status launch_attn_fwd_mfma(const AttnShape& s, const void* q, const void* k, const void* v, int64_t qs,
                               int64_t ks, int64_t vs, void* o, int64_t os, float* lse, void* workspace,
                               hipStream_t stream) {
  if (s.B > 65535) return fail(MB_ERR_UNSUPPORTED, "B=%d exceeds 65535 sequences per call", s.B);
  if (s.max_seqlen <= kBlockK) {
    if (s.token_rows)
      hipLaunchKernelGGL(attn_fwd_short_kernel<true>, dim3(s.H, s.B), dim3(256), 0, stream, (const uint16_t*)q,
                         (const uint16_t*)k, (const uint16_t*)v, qs, ks, vs, s.cu_seqlens, s.slopes, s.scale,
                         (uint16_t*)o, os, lse, s.T, s.token_rows, s.misuse, s.key_lens);
    else
      hipLaunchKernelGGL(attn_fwd_short_kernel<false>, dim3(s.H, s.B), dim3(256), 0, stream, (const uint16_t*)q,
                         (const uint16_t*)k, (const uint16_t*)v, qs, ks, vs, s.cu_seqlens, s.slopes, s.scale,
                         (uint16_t*)o, os, lse, s.T, s.token_rows, s.misuse, s.key_lens);
    return check_launch("attn_fwd_short_kernel");
  }
  // any length: plan (8 small workgroups), then one workgroup per plan slot
  const int64_t cap = attn_plan_cap(s.B, s.max_seqlen, s.H);
  if (cap * kPlanXcds >= ((int64_t)1 << 31)) return fail(MB_ERR_UNSUPPORTED, "B * H * max_seqlen is too large for one launch");
  const int32_t* plan = s.plan;
  if (plan == nullptr) {   // no plan of the caller's: build one in the workspace
    const mb_status st = launch_attn_plan(s, static_cast<int32_t*>(workspace), lse, stream);
    if (st != MB_OK) return st;
    plan = static_cast<const int32_t*>(workspace);
  }
  // descriptors: a sequence's rows within 2^31 bytes of its first
  const int64_t widest = ks > vs ? (ks > qs ? ks : qs) : (vs > qs ? vs : qs);
  const int64_t span = (int64_t)s.max_seqlen * widest * 2;
#define MB_LAUNCH_TILED(M)                                                                                         \
  hipLaunchKernelGGL(attn_fwd_tiled_kernel<M>, dim3((unsigned)(cap * kPlanXcds)), dim3(256), 0, stream,            \
                     (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, qs, ks, vs, s.slopes, s.scale,    \
                     (uint16_t*)o, os, lse, s.T, s.token_rows, plan, cap)
  if (span >= ((int64_t)1 << 31)) MB_LAUNCH_TILED(kRowsPerLane);
  else if (s.token_rows) MB_LAUNCH_TILED(kRowsMaybeContiguous);
  else MB_LAUNCH_TILED(kRowsIdentity);
#undef MB_LAUNCH_TILED
  return check_launch("attn_fwd_tiled_kernel");
}

size_t attn_fwd_mfma_workspace_bytes(int B, int max_seqlen, int H) {
  return max_seqlen <= kBlockK ? 0 : attn_plan_bytes(B, max_seqlen, H);
}

size_t attn_plan_workspace_bytes(int B, int max_seqlen, int H) { return attn_plan_bytes(B, max_seqlen, H); }

mb_status launch_attn_plan(const AttnShape& s, int32_t* plan, float* lse, hipStream_t stream) {
  hipLaunchKernelGGL(attn_plan_kernel, dim3(kPlanXcds), dim3(kPlanThreads), 0, stream, s.cu_seqlens, s.key_lens, s.B, s.H,
                     s.max_seqlen, attn_plan_cap(s.B, s.max_seqlen, s.H), plan, s.misuse, lse, s.T);
  return check_launch("attn_plan_kernel");
}

}  // namespace mb
