// Backward ALiBi attention on the matrix cores: bf16, head_dim 64, variable-length packed sequences.
//
// Gradient of sum(O * dO) for the attention of the paper's Eq. 1 (the paper prints no backward; this is
// the standard derivative, with P recomputed from Q, K and the saved row log-sum-exp instead of being
// stored -- the same trade the "FlashAttention" paragraph describes for the forward):
//   Delta_i = dO_i . O_i,  P_ij = exp(S_ij - lse_i),  dV_j = sum_i P_ij dO_i,  dP_ij = dO_i . v_j,
//   dS_ij = P_ij (dP_ij - Delta_i),  dQ_i = scale sum_j dS_ij k_j,  dK_j = scale sum_i dS_ij q_i.
//
// Two kernels for any length, no atomics (results are bitwise reproducible):
//   dq    : one workgroup per (sequence, head, 128 queries); wave w owns 32 queries and streams all keys.
//           Transposed scores S^T = K Q^T (as in the forward) so that dS^T is directly the B operand
//           of dQ^T += K^T dS^T, and lse_i / Delta_i are per-lane scalars.  It runs first and also
//           computes Delta = rowsum(dO * O) of its queries (it holds their dO rows anyway) into [H, T] floats.
//   dkv   : one workgroup per (sequence, head, 128 keys); wave w owns 32 keys and streams all queries.
//           Scores in natural orientation S = Q K^T (queries along accumulator rows, keys along
//           lanes) so that P and dS, rounded to bf16, are directly the B operands of
//           dV^T += dO^T P and dK^T += Q^T dS.  Reads the Delta the first kernel left.
// Masking costs nothing: rows beyond the sequence end are staged as zeros and their lse as +inf
// (P = 0); zero K/V rows make the products with out-of-range keys vanish.
#include "attn_plan.h"
#include "attn_stage.h"
#include "common.h"
#include "mfma_util.h"

#include <type_traits>

namespace mb {
namespace {

constexpr int kD = 64;
constexpr int kTile = 128;
constexpr int kPitch = 72;   // LDS row pitch in bf16 (144 B)

// ------------------------------------------------------------------------------------------------ any length
// Both kernels below stream their second operand in tiles of 64 rows, straight to LDS through a ring of regions
// (attn_stage.h), one barrier per tile.
// Global memory is touched only as full 128-byte rows of one head; fragments and output rows pass
// through LDS.  Which workgroup does what is read from the work plan (attn_plan.h).
constexpr int kTileS = 64;                          // rows of a streamed tile
constexpr int kRegion = 2 * kTileS * kD;            // elements of a region: two operand tiles as attn_stage.h stages them
constexpr int kRing = 4;                            // regions that the tiles of dK/dV go through

// ------------------------------------------------------------------------------------------------ dK, dV
// One workgroup per (sequence, head, 128 keys); wave w owns keys 32w.. and streams all queries.
// What bounds it: a wave issues an instruction every 5 cycles at best, and with 236 registers a SIMD holds two waves, so
// what counts is how few instructions and waits stand between the matrix instructions.  Hence tiles that go straight to LDS,
// three steps ahead, in a layout without bank conflicts (conflicts were a fifth of all LDS cycles), one barrier per 64
// queries, and the exponentials of one block written among the matrix instructions of the blocks before and behind it
// (two waves together take 1240 cycles for 32 matrix instructions of 32 cycles).  16 sequences of 2048 tokens, 16 heads:
// 620 -> 519 us (550 GFLOP); 64 of 64 .. 512 tokens, 12 heads: 90 -> 77 us; 64 of 512 with a key mask: 158 -> 130 us.
// Of the 519 us the loads cost 30, the tables of lse and Delta 15, the vector instructions 60 (each left out in turn).
// Tried: four steps unrolled so that every LDS address is a constant (1100 registers spilled).
//
// kMode (both kernels; see kRowsIdentity .. in common.h): the rows of a sequence whose tokens sit in consecutive
// rows of the activation buffers, spanning fewer than 2^31 bytes, are loaded through descriptors that start at its first row
// and end at its last one: a lane's offset grows by a constant from tile to tile, and rows past the end arrive as zeros
// without a compare.  Otherwise every lane forms its own address (row numbers out of token_rows, if given: StageRows).
constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)

template <int kMode>
__global__ __launch_bounds__(256, 2) void attn_bwd_dkv_kernel(
    const uint16_t* __restrict__ dout, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    const uint16_t* __restrict__ v, const float* __restrict__ lse, const float* __restrict__ delta, int64_t dos,
    int64_t qs, int64_t ks, int64_t vs, const float* __restrict__ slopes,
    float scale, uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int64_t dks, int64_t dvs, int T,
    const int32_t* __restrict__ token_rows, const int32_t* __restrict__ plan, int64_t plan_cap) {
  const int32_t* rows = kMode == kRowsIdentity ? nullptr : token_rows;
  // regions of a Q and a dO tile each; at the start the last two carry this workgroup's K and V rows
  __shared__ __attribute__((aligned(1024))) uint16_t smem[kRing * kRegion];
  __shared__ __attribute__((aligned(16))) float sRaw[3][kRing][kTileS];  // lse and Delta as they come, by tile; unused
  __shared__ __attribute__((aligned(16))) float sL[kRing][3][kTileS];    // -lse / scale (-inf past the end): alone, with the
                                                                         // row's bias left and right of the diagonal
  __shared__ __attribute__((aligned(16))) float sD[kRing][kTileS];       // -Delta
  __shared__ __attribute__((aligned(16))) int32_t sRows[kMode == kRowsIdentity ? 4 : StageRows::kWords];

  int start, n, nk, ktile, h;   // nk <= n: the sequence's first nk tokens are its keys
  if (!plan_fetch(plan, plan_cap, &start, &n, &nk, &ktile, &h)) return;   // this XCD's list is shorter
  const int kv0 = ktile * kTile;   // < n by construction of the plan
  if (kv0 >= nk) {   // a tile of tokens that are no keys (only when the call limits the keys): zero gradient rows
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int j = kv0 + (int)(threadIdx.x >> 3); j < min(kv0 + kTile, n); j += 32) {
      const int64_t gr = tok_row(rows, start + j);
      *reinterpret_cast<u32x4*>(dk + gr * dks + h * kD + (threadIdx.x & 7) * 8) = zero;
      *reinterpret_cast<u32x4*>(dv + gr * dvs + h * kD + (threadIdx.x & 7) * 8) = zero;
    }
    return;
  }
  // first buffer row of the sequence, and whether its tokens sit in consecutive rows
  const int row0 = kMode == kRowsMaybeContiguous ? __builtin_amdgcn_readfirstlane(rows[start]) : start;
  const bool contig =
      kMode == kRowsIdentity ||
      (kMode == kRowsMaybeContiguous && __builtin_amdgcn_readfirstlane(rows[start + n - 1]) - row0 == n - 1);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps per-wave branches scalar
  const int c = lane & 31, g = lane >> 5;
  const int kw = kv0 + 32 * wave;
  const bool wave_active = kw < nk;           // tokens at and beyond nk are no keys: their dK, dV are zero
  const int kj = kw + c;                      // this lane's key
  const int kblk = (kv0 >> 5) + wave;         // index of this wave's block of 32 keys
  const int ntiles = (n + kTileS - 1) / kTileS;
  const float cs = scale * kLog2e;
  const float k1 = slopes[h] / scale, inv_scale = 1.f / scale;

  // ---- loads: this wave's K and V rows, then its share of the Q / dO tiles
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint16_t*)smem);
  const StageRows where(rows, start, n, sRows, wave);
  int first_row[4];   // without descriptors: rows of the wave's share of two tiles
  if (!contig) {
    int own_row[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) own_row[j] = stage_row_of(rows, start, kw + 8 * j + (lane >> 3), nk);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      first_row[j] = stage_row_of(rows, start, (j >> 1) * kTileS + 8 * (wave + 4 * (j & 1)) + (lane >> 3), n);
    rows_known(own_row);
    rows_known(first_row);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t at = lds0 + (2 * kRegion + (32 * wave + 8 * j) * kD) * 2;
      const bool there = kw + 8 * j + (lane >> 3) < nk;
      stage_each(at, stage_address(k + h * kD, ks, own_row[j], there, stage_piece(lane, j & 1) * 16));
      stage_each(at + kRegion * 2, stage_address(v + h * kD, vs, own_row[j], there, stage_piece(lane, j & 1) * 16));
    }
  } else {
    const u32x4 k_rsrc = stage_rsrc(k + row0 * ks + h * kD, ks, nk), v_rsrc = stage_rsrc(v + row0 * vs + h * kD, vs, nk);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t at = lds0 + (2 * kRegion + (32 * wave + 8 * j) * kD) * 2, row = kw + 8 * j;
      stage_rows(at, stage_lane_off(lane, j & 1, ks) + row * (uint32_t)ks * 2u, k_rsrc);
      stage_rows(at + kRegion * 2, stage_lane_off(lane, j & 1, vs) + row * (uint32_t)vs * 2u, v_rsrc);
    }
  }
  const u32x4 q_rsrc = stage_rsrc(q + row0 * qs + h * kD, qs, n), g_rsrc = stage_rsrc(dout + row0 * dos + h * kD, dos, n);
  // the wave's first 8 rows of the tile to load next; its second 8 rows lie 32 behind them (without descriptors: the lane's
  // place among the row numbers, and inside a row)
  uint32_t q_off = stage_lane_off(lane, wave & 1, qs) + 8u * wave * (uint32_t)qs * 2u;
  uint32_t g_off = stage_lane_off(lane, wave & 1, dos) + 8u * wave * (uint32_t)dos * 2u;
  if (!contig) {
    q_off = StageRows::lane_off(wave, lane);
    g_off = stage_piece(lane, wave & 1) * 16;
  }
  constexpr int kRowLoads = 4;   // loads per wave and tile
  auto place = [&](int region, int j) {   // of the j-th of them: Q and dO rows by turns
    return lds0 + (uint32_t)(region * kRegion + ((j & 1) == 0 ? 0 : kTileS * kD) + 8 * (wave + 4 * (j >> 1)) * kD) * 2;
  };
  auto issue_row = [&](int region, int j) {   // with descriptors; the tiles are taken in order
    const bool is_q = (j & 1) == 0;
    uint32_t& off = is_q ? q_off : g_off;
    stage_rows(place(region, j), off, is_q ? q_rsrc : g_rsrc);
    off += 64u * (uint32_t)(is_q ? qs : dos);
  };
  auto issue_each = [&](int t, int region, const int* row) {   // without: tile t, whose rows are `row`
#pragma unroll
    for (int j = 0; j < kRowLoads; ++j) {
      const bool is_q = (j & 1) == 0;
      stage_each(place(region, j), stage_address((is_q ? q : dout) + h * kD, is_q ? qs : dos, row[j >> 1],
                                                 t * kTileS + 8 * (wave + 4 * (j >> 1)) + (lane >> 3) < n, g_off));
    }
  };
  // Requests tile t, and before it (without descriptors) the row numbers of tile `ahead`.
  auto issue_rows = [&](int t, int region, int ahead) {
    if (contig) {
#pragma unroll
      for (int j = 0; j < kRowLoads; ++j) issue_row(region, j);
    } else {
      const int row[2] = {where.get(t, 0, lane), where.get(t, 1, lane)};
      if (ahead > 0) where.request(ahead, q_off);
      issue_each(t, region, row);
    }
  };
  // lse and Delta of a tile: the first wave brings one and the second the other (the other waves' loads, which keep the
  // number of loads the same, read nothing).
  const u32x4 raw_rsrc = stage_rsrc_bytes((wave == 0 ? lse : delta) + ((int64_t)h * T + start), wave < 2 ? (uint32_t)n * 4u : 0u);
  const uint32_t raw0_at = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) float*)&sRaw[0][0][0]) +
                           min(wave, 2) * (kRing * kTileS * 4);
  auto issue_raw = [&](int t, int region) {   // of tile t
    const uint32_t at = raw0_at + region * (kTileS * 4);
    stage_words(at, (uint32_t)(t * kTileS + lane) * 4u, raw_rsrc);
  };
  auto store_tables = [&](int t, int to, float raw) {   // of tile t; `raw`: this lane's lse or Delta
    if (wave == 0) {
      const float l = t * kTileS + lane < n ? -raw * inv_scale : -INFINITY;
      sL[to][0][lane] = l;
      sL[to][1][lane] = fmaf((float)lane, k1, l);
      sL[to][2][lane] = fmaf((float)lane, -k1, l);
    } else if (wave == 1) {
      sD[to][lane] = t * kTileS + lane < n ? -raw : 0.f;
    }
  };
  auto first_raw = [&](int t) {
    const int i = min(t * kTileS + lane, n - 1);
    return (wave == 0 ? lse : delta)[(int64_t)h * T + start + i];
  };
  if (contig) {
    issue_rows(0, 0, 0);
  } else {
    issue_each(0, 0, first_row);
    where.request(2, q_off);
    where.request(3, q_off);
  }
  issue_raw(2, 2);
  issue_raw(3, 3);
  const float raw0 = first_raw(0), raw1 = first_raw(1);
  if (contig) issue_rows(1, 1, 0);
  else issue_each(1, 1, first_row + 2);
  store_tables(0, 0, raw0);
  store_tables(1, 1, raw1);

  // ---- places in a region (bytes): rows for S and dP, transposed patches for dV and dK
  uint32_t row_at[4], tr_at[2][2];
  stage_row_places(lane, row_at);
  stage_tr_places(lane, tr_at);
  const char* const lds = reinterpret_cast<const char*>(smem);
  // the wave's K^T, V^T fragments (B operands): lane = key column, 8 consecutive d per k-step
  bf16x8 bk[4], bv[4];
  staged_barrier<0>();
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    bk[s] = lds_read8(reinterpret_cast<const uint16_t*>(lds + row_at[s] + (2 * kRegion + 32 * wave * kD) * 2));
    bv[s] = lds_read8(reinterpret_cast<const uint16_t*>(lds + row_at[s] + (3 * kRegion + 32 * wave * kD) * 2));
  }

  f32x16 dkacc[2], dvacc[2];   // dK^T, dV^T: d along accumulator rows (two blocks of 32), keys along lanes
#pragma unroll
  for (int i = 0; i < 16; ++i) { dkacc[0][i] = dkacc[1][i] = dvacc[0][i] = dvacc[1][i] = 0.f; }

  // Blocks of 32 queries go through three stages: (1) S and dP, 8 matrix instructions; (2) P = exp2(S c + off) and
  // dS = P dP on the vector unit; (3) dV += dO^T P and dK += Q^T dS, 8 matrix instructions.  The S accumulator
  // starts from -lse_i / scale plus the query's part of the bias (off the diagonal block |i-j| is linear in i and j; one of
  // two tables in LDS, for either side), the key's part is the exponent's constant; the dP accumulator starts from -Delta_i.
  // Rows past the sequence end are staged as zeros with lse = +inf, which makes their P and dS exact zeros.
  // A slot runs stage 2 of block b among the matrix instructions of stage 3 of block b - 1 and stage 1 of block b + 1: 16
  // groups of one matrix instruction, the fragment reads of the matrix instruction four groups later and the vector
  // instructions of one accumulator register, kept in this order.
  struct Block {
    f32x16 s, p;         // S, dP; then P, dS
  };
  struct Packed {
    uint32_t p[8], s[8];   // P and dS as operands
  };
  auto operand = [](const uint32_t(&w)[8], int kk) {
    return as_bf16x8(u32x4{w[4 * kk], w[4 * kk + 1], w[4 * kk + 2], w[4 * kk + 3]});
  };
  bf16x8 f[16];   // A operands by group
  // group -> what its matrix instruction is: stage 3 (0: dV, 1: dK; db; kk) or stage 1 (0: S, 1: dP; k-step)
  constexpr int kStage3[16] = {1, 1, 1, 1, 0, 0, 1, 0, 0, 1, 0, 0, 0, 0, 1, 1};
  constexpr int kWhat[16] = {0, 1, 0, 1, 0, 1, 0, 0, 1, 1, 0, 1, 0, 1, 0, 1};
  constexpr int kDb[16] = {0, 0, 1, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 1, 1};
  constexpr int kStep[16] = {0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 2, 2, 3, 3, 1, 1};   // kk or k-step
  struct Places {
    uint32_t a[4];   // in a region: what the lane reads of Q rows by k-step, or of Q patches by d block and half
  };
  auto places_row = [&](uint32_t region_bytes) {
    return Places{{row_at[0] + region_bytes, row_at[1] + region_bytes, row_at[2] + region_bytes, row_at[3] + region_bytes}};
  };
  auto places_tr = [&](uint32_t region_bytes) {
    return Places{{tr_at[0][0] + region_bytes, tr_at[0][1] + region_bytes, tr_at[1][0] + region_bytes,
                   tr_at[1][1] + region_bytes}};
  };
  auto read_tr = [&](const Places& at, int ib, int what, int db, int kk) {   // dO^T or Q^T of the tile's block ib
    const uint32_t off = (32 * ib + 16 * kk + (what == 0 ? kTileS : 0)) * kD * 2;
    return join_tr(lds_read_tr4(reinterpret_cast<const uint16_t*>(lds + at.a[2 * db] + off)),
                   lds_read_tr4(reinterpret_cast<const uint16_t*>(lds + at.a[2 * db + 1] + off)));
  };
  auto read_row = [&](const Places& at, int ib, int what, int s) {
    return lds_read8(reinterpret_cast<const uint16_t*>(lds + at.a[s] + (32 * ib + (what == 0 ? 0 : kTileS)) * kD * 2));
  };
  auto start_row = [&](Block& b, int what, int r, const float* table, const float* dl) {   // start values of S and dP
    const float4 x = *reinterpret_cast<const float4*>((what == 0 ? table : dl) + 8 * r + 4 * g);
    f32x16& a = what == 0 ? b.s : b.p;
    a[4 * r] = x.x; a[4 * r + 1] = x.y; a[4 * r + 2] = x.z; a[4 * r + 3] = x.w;
  };
  auto table_of = [&](int region, int qb, int ib) -> const float* {   // of query block qb, block ib of tile `region`
    return &sL[0][qb == kblk ? 0 : qb < kblk ? 1 : 2][0] + region * (3 * kTileS) + 32 * ib;
  };
  const float k1cs = k1 * cs, kjf = (float)kj;
  // stage 2 of block qb in `b` -> `to`; stage 3 of the block before it (its LDS place `tr`, its operands `from`); stage 1
  // of the block behind it (`row`, `nx`).  `i0f`: first query of block qb's tile.  `tr_next`: the place that stage 3 reads in the next slot.
  auto slot = [&](auto with3, auto with1, Block& b, int qb, float i0f, Packed& to, const Places& tr, int tr_ib,
                  const Packed& from, const Places& row, int row_ib, Block& nx, const float* table, const float* dl,
                  const Places& tr_next, int tr_next_ib, auto load) {
    constexpr bool k3 = decltype(with3)::value, k1st = decltype(with1)::value;
    if (qb == kblk) {   // block with the diagonal
      float d0 = (float)(32 * qb - kj + 4 * g);
      asm volatile("" : "+v"(d0));   // (else the 16 distances are kept in registers all the time)
#pragma unroll
      for (int i = 0; i < 16; ++i) b.s[i] = fmaf(-k1, fabsf(d0 + (float)(8 * (i >> 2) + (i & 3))), b.s[i]);
    }
    const float off = (i0f - kjf) * (qb == kblk ? 0.f : qb < kblk ? k1cs : -k1cs);
    // (the empty assembly keeps the vector instructions in this slot: the compiler would move them to where their results
    // are used, behind the next slot's branch)
    auto put = [](uint32_t& to, float lo, float hi) {
      to = pack_bf16(lo, hi);
      asm volatile("" : "+v"(to));
    };
    auto second = [&](int i) {   // dS of register i, and the operand words that are complete
      b.p[i] = b.s[i] * b.p[i];
      if (i & 1) put(to.p[i >> 1], b.s[i - 1], b.s[i]);
      if (i > 0 && !(i & 1)) put(to.s[(i >> 1) - 1], b.p[i - 2], b.p[i - 1]);
    };
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      if (k1st && x < 4) {
        start_row(nx, 0, x, table, dl);
        start_row(nx, 1, x, table, dl);
      }
      if (x < 12) {
        const int y = x + 4;
        if (kStage3[y] ? k3 : k1st)
          f[y] = kStage3[y] ? read_tr(tr, tr_ib, kWhat[y], kDb[y], kStep[y]) : read_row(row, row_ib, kWhat[y], kStep[y]);
      } else {
        f[x - 12] = read_tr(tr_next, tr_next_ib, kWhat[x - 12], kDb[x - 12], kStep[x - 12]);
      }
      if (kStage3[x]) {
        if (k3) {
          f32x16& acc = kWhat[x] == 0 ? dvacc[kDb[x]] : dkacc[kDb[x]];
          acc = mfma32(f[x], operand(kWhat[x] == 0 ? from.p : from.s, kStep[x]), acc);
        }
      } else if (k1st) {
        f32x16& acc = kWhat[x] == 0 ? nx.s : nx.p;
        acc = mfma32(f[x], kWhat[x] == 0 ? bk[kStep[x]] : bv[kStep[x]], acc);
      }
      b.s[x] = fast_exp2(fmaf(b.s[x], cs, off));
      if (x > 0) second(x - 1);
      if ((x & 3) == 1) load(x >> 2);
      if (x == 15) {
        second(15);
        put(to.s[7], b.p[14], b.p[15]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto none = [](int) {};
  using Yes = std::true_type;
  using No = std::false_type;
  constexpr uint32_t kRegionBytes = kRegion * 2;

  Block b0, b1;
  Packed w0, w1;
  if (wave_active) {   // stage 1 of block 0, stage 2 of it beside stage 1 of block 1
    const float* table = table_of(0, 0, 0);
    const Places tr = places_tr(0), row = places_row(0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      start_row(b0, 0, r, table, sD[0]);
      start_row(b0, 1, r, table, sD[0]);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      b0.s = mfma32(read_row(row, 0, 0, s), bk[s], b0.s);
      b0.p = mfma32(read_row(row, 0, 1, s), bv[s], b0.p);
    }
    slot(No{}, Yes{}, b0, 0, 0.f, w0, tr, 0, w1, row, 1, b1, table_of(0, 1, 1), sD[0] + 32, tr, 0, none);
  }
  // Step t: what the step before the last one requested has arrived (tile t + 1, and lse and Delta of tile t + 2, which
  // become tables here), and tile t + 3 is requested.  Loads past the end are issued too: their number stays the same.
  if (!wave_active) {   // (a loop of its own: inside the other one the accumulators would be copied in every step)
    for (int t = 0; t + 1 < ntiles; ++t) {
      staged_barrier<kRowLoads + 1>();
      if (t == 0) issue_rows(2, 2, 0);
      issue_rows(t + 3, (t + 3) & (kRing - 1), t + 4);
      issue_raw(t + 4, t & (kRing - 1));
      if (wave < 2) store_tables(t + 2, (t + 2) & (kRing - 1), sRaw[wave][(t + 2) & (kRing - 1)][lane]);
    }
    staged_barrier<0>();
    // tokens that are no keys (only when the call limits the keys): zero gradient rows
    for (int row = lane >> 3; row < 32 && kw + row < n; row += 8) {
      const u32x4 zero = {0u, 0u, 0u, 0u};
      const int64_t gr = tok_row(rows, start + kw + row);
      *reinterpret_cast<u32x4*>(dk + gr * dks + h * kD + (lane & 7) * 8) = zero;
      *reinterpret_cast<u32x4*>(dv + gr * dvs + h * kD + (lane & 7) * 8) = zero;
    }
    return;
  }
  float i0f = 0.f;   // first query of tile t
#pragma unroll 1
  for (int t = 0; t + 1 < ntiles; ++t) {
    const int here = t & (kRing - 1), next = (t + 1) & (kRing - 1), after = (t + 2) & (kRing - 1), to = (t + 3) & (kRing - 1);
    staged_barrier<kRowLoads + 1>();
    if (t == 0) issue_rows(2, 2, 0);   // (the region of the K rows)
    // Loads in one go block the waves for 300 to 500 cycles, so they are spread over the step's matrix instructions (not
    // the ones with an address per lane: there are no registers left for those).
    if (!contig) issue_rows(t + 3, to, t + 4);
    const Places tr = places_tr(here * kRegionBytes), row = places_row(next * kRegionBytes);
    float raw = 0.f;
    auto first_half = [&](int j) {
      if ((j == 0 || j == 2) && contig) issue_row(to, j >> 1);
      if (j == 3) issue_raw(t + 4, here);
    };
    auto second_half = [&](int j) {
      if ((j == 0 || j == 2) && contig) issue_row(to, 2 + (j >> 1));
      if (j == 1 && wave < 2) raw = sRaw[wave][after][lane];
      if (j == 3 && wave < 2) store_tables(t + 2, after, raw);
    };
    slot(Yes{}, Yes{}, b1, 2 * t + 1, i0f, w1, tr, 0, w0, row, 0, b0, table_of(next, 2 * t + 2, 0), sD[next], tr, 1,
         first_half);
    i0f += (float)kTileS;
    slot(Yes{}, Yes{}, b0, 2 * t + 2, i0f, w0, tr, 1, w1, row, 1, b1, table_of(next, 2 * t + 3, 1), sD[next] + 32,
         places_tr(next * kRegionBytes), 0, second_half);
  }
  {   // the last tile's second block
    const Places tr = places_tr(((ntiles - 1) & (kRing - 1)) * kRegionBytes);
    slot(Yes{}, No{}, b1, 2 * ntiles - 1, i0f, w1, tr, 0, w0, tr, 0, b0, nullptr, nullptr, tr, 1, none);
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      if (!kStage3[x]) continue;
      if (x >= 4) f[x] = read_tr(tr, 1, kWhat[x], kDb[x], kStep[x]);
      f32x16& acc = kWhat[x] == 0 ? dvacc[kDb[x]] : dkacc[kDb[x]];
      acc = mfma32(f[x], operand(kWhat[x] == 0 ? w1.p : w1.s, kStep[x]), acc);
    }
  }
  staged_barrier<0>();   // the regions are free: they now carry the output rows
  const int orow = lane >> 3, ocol = (lane & 7) * 8;
  uint16_t* slab = &smem[(32 * wave) * kPitch];   // 32 rows private to this wave
  auto store_rows = [&](const f32x16(&acc)[2], float mul, uint16_t* __restrict__ out, int64_t stride) {
#pragma unroll
    for (int db = 0; db < 2; ++db) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        u32x2 w;
        w[0] = pack_bf16(acc[db][4 * r + 0] * mul, acc[db][4 * r + 1] * mul);
        w[1] = pack_bf16(acc[db][4 * r + 2] * mul, acc[db][4 * r + 3] * mul);
        *reinterpret_cast<u32x2*>(&slab[c * kPitch + 32 * db + 8 * r + 4 * g]) = w;
      }
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int row = 8 * it + orow;
      u32x4 w = *reinterpret_cast<const u32x4*>(&slab[row * kPitch + ocol]);
      if (kw + row >= nk) w = u32x4{0u, 0u, 0u, 0u};   // a token that is no key
      if (kw + row < n) *reinterpret_cast<u32x4*>(out + tok_row(rows, start + kw + row) * stride + h * kD + ocol) = w;
    }
  };
  store_rows(dkacc, scale, dk, dks);
  store_rows(dvacc, 1.f, dv, dvs);
}

// ------------------------------------------------------------------------------------------------ dQ
// One workgroup per (sequence, head, 128 queries); wave w owns queries 32w.. and streams all keys.
// At most 168 registers, so that three workgroups share a compute unit; the tiles arrive two steps ahead.
// Bound by vector issue as the forward is: 57 vector instructions and 16 exponentials a block of 32 keys, beside 12 matrix
// instructions.  -Delta is the start value of dP out of registers that hold it 16 times (16 instructions a block less).  With
// tiles through registers, before and after: 16 x 2048 tokens, 16 heads 455 and 400 us; 64 x 64 .. 512 tokens, 12 heads 70
// and 62 us; 64 x 512 with a key mask 112 and 102 us.
template <int kMode>
__global__ __launch_bounds__(256, 3) void attn_bwd_dq_kernel(
    const uint16_t* __restrict__ dout, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    const uint16_t* __restrict__ v, const uint16_t* __restrict__ o, const float* __restrict__ lse,
    float* __restrict__ delta, int64_t dos, int64_t qs, int64_t ks, int64_t vs, int64_t os,
    const float* __restrict__ slopes, float scale, uint16_t* __restrict__ dq, int64_t dqs, int T,
    const int32_t* __restrict__ token_rows, const int32_t* __restrict__ plan, int64_t plan_cap) {
  const int32_t* rows = kMode == kRowsIdentity ? nullptr : token_rows;
  __shared__ __attribute__((aligned(1024))) uint16_t smem[3 * kRegion];   // regions of a K and a V tile each
  __shared__ __attribute__((aligned(16))) float sDelta[kTile];       // -Delta of this workgroup's queries
  __shared__ __attribute__((aligned(16))) int32_t sRows[kMode == kRowsIdentity ? 4 : StageRows::kWords];

  int start, n, nk, qtile, h;   // nk <= n: the sequence's first nk tokens are its keys
  if (!plan_fetch(plan, plan_cap, &start, &n, &nk, &qtile, &h)) return;
  const int q0 = qtile * kTile;
  const int row0 = kMode == kRowsMaybeContiguous ? __builtin_amdgcn_readfirstlane(rows[start]) : start;
  const bool contig =
      kMode == kRowsIdentity ||
      (kMode == kRowsMaybeContiguous && __builtin_amdgcn_readfirstlane(rows[start + n - 1]) - row0 == n - 1);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, g = lane >> 5;
  const int qw = q0 + 32 * wave;
  const bool wave_active = qw < n;
  const int qi = qw + c;
  const bool q_ok = wave_active && qi < n;
  const int qblk = (q0 >> 5) + wave;
  const int ntiles = (nk + kTileS - 1) / kTileS;
  const int st_row = tid >> 3, st_col = (tid & 7) * 8;
  const float cs = scale * kLog2e;
  const float k1 = slopes[h] / scale;

  // ---- loads: this wave's Q and dO rows, then its share of the K / V tiles
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint16_t*)smem);
  const StageRows where(rows, start, nk, sRows, wave);
  int first_row[2], o_row[4];   // without descriptors: rows of the wave's share of the first tile, and of O
  if (!contig) {
    int own_row[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) own_row[j] = stage_row_of(rows, start, qw + 8 * j + (lane >> 3), n);
#pragma unroll
    for (int j = 0; j < 4; ++j) o_row[j] = stage_row_of(rows, start, q0 + 32 * j + st_row, n);
#pragma unroll
    for (int j = 0; j < 2; ++j) first_row[j] = stage_row_of(rows, start, 8 * (wave + 4 * j) + (lane >> 3), nk);
    rows_known(own_row);
    rows_known(o_row);
    rows_known(first_row);
    where.request(1, StageRows::lane_off(wave, lane));
    where.request(2, StageRows::lane_off(wave, lane));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t at = lds0 + (kRegion + (32 * wave + 8 * j) * kD) * 2;
      const bool there = qw + 8 * j + (lane >> 3) < n;
      stage_each(at, stage_address(q + h * kD, qs, own_row[j], there, stage_piece(lane, j & 1) * 16));
      stage_each(at + kRegion * 2, stage_address(dout + h * kD, dos, own_row[j], there, stage_piece(lane, j & 1) * 16));
    }
  } else {
    const u32x4 q_rsrc = stage_rsrc(q + row0 * qs + h * kD, qs, n), g_rsrc = stage_rsrc(dout + row0 * dos + h * kD, dos, n);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t at = lds0 + (kRegion + (32 * wave + 8 * j) * kD) * 2, row = qw + 8 * j;
      stage_rows(at, stage_lane_off(lane, j & 1, qs) + row * (uint32_t)qs * 2u, q_rsrc);
      stage_rows(at + kRegion * 2, stage_lane_off(lane, j & 1, dos) + row * (uint32_t)dos * 2u, g_rsrc);
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
    return lds0 + (uint32_t)(region * kRegion + ((j & 1) == 0 ? 0 : kTileS * kD) + 8 * (wave + 4 * (j >> 1)) * kD) * 2;
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
                                                 t * kTileS + 8 * (wave + 4 * (j >> 1)) + (lane >> 3) < nk, v_off));
    }
  };
  // Requests tile t, and before it (without descriptors) the row numbers of the tile behind it.
  auto issue_tile = [&](int t, int region) {
    if (contig) {
#pragma unroll
      for (int j = 0; j < kRowLoads; ++j) issue_row(region, j);
    } else {
      const int row[2] = {where.get(t, 0, lane), where.get(t, 1, lane)};
      if (t > 1) where.request(t + 1, k_off);   // (those of tiles 1 and 2 are here)
      issue_each(t, region, row);
    }
  };
  if (contig) issue_tile(0, 0);
  else issue_each(0, 0, first_row);

  // ---- places in a region (bytes): K and V rows, transposed patches of K
  const char* const lds = reinterpret_cast<const char*>(smem);
  uint32_t row_at[4], tr_at[2][2];
  stage_row_places(lane, row_at);
  stage_tr_places(lane, tr_at);
  // The O rows only serve Delta_i = dO_i . O_i (8 lanes per row, 8 elements each), kept in LDS for this kernel and written to
  // [H, T] for the dK/dV kernel.
  {
    u32x4 to[4];
    // (row st_row + 32 it of the workgroup: as staged)
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      to[it] = u32x4{0u, 0u, 0u, 0u};
      const int i = q0 + 32 * it + st_row;
      if (i < n) to[it] = *reinterpret_cast<const u32x4*>(o + (contig ? (int64_t)(row0 + i) : (int64_t)o_row[it]) * os + h * kD + st_col);
    }
    staged_barrier<0>();
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int row = 32 * it + st_row;
      const u32x4 tg = *reinterpret_cast<const u32x4*>(
          lds + (2 * kRegion + row * kD) * 2 + (((st_col >> 3) ^ stage_swizzle(row)) * 16));
      float acc = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc = fmaf(__uint_as_float(tg[e] << 16), __uint_as_float(to[it][e] << 16), acc);
        acc = fmaf(__uint_as_float(tg[e] & 0xffff0000u), __uint_as_float(to[it][e] & 0xffff0000u), acc);
      }
      acc += __shfl_xor(acc, 1, 64);
      acc += __shfl_xor(acc, 2, 64);
      acc += __shfl_xor(acc, 4, 64);
      if ((tid & 7) == 0) {
        sDelta[row] = -acc;
        if (q0 + row < n) delta[(int64_t)h * T + start + q0 + row] = acc;
      }
    }
  }
  bf16x8 bq[4], bg[4];   // Q^T, dO^T fragments of the wave's own rows
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    bq[s] = lds_read8(reinterpret_cast<const uint16_t*>(lds + row_at[s] + (kRegion + 32 * wave * kD) * 2));
    bg[s] = lds_read8(reinterpret_cast<const uint16_t*>(lds + row_at[s] + (2 * kRegion + 32 * wave * kD) * 2));
  }
  staged_barrier<0>();   // Delta is in LDS, and nobody reads Q or dO any more
  issue_tile(1, 1);
  const float nlse2 = q_ok ? -lse[(int64_t)h * T + start + qi] * kLog2e : -INFINITY;   // -inf: P = 0
  f32x16 ndlt;               // -Delta of the lane's query: the start value of dP
  {
    const float d = q_ok ? sDelta[32 * wave + c] : 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) ndlt[i] = d;
    asm volatile("" : "+v"(ndlt));   // (16 registers, which save 16 instructions in every block)
  }

  f32x16 dqacc[2];   // dQ^T: d along accumulator rows, queries along lanes
#pragma unroll
  for (int i = 0; i < 16; ++i) { dqacc[0][i] = 0.f; dqacc[1][i] = 0.f; }
  f32x16 row_bias;      // (m_h / scale) * (accumulator row) left of the diagonal, its negative right of it
#pragma unroll
  for (int i = 0; i < 16; ++i) row_bias[i] = k1 * (float)(8 * (i >> 2) + (i & 3));
  // in vector registers, where there is room: the compiler would keep it in scalar ones and copy it each time
  if (kMode == kRowsIdentity) asm volatile("" : "+v"(row_bias));

  // One block of 32 keys (rows 32jb.. of the staged tile) against this wave's queries, transposed
  // orientation: S^T = K Q^T (bias/scale in the C operand), dP^T = V dO^T (- Delta pre-loaded).  The code
  // that accumulates dQ exists once with no branch around it; a ragged last tile only zeroes the dS of
  // the keys that do not exist.
  auto kblock = [&](const uint32_t(&ra)[4], const uint32_t(&ta)[2][2], int j0, int jb, int rem) {
    auto read_row = [&](int what, int s) {   // 0: K, 1: V
      return lds_read8(reinterpret_cast<const uint16_t*>(lds + ra[s] + (32 * jb + what * kTileS) * (kD * 2)));
    };
    float fi = (float)(qi - j0 - 4 * g);   // i - j = fi - cj with cj = 32jb + 8*(v/4) + v%4
    asm volatile("" : "+v"(fi));
    f32x16 sacc, pacc;
    const int kb = (j0 >> 5) + jb;
    const bf16x8 ak0 = read_row(0, 0);
    float e0 = nlse2;   // the exponent's constant
    if (kb == qblk) {
      f32x16 diag;
#pragma unroll
      for (int i = 0; i < 16; ++i) diag[i] = -k1 * fabsf(fi - (float)(jb * 32 + 8 * (i >> 2) + (i & 3)));
      sacc = mfma32(ak0, bq[0], diag);
#pragma unroll
      for (int i = 0; i < 16; ++i) row_bias[i] = -row_bias[i];
    } else {   // (see the forward: the bias per accumulator row is the C operand, the bias per lane goes to the exponent)
      sacc = mfma32(ak0, bq[0], row_bias);
      e0 = fmaf((kb < qblk ? -k1 : k1) * (fi - (float)(32 * jb)), cs, e0);
    }
    pacc = mfma32(read_row(1, 0), bg[0], ndlt);
#pragma unroll
    for (int s = 1; s < 4; ++s) {
      sacc = mfma32(read_row(0, s), bq[s], sacc);
      pacc = mfma32(read_row(1, s), bg[s], pacc);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) pacc[i] = fast_exp2(fmaf(sacc[i], cs, e0)) * pacc[i];
    if (rem < kTileS) {
      // a key past the sequence end has a zero K row, but its p may overflow (its score was never part
      // of lse): force the product with that zero row to be 0, not inf * 0
      const int lim = rem - 4 * g;
#pragma unroll
      for (int i = 0; i < 16; ++i) pacc[i] = (32 * jb + 8 * (i >> 2) + (i & 3)) >= lim ? 0.f : pacc[i];
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const bf16x8 bs = pack8(pacc[8 * kk + 0], pacc[8 * kk + 1], pacc[8 * kk + 2], pacc[8 * kk + 3],
                              pacc[8 * kk + 4], pacc[8 * kk + 5], pacc[8 * kk + 6], pacc[8 * kk + 7]);
      const uint32_t at = (32 * jb + 16 * kk) * kD * 2;
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        const bf16x8 ak = join_tr(lds_read_tr4(reinterpret_cast<const uint16_t*>(lds + ta[db][0] + at)),
                                  lds_read_tr4(reinterpret_cast<const uint16_t*>(lds + ta[db][1] + at)));
        dqacc[db] = mfma32(ak, bs, dqacc[db]);
      }
    }
  };

  // Step jt: tile jt has arrived, the next one is on its way and the one behind that is requested.  Loads past the end are
  // issued too: their number stays the same.
  int region = 0;
  if (!wave_active) {   // (a loop of its own: inside the other one the accumulators would be copied in every step)
    for (int jt = 0; jt < ntiles; ++jt) {
      staged_barrier<kRowLoads>();
      issue_tile(jt + 2, region == 0 ? 2 : region - 1);
      region = region == 2 ? 0 : region + 1;
    }
    staged_barrier<0>();
    return;
  }
#pragma unroll 1
  for (int jt = 0; jt < ntiles; ++jt) {
    const int j0 = jt * kTileS, to = region == 0 ? 2 : region - 1;   // of tile jt + 2: the region of tile jt - 1
    staged_barrier<kRowLoads>();
    if (!contig) issue_tile(jt + 2, to);
    uint32_t ra[4], ta[2][2];
    // (k-step s reads piece (2 s + g) ^ swizzle: the first one's place with bits 5 and 6 exchanged, so that one register and
    // not four is kept from step to step: with four there were two too many)
#pragma unroll
    for (int s = 0; s < 4; ++s) ra[s] = (row_at[0] + region * (kRegion * 2)) ^ (32 * s);
#pragma unroll
    for (int s = 0; s < 4; ++s) ta[s >> 1][s & 1] = tr_at[s >> 1][s & 1] + region * (kRegion * 2);
    const int rem = nk - j0;
    if (contig) {
      issue_row(to, 0);
      issue_row(to, 1);
    }
    kblock(ra, ta, j0, 0, rem);
    if (contig) {
      issue_row(to, 2);
      issue_row(to, 3);
    }
    kblock(ra, ta, j0, 1, rem);
    region = region == 2 ? 0 : region + 1;
  }
  staged_barrier<0>();

  uint16_t* slab = &smem[(32 * wave) * kPitch];
#pragma unroll
  for (int db = 0; db < 2; ++db) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      u32x2 w;
      w[0] = pack_bf16(dqacc[db][4 * r + 0] * scale, dqacc[db][4 * r + 1] * scale);
      w[1] = pack_bf16(dqacc[db][4 * r + 2] * scale, dqacc[db][4 * r + 3] * scale);
      *reinterpret_cast<u32x2*>(&slab[c * kPitch + 32 * db + 8 * r + 4 * g]) = w;
    }
  }
  const int orow = lane >> 3, ocol = (lane & 7) * 8;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int row = 8 * it + orow;
    const u32x4 w = *reinterpret_cast<const u32x4*>(&slab[row * kPitch + ocol]);
    if (qw + row < n) *reinterpret_cast<u32x4*>(dq + tok_row(rows, start + qw + row) * dqs + h * kD + ocol) = w;
  }
}

// ------------------------------------------------------------------------------------------------ fused, n <= 128
// Whole backward of one (sequence, head) with at most 128 tokens in one workgroup: every input is read
// from HBM once and every output written once, always as full 128-byte rows shared by 8 lanes; the
// fragment layouts of the matrix cores are produced by passing through LDS.
//   phase 0  K, V, Q, dO rows -> LDS (K and V into the dS buffer, which is idle until phase 1), Delta = rowsum(dO * O)
//            and -lse -> LDS; one barrier; each wave takes the K^T, V^T fragments of its own 32 keys into registers.
//   phase 1  wave w owns keys 32w..: for every block of 32 queries, S = Q K^T, dP = dO V^T, P, dS in
//            registers; dV^T += dO^T P, dK^T += Q^T dS; dS (bf16) is also written to LDS as [key][query].
//   phase 2  dK, dV leave through the (now free) dO tile; the K registers go back to LDS over the Q
//            tile; wave w then owns queries 32w.. and accumulates dQ^T += K^T dS^T, both operands read
//            with transposing LDS reads.
// The kernel is bound by memory latency, not arithmetic: with 73 KB of LDS and about 170 registers only two
// workgroups fit a compute unit, and a workgroup spends half its life waiting for its first rows (measured with
// timestamps: 6.2 of 12.9 us at n = 128), while a traffic-only kernel with the same access pattern runs 1.4x as
// fast in the same place.  With kUnits = 2 a workgroup handles two consecutive (sequence, head) units and requests
// the second unit's rows in phase 2 of the first, when the dK / dV accumulators and the K fragments
// have left their registers: the rows travel while dQ is computed and stored.  (Requesting them earlier, during
// phase 1, needs more registers than there are: the compiler then spills, and a spill reload waits for every
// load in flight, which undoes the overlap.  Measured inside the benchmark step: 76 -> 70 us.)  With packed tokens
// the 40 loads of a thread are not issued in one burst, during which the wave can do nothing else (timestamps: 2.5 us
// for the burst), but five at a time between the four steps of the dQ loop (another 1.1 us off).
constexpr int kDsPitch = 136;   // LDS row pitch of dS in bf16 (272 B)

// kMode (see kRowsIdentity .. in common.h): a unit whose tokens sit in consecutive buffer rows moves all its rows with
// buffer instructions: one descriptor per tensor and unit that starts at the unit's first row and ends with its last
// (built with scalar arithmetic) and one per-lane byte offset per tensor that is the same for every unit, to which
// the step from one group of rows to the next is added.  Rows past the unit's end then read as zeros and
// are dropped on a store without a compare, and forming an address is one 32-bit add.  (With per-lane 64-bit
// addresses every row access costs a 64-bit multiply, three quarter-rate vector instructions: a fifth of all vector
// instructions of this kernel were address arithmetic.)
// kUnits: (sequence, head) units per workgroup, 1 or 2.
template <int kMode, int kUnits>
__global__ __launch_bounds__(256, 2) void attn_bwd_fused128_kernel(
    const uint16_t* __restrict__ dout, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    const uint16_t* __restrict__ v, const uint16_t* __restrict__ o, const float* __restrict__ lse, int64_t dos,
    int64_t qs, int64_t ks, int64_t vs, int64_t os, const int32_t* __restrict__ cu,
    const float* __restrict__ slopes, float scale, uint16_t* __restrict__ dq, uint16_t* __restrict__ dk,
    uint16_t* __restrict__ dv, int64_t dqs, int64_t dks, int64_t dvs, int T, const int32_t* __restrict__ rows,
    int32_t* __restrict__ misuse, const int32_t* __restrict__ key_lens, int H, int n_units) {
  constexpr bool kRows = kMode != kRowsIdentity;   // token t may sit at another row than t
  if (kMode == kRowsIdentity) rows = nullptr;
  __shared__ __attribute__((aligned(16))) uint16_t sA[kTile * kPitch];      // Q, then K
  __shared__ __attribute__((aligned(16))) uint16_t sB[kTile * kPitch];      // dO, then output rows
  __shared__ __attribute__((aligned(16))) uint16_t sDs[kTile * kDsPitch];   // K and V rows on their way in, then dS as [key][query]
  __shared__ __attribute__((aligned(16))) float sLse[kTile];                // -lse, base-2 units
  __shared__ __attribute__((aligned(16))) float sDelta[kTile];              // -Delta

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 31, g = lane >> 5;
  const int kw = 32 * wave;
  const int kj = kw + c;
  const float cs = scale * kLog2e;
  const int st_row = tid >> 3, st_col = (tid & 7) * 8;
  const int tr_i = lane & 15, tr_q = lane >> 4;
  const int tr_row = (tr_i >> 2) + 4 * (tr_q >> 1);
  const int tr_col = 16 * (tr_q & 1) + 4 * (tr_i & 3);
  const int orow = lane >> 3, ocol = (lane & 7) * 8;

  // A unit: head h of the sequence that starts at packed token `start` and has n tokens, the first nk of which
  // are keys (n = 0: nothing to do).  Token r of the sequence sits at buffer row row_of(r).  With token_rows, rows listed in ascending
  // order whose first and last differ by n - 1 are consecutive (the usual case: padding is a suffix of each
  // batch row); then no per-token index load is needed.
  struct Unit {
    int h, start, n, nk;
    int64_t row0;
    bool contig;
  };
  auto find_unit = [&](int u) -> Unit {
    Unit U{0, 0, 0, 0, 0, kMode != kRowsPerLane};
    if (u >= n_units) return U;
    const int b = u / H;
    U.h = u - b * H;
    U.start = __builtin_amdgcn_readfirstlane(cu[b]);
    U.n = __builtin_amdgcn_readfirstlane(cu[b + 1]) - U.start;
    if (U.n > kTile) {   // the caller promised max_seqlen <= 128: skipped, never truncated
      raise_misuse(misuse);
      U.n = 0;
    }
    U.nk = key_lens ? min(__builtin_amdgcn_readfirstlane(key_lens[b]), U.n) : U.n;
    if (U.n <= 0 || U.nk <= 0) {   // empty, or no keys: skipped
      U.n = 0;
      return U;
    }
    U.row0 = U.start;
    if (kMode == kRowsMaybeContiguous) {
      const int r0 = __builtin_amdgcn_readfirstlane(rows[U.start]);
      U.row0 = r0;
      U.contig = __builtin_amdgcn_readfirstlane(rows[U.start + U.n - 1]) - r0 == U.n - 1;
    }
    return U;
  };
  // (only for units that are not moved with buffer instructions)
  auto row_of = [&](const Unit& U, int r) -> int64_t { return tok_row(rows, U.start + r); };
  // descriptor of head h of rows row0 .. row0 + cnt - 1 of a tensor with `stride` elements per row (cnt <= 0: of nothing)
  auto unit_rsrc = [&](const uint16_t* base, int64_t stride, const Unit& U, int cnt) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base) + (U.row0 * stride + U.h * kD), 0,
                                             cnt > 0 ? ((cnt - 1) * (int)stride + kD) * 2 : 0, kRsrcFlags);
  };
  constexpr int kNt = 2;   // cache policy of a buffer instruction: non-temporal

  // ---- coalesced row loads; thread (st_row, st_col) moves 16 bytes of rows st_row, +32, +64, +96.
  // The backward is the last reader of the forward's activations: non-temporal loads keep this one-pass
  // stream from evicting what other kernels of the step still need from L2 / the memory-side cache.
  u32x4 tk[4], tv[4], tq[4], tg[4], to[4];
  auto issue_kv = [&](const Unit& U) {
    if (kMode != kRowsPerLane && U.contig) {
      const __amdgpu_buffer_rsrc_t kr = unit_rsrc(k, ks, U, U.nk), vr = unit_rsrc(v, vs, U, U.nk);
      const uint32_t ko = ((uint32_t)st_row * (uint32_t)ks + (uint32_t)st_col) * 2u;
      const uint32_t vo = ((uint32_t)st_row * (uint32_t)vs + (uint32_t)st_col) * 2u;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        tk[it] = __builtin_amdgcn_raw_buffer_load_b128(kr, ko + (uint32_t)(it * 64) * (uint32_t)ks, 0, kNt);
        tv[it] = __builtin_amdgcn_raw_buffer_load_b128(vr, vo + (uint32_t)(it * 64) * (uint32_t)vs, 0, kNt);
      }
      return;
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      tk[it] = tv[it] = u32x4{0u, 0u, 0u, 0u};
      if (32 * it + st_row < U.nk) {
        const int64_t gr = row_of(U, 32 * it + st_row);
        tk[it] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(k + gr * ks + U.h * kD + st_col));
        tv[it] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(v + gr * vs + U.h * kD + st_col));
      }
    }
  };
  auto issue_qgo = [&](const Unit& U) {
    if (kMode != kRowsPerLane && U.contig) {
      const __amdgpu_buffer_rsrc_t qr = unit_rsrc(q, qs, U, U.n), gr = unit_rsrc(dout, dos, U, U.n),
                                   orr = unit_rsrc(o, os, U, U.n);
      const uint32_t qo = ((uint32_t)st_row * (uint32_t)qs + (uint32_t)st_col) * 2u;
      const uint32_t go = ((uint32_t)st_row * (uint32_t)dos + (uint32_t)st_col) * 2u;
      const uint32_t oo = ((uint32_t)st_row * (uint32_t)os + (uint32_t)st_col) * 2u;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        tq[it] = __builtin_amdgcn_raw_buffer_load_b128(qr, qo + (uint32_t)(it * 64) * (uint32_t)qs, 0, kNt);
        tg[it] = __builtin_amdgcn_raw_buffer_load_b128(gr, go + (uint32_t)(it * 64) * (uint32_t)dos, 0, kNt);
        to[it] = __builtin_amdgcn_raw_buffer_load_b128(orr, oo + (uint32_t)(it * 64) * (uint32_t)os, 0, kNt);
      }
      return;
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      tq[it] = tg[it] = to[it] = u32x4{0u, 0u, 0u, 0u};
      if (32 * it + st_row < U.n) {
        const int64_t gr = row_of(U, 32 * it + st_row);
        tq[it] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(q + gr * qs + U.h * kD + st_col));
        tg[it] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(dout + gr * dos + U.h * kD + st_col));
        to[it] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(o + gr * os + U.h * kD + st_col));
      }
    }
  };

  // rows 32 it + st_row of all five tensors of a unit that is moved with buffer instructions
  auto issue_group = [&](const Unit& U, int it) {
    const __amdgpu_buffer_rsrc_t kr = unit_rsrc(k, ks, U, U.nk), vr = unit_rsrc(v, vs, U, U.nk);
    const __amdgpu_buffer_rsrc_t qr = unit_rsrc(q, qs, U, U.n), gr = unit_rsrc(dout, dos, U, U.n),
                                 orr = unit_rsrc(o, os, U, U.n);
    const uint32_t r = (uint32_t)(32 * it + st_row);
    const uint32_t c2 = (uint32_t)st_col * 2u;
    tk[it] = __builtin_amdgcn_raw_buffer_load_b128(kr, r * (uint32_t)ks * 2u + c2, 0, kNt);
    tv[it] = __builtin_amdgcn_raw_buffer_load_b128(vr, r * (uint32_t)vs * 2u + c2, 0, kNt);
    tq[it] = __builtin_amdgcn_raw_buffer_load_b128(qr, r * (uint32_t)qs * 2u + c2, 0, kNt);
    tg[it] = __builtin_amdgcn_raw_buffer_load_b128(gr, r * (uint32_t)dos * 2u + c2, 0, kNt);
    to[it] = __builtin_amdgcn_raw_buffer_load_b128(orr, r * (uint32_t)os * 2u + c2, 0, kNt);
  };

  Unit nxt = find_unit(kUnits * blockIdx.x);
  issue_kv(nxt);
  issue_qgo(nxt);

#pragma unroll
  for (int iu = 0; iu < kUnits; ++iu) {
    const Unit U = nxt;
    const bool more = iu + 1 < kUnits;
    if (more) nxt = find_unit(kUnits * blockIdx.x + iu + 1);
    // n, h and nblk are uniform over the workgroup: every thread takes the same branches around the barriers
    const int n = U.n, nk = U.nk, h = U.h;
    const int nblk = (n + 31) >> 5;        // blocks of 32 queries
    const int nblk_k = (nk + 31) >> 5;     // blocks of 32 keys
    const bool wave_active = wave < nblk;  // this wave's tokens exist: phase 2 (queries) and the gradient rows
    const bool wave_keys = wave < nblk_k;  // ... and are keys: phase 1
    bf16x8 bk[4], bv[4];   // K^T, V^T fragments (B operands): lane = key column, 8 consecutive d per k-step

    if (n > 0) {
      // ---- phase 0
      // stored negated: -lse in base-2 units (-inf past the end, which makes P = 0 there)
      if (tid < kTile) sLse[tid] = tid < n ? -lse[(int64_t)h * T + U.start + tid] * kLog2e : -INFINITY;
      // K and V rows are staged in the dS buffer, which is free until phase 1: the 32 rows of K and of V that wave
      // `it` will own go into the very part of it that this wave later fills with dS (rows of 128 bytes, the 16-byte
      // pieces of a row rotated by the row number so that a wave's fragment reads spread over the banks).  A wave thus
      // overwrites only K/V rows it has already taken into registers, and one barrier serves all four tiles.
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int row = 32 * it + st_row;
        if (it < nblk) {   // rows n..32*nblk-1 are zeros; rows >= 32*nblk are never read
          uint16_t* part = &sDs[it * 32 * kDsPitch];
          const int piece = ((st_col >> 3) ^ (st_row & 7)) * 8;
          *reinterpret_cast<u32x4*>(&part[st_row * 64 + piece]) = tk[it];
          *reinterpret_cast<u32x4*>(&part[2048 + st_row * 64 + piece]) = tv[it];
          *reinterpret_cast<u32x4*>(&sA[row * kPitch + st_col]) = tq[it];
          *reinterpret_cast<u32x4*>(&sB[row * kPitch + st_col]) = tg[it];
        }
        float acc = 0.f;   // Delta = rowsum(dO * O): 8 lanes per row, 8 elements each
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc = fmaf(__uint_as_float(tg[it][i] << 16), __uint_as_float(to[it][i] << 16), acc);
          acc = fmaf(__uint_as_float(tg[it][i] & 0xffff0000u), __uint_as_float(to[it][i] & 0xffff0000u), acc);
        }
        acc += __shfl_xor(acc, 1, 64);
        acc += __shfl_xor(acc, 2, 64);
        acc += __shfl_xor(acc, 4, 64);
        if ((tid & 7) == 0) sDelta[row] = -acc;
      }
      __syncthreads();
      {
        const uint16_t* part = &sDs[wave * 32 * kDsPitch];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int piece = ((2 * s + g) ^ (c & 7)) * 8;
          bk[s] = lds_read8(&part[c * 64 + piece]);
          bv[s] = lds_read8(&part[2048 + c * 64 + piece]);
        }
      }
    }
    if (n <= 0) {
      if (more) {
        issue_kv(nxt);
        issue_qgo(nxt);
      }
      continue;
    }

    // ---- phase 1
    f32x16 dkacc[2], dvacc[2];   // dK^T, dV^T: d along accumulator rows, this wave's keys along lanes
#pragma unroll
    for (int i = 0; i < 16; ++i) { dkacc[0][i] = dkacc[1][i] = dvacc[0][i] = dvacc[1][i] = 0.f; }
    if (wave_keys) {
      // The S accumulator is pre-loaded with bias/scale = -(m_h/scale)|i-j| and the dP accumulator with
      // -Delta_i, so that after the matrix products  P = exp2(acc_S * c - lse2_i)  and  dS = P * acc_dP.
      const float k1 = slopes[h] / scale;
      float fj = (float)(kj - 4 * g);   // i - j = ci - fj with ci = 32ib + 8*(v/4) + v%4
      asm volatile("" : "+v"(fj));
#pragma unroll 1
      for (int ib = 0; ib < nblk; ++ib) {
        f32x16 sacc, pacc;
        const float d0 = (float)(32 * ib) - fj;
        if (ib == wave) {   // block with the diagonal
#pragma unroll
          for (int i = 0; i < 16; ++i) sacc[i] = -k1 * fabsf(d0 + (float)(8 * (i >> 2) + (i & 3)));
        } else {            // |i-j| = +-(ci - fj) on the whole block
          const float sk = ib < wave ? k1 : -k1;
          const float a = sk * d0;
#pragma unroll
          for (int i = 0; i < 16; ++i) sacc[i] = fmaf((float)(8 * (i >> 2) + (i & 3)), sk, a);
        }
        float nl[16];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float4 l4 = *reinterpret_cast<const float4*>(&sLse[32 * ib + 8 * r + 4 * g]);
          const float4 d4 = *reinterpret_cast<const float4*>(&sDelta[32 * ib + 8 * r + 4 * g]);
          nl[4 * r + 0] = l4.x; nl[4 * r + 1] = l4.y; nl[4 * r + 2] = l4.z; nl[4 * r + 3] = l4.w;
          pacc[4 * r + 0] = d4.x; pacc[4 * r + 1] = d4.y; pacc[4 * r + 2] = d4.z; pacc[4 * r + 3] = d4.w;
        }
        const uint16_t* qrow = &sA[(32 * ib + c) * kPitch + 8 * g];
        const uint16_t* grow = &sB[(32 * ib + c) * kPitch + 8 * g];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          sacc = mfma32(lds_read8(qrow + 16 * s), bk[s], sacc);
          pacc = mfma32(lds_read8(grow + 16 * s), bv[s], pacc);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int i = 4 * r + e;
            const float p = fast_exp2(fmaf(sacc[i], cs, nl[i]));
            sacc[i] = p;
            pacc[i] = p * pacc[i];
          }
          // dS of queries 32ib + 8r + 4g + 0..3 for this lane's key.  A key past the sequence end may hold
          // inf/NaN here (its score never entered lse) and phase 2 multiplies it with a zero K row, so it
          // must be an exact zero in LDS.
          u32x2 w;
          w[0] = kj < nk ? pack_bf16(pacc[4 * r + 0], pacc[4 * r + 1]) : 0u;
          w[1] = kj < nk ? pack_bf16(pacc[4 * r + 2], pacc[4 * r + 3]) : 0u;
          *reinterpret_cast<u32x2*>(&sDs[kj * kDsPitch + 32 * ib + 8 * r + 4 * g]) = w;
        }
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const bf16x8 bp = pack8(sacc[8 * kk + 0], sacc[8 * kk + 1], sacc[8 * kk + 2], sacc[8 * kk + 3],
                                  sacc[8 * kk + 4], sacc[8 * kk + 5], sacc[8 * kk + 6], sacc[8 * kk + 7]);
          const bf16x8 bs = pack8(pacc[8 * kk + 0], pacc[8 * kk + 1], pacc[8 * kk + 2], pacc[8 * kk + 3],
                                  pacc[8 * kk + 4], pacc[8 * kk + 5], pacc[8 * kk + 6], pacc[8 * kk + 7]);
          const int roff = (32 * ib + 16 * kk + tr_row) * kPitch + tr_col;
#pragma unroll
          for (int db = 0; db < 2; ++db) {
            const bf16x8 ag = join_tr(lds_read_tr4(&sB[roff + 32 * db]), lds_read_tr4(&sB[roff + 32 * db + 8 * kPitch]));
            dvacc[db] = mfma32(ag, bp, dvacc[db]);
            const bf16x8 aq = join_tr(lds_read_tr4(&sA[roff + 32 * db]), lds_read_tr4(&sA[roff + 32 * db + 8 * kPitch]));
            dkacc[db] = mfma32(aq, bs, dkacc[db]);
          }
        }
      }
    }
    __syncthreads();   // Q and dO have been read by everyone, all of dS is written

    // Accumulators (lane = token, 4 consecutive d per register group) -> this wave's 32 rows of sB ->
    // full rows of 128 bytes to global memory.  The slab is private to the wave, and the LDS operations
    // of one wave complete in order, so no barrier is needed between its uses.
    uint16_t* slab = &sB[kw * kPitch];
    // (rows at and beyond `live` are written as zeros: tokens that are no keys have zero dK and dV)
    auto store_rows = [&](const f32x16(&acc)[2], float mul, uint16_t* __restrict__ out, int64_t stride, int live) {
#pragma unroll
      for (int db = 0; db < 2; ++db) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          u32x2 w;
          w[0] = pack_bf16(acc[db][4 * r + 0] * mul, acc[db][4 * r + 1] * mul);
          w[1] = pack_bf16(acc[db][4 * r + 2] * mul, acc[db][4 * r + 3] * mul);
          *reinterpret_cast<u32x2*>(&slab[c * kPitch + 32 * db + 8 * r + 4 * g]) = w;
        }
      }
      if (kMode != kRowsPerLane && U.contig) {
        const __amdgpu_buffer_rsrc_t wr = unit_rsrc(out, stride, U, n);   // rows at and beyond n are dropped
        const uint32_t wo = ((uint32_t)(kw + orow) * (uint32_t)stride + (uint32_t)ocol) * 2u;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int row = 8 * it + orow;
          u32x4 w = *reinterpret_cast<const u32x4*>(&slab[row * kPitch + ocol]);
          if (kw + row >= live) w = u32x4{0u, 0u, 0u, 0u};
          __builtin_amdgcn_raw_buffer_store_b128(w, wr, wo + (uint32_t)(it * 16) * (uint32_t)stride, 0, kRows ? kNt : 0);
        }
        return;
      }
      uint16_t* oh = out + h * kD + ocol;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int row = 8 * it + orow;
        u32x4 w = *reinterpret_cast<const u32x4*>(&slab[row * kPitch + ocol]);
        if (kw + row >= live) w = u32x4{0u, 0u, 0u, 0u};
        if (kw + row < n) {
          // written into the padded layout these rows are final results of the step: stream them out
          if (rows) __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(oh + row_of(U, kw + row) * stride));
          else *reinterpret_cast<u32x4*>(oh + row_of(U, kw + row) * stride) = w;
        }
      }
    };

    // ---- phase 2
    if (wave_active) {
      store_rows(dkacc, scale, dk, dks, nk);
      store_rows(dvacc, 1.f, dv, dvs, nk);
    }
    if (wave_keys) {
      // K registers -> LDS over Q; rows of keys >= nk are zeros because they were staged as zeros
#pragma unroll
      for (int s = 0; s < 4; ++s)
        *reinterpret_cast<u32x4*>(&sA[kj * kPitch + 16 * s + 8 * g]) = __builtin_bit_cast(u32x4, bk[s]);
    }
    // dK, dV and the K fragments have left their registers: room for the next unit's rows, which travel while
    // dQ is computed and stored (the fences keep the compiler from moving the loads further up, where the
    // registers are still taken)
    // packed tokens: the next unit's loads go out in four groups between the steps of the dQ loop (with token_rows
    // the compiler runs out of registers for that: there they go out in one burst, before the loop)
    const bool spread = more && kMode == kRowsIdentity;
    __builtin_amdgcn_sched_barrier(0);
    if (more && !spread) {
      issue_kv(nxt);
      issue_qgo(nxt);
    }
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    {
      f32x16 dqacc[2];
#pragma unroll
      for (int i = 0; i < 16; ++i) { dqacc[0][i] = 0.f; dqacc[1][i] = 0.f; }
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        if (spread) issue_group(nxt, jb);
        __builtin_amdgcn_sched_barrier(0);
        if (wave_active && jb < nblk_k)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const int krow = 32 * jb + 16 * kk + tr_row;
          const bf16x8 bs = join_tr(lds_read_tr4(&sDs[krow * kDsPitch + kw + tr_col]),
                                    lds_read_tr4(&sDs[(krow + 8) * kDsPitch + kw + tr_col]));
#pragma unroll
          for (int db = 0; db < 2; ++db) {
            const bf16x8 ak = join_tr(lds_read_tr4(&sA[krow * kPitch + tr_col + 32 * db]),
                                      lds_read_tr4(&sA[(krow + 8) * kPitch + tr_col + 32 * db]));
            dqacc[db] = mfma32(ak, bs, dqacc[db]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (wave_active) store_rows(dqacc, scale, dq, dqs, n);
    }
    if (more) __syncthreads();   // the next unit's phase 0 overwrites sA, sB, sLse and sDelta
  }
}

}  // namespace

mb_status launch_attn_bwd_mfma(const AttnShape& s, const void* dout, const void* q, const void* k, const void* v,
                               const void* o, const float* lse, int64_t dos, int64_t qs, int64_t ks, int64_t vs,
                               int64_t os, void* dq, void* dk, void* dv, int64_t dqs, int64_t dks, int64_t dvs,
                               float* delta_ws, hipStream_t stream) {
  if (s.B > 65535) return fail(MB_ERR_UNSUPPORTED, "B=%d exceeds 65535 sequences per call", s.B);
  if (s.max_seqlen <= kTile) {
    const int64_t units = (int64_t)s.B * s.H;   // (sequence, head) pairs, head fastest; < 2^30 (checked by the caller)
#define MB_LAUNCH_FUSED(R, U)                                                                                        \
  hipLaunchKernelGGL((attn_bwd_fused128_kernel<R, U>), dim3((unsigned)((units + U - 1) / U)), dim3(256), 0,       \
                     stream, (const uint16_t*)dout, (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v,    \
                     (const uint16_t*)o, lse, dos, qs, ks, vs, os, s.cu_seqlens, s.slopes, s.scale, (uint16_t*)dq, \
                     (uint16_t*)dk, (uint16_t*)dv, dqs, dks, dvs, s.T, s.token_rows, s.misuse, s.key_lens, s.H,    \
                     (int)units)
    // buffer instructions: the 128 rows a unit can have must lie within 2^31 bytes in every tensor
    int64_t widest = 0;
    for (const int64_t st : {dos, qs, ks, vs, os, dqs, dks, dvs}) widest = st > widest ? st : widest;
    const bool narrow = (int64_t)kTile * widest * 2 < ((int64_t)1 << 31);
    // Up to two units per compute unit all fit the chip at once, a workgroup each: then a second unit per workgroup only
    // makes the chain longer (128 positions, two and one, replayed: 96 units 15.0 and 8.8 us, 252 units 16.8 and 10.7, 384
    // units 18.1 and 14.8, 512 units 18.9 and 16.1).  From 516 on two are taken: 20.7 us.
    if (units <= 2 * kComputeUnits) {
      if (!narrow) MB_LAUNCH_FUSED(kRowsPerLane, 1);
      else if (s.token_rows) MB_LAUNCH_FUSED(kRowsMaybeContiguous, 1);
      else MB_LAUNCH_FUSED(kRowsIdentity, 1);
    } else if (!narrow) {
      MB_LAUNCH_FUSED(kRowsPerLane, 2);
    } else if (s.token_rows) {
      MB_LAUNCH_FUSED(kRowsMaybeContiguous, 2);
    } else {
      MB_LAUNCH_FUSED(kRowsIdentity, 2);
    }
#undef MB_LAUNCH_FUSED
    return check_launch("attn_bwd_fused128_kernel");
  }
  // the work plan: the caller's, or built behind Delta in the workspace
  const int64_t cap = attn_plan_cap(s.B, s.max_seqlen, s.H);
  if (cap * kPlanXcds >= ((int64_t)1 << 31)) return fail(MB_ERR_UNSUPPORTED, "B * H * max_seqlen is too large for one launch");
  const int32_t* plan = s.plan;
  mb_status st = MB_OK;
  if (plan == nullptr) {
    int32_t* own = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(delta_ws) + attn_bwd_delta_bytes(s.H, s.T));
    st = launch_attn_plan(s, own, nullptr, stream);
    if (st != MB_OK) return st;
    plan = own;
  }
  // buffer-load path: a sequence's rows within 2^31 bytes of its first
  int64_t widest = qs > ks ? qs : ks;
  widest = widest > vs ? widest : vs;
  widest = widest > dos ? widest : dos;
  const bool narrow = (int64_t)s.max_seqlen * widest * 2 < ((int64_t)1 << 31);
  const dim3 grid((unsigned)(cap * kPlanXcds));
  // dQ first: it also leaves Delta for the dK/dV kernel
#define MB_LAUNCH_DQ(R)                                                                                            \
  hipLaunchKernelGGL(attn_bwd_dq_kernel<R>, grid, dim3(256), 0, stream, (const uint16_t*)dout, (const uint16_t*)q,  \
                     (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)o, lse, delta_ws, dos, qs, ks, vs,    \
                     os, s.slopes, s.scale, (uint16_t*)dq, dqs, s.T, s.token_rows, plan, cap)
  if (!narrow) MB_LAUNCH_DQ(kRowsPerLane);
  else if (s.token_rows) MB_LAUNCH_DQ(kRowsMaybeContiguous);
  else MB_LAUNCH_DQ(kRowsIdentity);
#undef MB_LAUNCH_DQ
  st = check_launch("attn_bwd_dq_kernel");
  if (st != MB_OK) return st;
#define MB_LAUNCH_DKV(R)                                                                                           \
  hipLaunchKernelGGL(attn_bwd_dkv_kernel<R>, grid, dim3(256), 0, stream, (const uint16_t*)dout, (const uint16_t*)q, \
                     (const uint16_t*)k, (const uint16_t*)v, lse, delta_ws, dos, qs, ks, vs, s.slopes, s.scale,     \
                     (uint16_t*)dk, (uint16_t*)dv, dks, dvs, s.T, s.token_rows, plan, cap)
  if (!narrow) MB_LAUNCH_DKV(kRowsPerLane);
  else if (s.token_rows) MB_LAUNCH_DKV(kRowsMaybeContiguous);
  else MB_LAUNCH_DKV(kRowsIdentity);
#undef MB_LAUNCH_DKV
  return check_launch("attn_bwd_dkv_kernel");
}

size_t attn_bwd_mfma_workspace_bytes(int B, int T, int max_seqlen, int H) {
  return attn_bwd_delta_bytes(H, T) + (max_seqlen <= kTile ? 0 : attn_plan_bytes(B, max_seqlen, H));
}

}  // namespace mb
