// GeGLU feed-forward of the encoder block (Eq. 2 of the paper):  y = (GeLU(x W1) (*) x V) W2,
// forward, bf16 storage, fp32 accumulation on the matrix cores.
//
// Two launches of one tiled GEMM kernel, both of the form  out[t, n] = sum_k X[t, k] * Wt[n, k]
// (token rows and weight rows are both contiguous along k, the storage of a linear layer):
//   1. gated:  the weight is the fused [2*inter, hidden] matrix of the appendix on GLU implementations
//      (rows 0..inter-1 = W1^T, rows inter.. = V^T).  A tile is, for its 64 to 320 tokens, 128 columns
//      of x W1 and THE SAME 128 columns of x V, so the slice and the product GeLU(.) (*) (.) happen on
//      the accumulators: neither projection is ever written to memory.
//   2. plain:  y = a W2 with the [hidden, inter] matrix W2^T.
//
// Tiling: 64 to 320 tokens x 256 weight rows per workgroup of 8 waves (2 x 4, each up to 160 x 64 = 10 accumulator tiles
// of v_mfma_f32_32x32x16_bf16), k in steps of 64 through two or three LDS stages that are filled by loads straight from
// global memory.  One workgroup per compute unit walks its tiles without a break in the stream of loads.
// The products are formed transposed (weight rows along accumulator rows, tokens along lanes), so a
// lane owns runs of 4 consecutive output columns of one token; the tile is turned into row segments through a
// wave-private LDS slab before it is stored.
//
// What bounds it, measured: the loads into LDS (without them the k loop runs 1.2 to 1.5 times as fast; beside the LDS reads
// they take 32 cycles per KB and compute unit, alone 16, in 64-byte pieces half as long again), and the power limit: at
// 1380 TFLOP/s (8192^3) the clock is down to 1.7 GHz and the matrix cores are busy 72 % of the time.  Hence the largest
// tile that fits the registers (fewest bytes per product), no pass of the operands through registers, and whole cache
// lines.  Tried: 256 x 128 tiles, two workgroups per compute unit (1035 TFLOP/s at 8192^3), four waves of 128 x 128 (1210),
// rows of 64 bytes in four stages (1284); the former kernel, four waves of 128 x 128 staged through registers, one tile per
// workgroup: 1262, and at K = 768 or 768 columns, where a tile's start and end or an empty last round weigh most:
//   26963 x 768, K = 3072: 135 -> 101 us;  26963 x 6144, K = 768: 283 -> 224 us;  26963 x 768, K = 6144: 292 -> 220 us;
//   8089 x 30528, K = 768: 496 -> 371 us (494 MB of output).
#include "common.h"
#include "mfma_util.h"

namespace mb {
namespace {

constexpr int kBK = 64;                               // k per stage
constexpr int kGroupM = 4;                            // token panels walked together (L2 reuse of the weight tiles)

// GeLU(h) = h * Phi(h), the exact (error-function) form, with Phi evaluated by the classic five-term
// rational approximation of erfc (Abramowitz & Stegun 7.1.26, absolute error below 1.5e-7):
//   x = |h| / sqrt 2,  t = 1 / (1 + p x),  u = (1/2) (a1 t + ... + a5 t^5) exp(-x^2) = Phi(-|h|),
//   Phi(h) = u for h < 0 and 1 - u otherwise,  hence  h Phi(h) = max(h, 0) - |h| u  for either sign.
// 12 vector instructions and two transcendentals per value; the result is rounded to bf16 (relative
// 2^-9) right after, so the approximation error is invisible.
__device__ __forceinline__ float gelu_exact(float h) {
  const float ah = fabsf(h);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, ah, 1.0f));
  float poly = fmaf(0.5f * 1.061405429f, t, 0.5f * -1.453152027f);
  poly = fmaf(poly, t, 0.5f * 1.421413741f);
  poly = fmaf(poly, t, 0.5f * -0.284496736f);
  poly = fmaf(poly, t, 0.5f * 0.254829592f);
  const float e = __builtin_amdgcn_exp2f(h * h * (-0.5f * kLog2e));
  const float u = poly * t * e;                       // Phi(-|h|), in (0, 1/2]
  return fmaf(-ah, u, fmaxf(h, 0.0f));
}

// GeLU and its derivative Phi(h) + h phi(h) from the same intermediates (phi = the normal density).
__device__ __forceinline__ void gelu_and_grad(float h, float& val, float& grad) {
  const float ah = fabsf(h);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, ah, 1.0f));
  float poly = fmaf(0.5f * 1.061405429f, t, 0.5f * -1.453152027f);
  poly = fmaf(poly, t, 0.5f * 1.421413741f);
  poly = fmaf(poly, t, 0.5f * -0.284496736f);
  poly = fmaf(poly, t, 0.5f * 0.254829592f);
  const float e = __builtin_amdgcn_exp2f(h * h * (-0.5f * kLog2e));   // exp(-h^2 / 2)
  const float u = poly * t * e;                                      // Phi(-|h|)
  val = fmaf(-ah, u, fmaxf(h, 0.0f));
  const float phi_cdf = h < 0.f ? u : 1.0f - u;
  grad = fmaf(h * 0.3989422804014327f, e, phi_cdf);
}

// Epilogues of the GEMM kernel.
constexpr int kPlain = 0;      // out = product
constexpr int kGatedFwd = 1;   // out = GeLU(x W1) (*) x V on the accumulators (weight = W1^T over V^T)
constexpr int kPartial = 3;    // out = fp32 sums of one of several splits of the contraction
constexpr int kGateBwd = 2;    // the product is dA; with h | g read from `aux`: out = dA g GeLU'(h) | dA GeLU(h)

// Descriptor of `bytes` bytes from `base` (both wave-uniform).
__device__ __forceinline__ u32x4 raw_rsrc(const uint16_t* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  u32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu);
  r[2] = __builtin_amdgcn_readfirstlane(bytes);
  r[3] = 0x00020000u;   // raw buffer, 32-bit data format (gfx9 family)
  return r;
}
// All but the newest `kNewer` loads of this wave have arrived and its LDS reads are done; then the workgroup's barrier.
template <int kNewer>
__device__ __forceinline__ void stage_ready() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(kNewer) : "memory");
}

// The lane's number, counted afresh: unlike a copy it costs no register between two uses that are far apart.  The gate
// backward in tiles of 320 tokens needs all 256 (160 sums, 28 of fragments, 48 of h and g): with the lane and the epilogue's
// places kept across the products it had 3 and 4 (row count on the device) in memory, and taking them back made every
// epilogue wait for all loads in flight.
__device__ __forceinline__ int lane_again() {
  uint32_t all = ~0u;
  asm volatile("" : "+s"(all));   // (else the compiler keeps the first one)
  return __builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
}

constexpr int kSlabElems = 32 * 32;   // per wave: 32 tokens x 32 columns on their way out
// LDS of a tile shape, elements: kStages stages of 64 kMB token rows and 32 kWN kNB weight rows, and the waves' slabs.
template <int kMB, int kWN, int kNB, int kStages>
constexpr int kGemmLds = kStages * (64 * kMB + 32 * kWN * kNB) * kBK + 2 * kWN * kSlabElems;

// Wide tiles of 64 and 128 tokens leave room for a third stage, which pays from this many k steps on where the weights come
// from memory (two and three stages, 48 weights in turn; 64-token tiles: 8 steps 945 x 1536 8.5 and 7.3 us, 12 steps
// 1500 x 768 11.4 and 8.9, 200 x 6144 15.5 and 12.0, 48 steps 4000 x 768 38 and 26, 4 steps 5.9 and 5.9; 128-token tiles: 12
// steps 2500 x 2304 15.1 and 14.0, 945 x 6144 18.7 and 15.6, 16 steps 1500 x 3072 22.7 and 17.5).  Out of a warm L2 it makes
// little difference up to 12 steps (6.74 and 6.80, 8.19 and 8.24, 8.25 and 8.32, 14.3 and 13.8, 14.0 and 13.9; a gated product
// of 80 to 350 tokens 0.1 us more, 24505 x 192 with 8 steps 10.9 and 11.2); with the third stage's loads in front of the first
// products and behind the last ones it cost 0.3 us.
constexpr int kThirdStageFrom = 8;

// One workgroup of 2 kWN waves (2 along the tokens by kWN along the weight rows) per compute unit walks the tiles
// blockIdx.x, + gridDim.x, ...  A tile is 64 kMB tokens x 32 kWN kNB weight rows; a wave computes 32 kMB x 32 kNB of it.
// Wide (4 x 2 blocks, two stages, for 64 and 128 tokens three from kThirdStageFrom steps on): 64 to 320 tokens x 256.  Narrow (2 x 1 blocks, eight stages): 64 x 64 for products of
// few rows and columns, whose time is the latency of a step: a sixteenth of the bytes per step, seven steps in flight.
// X rows are K elements long.  The weight is stored by output column, rows of K elements (kWT false), or the other way round,
// K rows of ldw elements with the output columns along them (kWT: the weights of the forward, contracted over their other
// index): then a stage holds 64 of its rows as they are, and the matrix-core operand (8 consecutive k of one column per
// lane) comes out of transposing LDS reads, which take no longer (and no transposed copies are made of 14 MB of weights:
// 10 us a call at 768 x 3072).  kPartial: the contraction is split, tile id = split * tiles + tile, and
// the split's fp32 sums go to out (as float) + split * T_cap * ldo.
template <int kMode, bool kWT, int kMB, int kWN, int kNB, int kStages>
__device__ __forceinline__ void gemm_tiles(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W, int K, int ldw,
                                           int n_tiles, int splits, int gate_row, int w_rows, int T, int T_cap,
                                           uint16_t* __restrict__ out, int ldo, const uint16_t* __restrict__ aux,
                                           int gate_col, uint16_t* __restrict__ smem, int wave) {
  constexpr bool kGated = kMode == kGatedFwd;
  constexpr int kBM = 64 * kMB, kBN = 32 * kWN * kNB, kWaves = 2 * kWN;
  static_assert(!kGated || (kNB == 2 && !kWT), "the gated epilogue pairs the wave's two weight blocks");
  static_assert(!kWT || kBN == 256 || kBN == 64, "swizzles of a weight row");
  constexpr int kRows = kBM + kBN;                  // rows of a stage: tokens, then weight rows
  constexpr int kStageElems = kRows * kBK;
  constexpr int kLoads = kRows / (8 * kWaves);      // 8-row loads per wave and k step

  // (the grid is sized for T_cap rows; the tile map uses the token panels that hold tokens, so that the
  // idle workgroups are the last ones and not the share of one XCD)
  const int m_tiles = (T + kBM - 1) / kBM;
  const int tiles = m_tiles * n_tiles;
  const int total = kMode == kPartial ? tiles * splits : tiles;
  if ((int)blockIdx.x >= total) return;
  constexpr int kOutCols = kGated ? kBN / 2 : kBN;    // output columns per tile
  const int nk = kMode == kPartial ? K / (kBK * splits) : K / kBK;   // k steps per tile

  // Tile id -> token panel, weight tile and first k step.  Consecutive workgroup ids go round-robin to the 8 XCDs; give
  // every XCD a contiguous run of tiles, walked kGroupM token panels at a time, so that the tiles resident on one
  // XCD share their token panels and weight tiles in that XCD's L2.
  auto locate = [&](int id, int& m0, int& n0, int& k0) {
    const int per = total >> 3;
    int lin = id;
    if (lin < (per << 3)) lin = (lin & 7) * per + (lin >> 3);
    k0 = 0;
    if (kMode == kPartial) {
      k0 = __builtin_amdgcn_readfirstlane(lin / tiles) * nk;
      lin = lin % tiles;
    }
    const int group = lin / (kGroupM * n_tiles);
    const int first_m = group * kGroupM;
    const int gsize = min(m_tiles - first_m, kGroupM);
    const int rem = lin - group * (kGroupM * n_tiles);
    // (the divisions run on the vector unit; readfirstlane moves the wave-uniform results back to scalars)
    m0 = __builtin_amdgcn_readfirstlane(first_m + rem % gsize) * kBM;
    n0 = __builtin_amdgcn_readfirstlane(rem / gsize) * kOutCols;
  };

  const int lane = kMode == kGateBwd ? lane_again() : (int)(threadIdx.x & 63), c = lane & 31, g = lane >> 5;
  const int wm = wave / kWN, wn = wave % kWN;

  // Global -> LDS: a row of a stage is 128 bytes = 8 pieces, a load carries 8 rows (whole cache lines: rows of 64 bytes,
  // with twice the stages, measured a fifth slower).  Piece x of row r sits at position x ^ (r / 2) % 8, so that a
  // fragment read (one piece of 16 consecutive rows per quarter wave) touches every bank once.  Row bounds are the
  // descriptors': token rows at or beyond T and weight rows past the matrix deposit zeros.
  // (The k offset is the scalar operand.  The range check counts it, and it stays within a row of K elements.)
  // Load i of wave w carries rows 8 (w + kWaves i) .. of the stage.
  const uint32_t lane_off =
      ((uint32_t)(lane >> 3) * (uint32_t)K + (((lane & 7) ^ (4 * (wave & 1) + (lane >> 4))) * 8)) * 2u;
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(
      (__attribute__((address_space(3))) uint16_t*)smem);
  // kWT: a load of the weight carries 512 / kBN of its rows.  Piece x of row r sits at x ^ 4 (r % 4) (rows of 512 bytes)
  // or x ^ 4 (r / 2 % 2) (rows of 128 bytes): the four rows that a transposing read touches lie in different banks.
  constexpr int kTRows = 512 / kBN;
  constexpr int kXLoads = kBM / (8 * kWaves);       // the first kXLoads of a wave's loads are token rows
  const int trow = lane / (kBN / 8);
  auto tr_swizzle = [](int r) { return kBN == 256 ? 4 * (r & 3) : 4 * ((r >> 1) & 1); };
  static_assert(!kWT || kTRows * kWaves % 4 == 0, "a lane's swizzle is the same in all its loads");
  const uint32_t wlane_off = ((uint32_t)trow * (uint32_t)ldw +
                              (((lane % (kBN / 8)) ^ tr_swizzle(kTRows * wave + trow)) * 8)) * 2u;
  u32x4 rsrc[kLoads];
  uint32_t k_bytes = 0;              // scalar offset of the tile's first k step, in X and in a weight stored by column
  uint32_t wk_bytes = 0;             // the same in a weight stored by k
  auto aim = [&](int id) {           // descriptors of this wave's share of a tile's rows
    int m0, n0, k0;
    locate(id, m0, n0, k0);
    k_bytes = (uint32_t)k0 * (kBK * 2);
    wk_bytes = (uint32_t)k0 * (uint32_t)(kBK * 2) * (uint32_t)ldw;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      if (kWT && i >= kXLoads) {   // (all K rows and all kBN columns exist, and the weight is less than 2^32 bytes: the scalar
        // offset counts in the range check, a descriptor of 2^31 bytes took what lies behind them for zeros)
        const int row = kTRows * (wave + kWaves * (i - kXLoads));
        rsrc[i] = raw_rsrc(W + (int64_t)row * ldw + n0, 0xffffffffu);
        continue;
      }
      const int row = 8 * (wave + kWaves * i), r = row - kBM;   // r: row of the weight tile
      const bool token = row < kBM;
      const int first = token ? m0 + row : kGated ? (r < kBN / 2 ? n0 + r : gate_row + n0 + r - kBN / 2) : n0 + r;
      const int rows = max(min((token ? T : w_rows) - first, 8), 0);
      rsrc[i] = raw_rsrc((token ? X : W) + (int64_t)first * K, (uint32_t)rows * (uint32_t)K * 2u);
    }
  };
  auto fetch_one = [&](int i, int stage, int kt) {
    const bool by_k = kWT && i >= kXLoads;
    load_to_lds(lds0 + (stage * kStageElems + 8 * (wave + kWaves * i) * kBK) * 2, by_k ? wlane_off : lane_off, rsrc[i],
                by_k ? wk_bytes + (uint32_t)kt * (uint32_t)(kBK * 2) * (uint32_t)ldw : k_bytes + kt * (kBK * 2));
  };

  // Fragments of this wave inside a stage: tokens at rows 0 .., weight rows from kBM on.  Gated: the first weight block
  // holds columns of x W1, the second the same columns of x V.
  // (row r = multiple of 32 + c: its swizzle is (c / 2) % 8; piece 2 kk + g of the row)
  uint32_t frag[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) frag[kk] = c * kBK + (((2 * kk + g) ^ ((c >> 1) & 7)) * 8);
  const uint32_t xrow = wm * (32 * kMB) * kBK;
  constexpr int kWaveCols = kGated ? 32 : 32 * kNB;   // output columns per wave
  const uint32_t wrow = (kBM + wn * kWaveCols) * kBK;
  constexpr uint32_t kWBlock = (kGated ? kBN / 2 : 32) * kBK;   // from the first weight block of the wave to the second
  // (Narrow: a step is a chain of latencies, so the sums are kept and one addition per read is left.  1000 x 768, K = 3072:
  // 13.9 us with the additions as the compiler orders them, 13.3 us so.)
  constexpr bool kKeepSums = kWN == 2;
  uint32_t xfrag[4], wfrag[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    xfrag[kk] = xrow + frag[kk];
    wfrag[kk] = wrow + frag[kk];
    if (kKeepSums) asm volatile("" : "+v"(xfrag[kk]), "+v"(wfrag[kk]));
  }
  // kWT: weight columns 32 (kNB wn + i) .., rows 16 kk + 8 g .. of the stage; lane -> row (+ 4) and 4 columns
  uint32_t tfrag[kNB];
  {
    const int tr_i = lane & 15, tr_q = lane >> 4;
    const int r = (tr_i >> 2) + 8 * (tr_q >> 1);
#pragma unroll
    for (int i = 0; i < kNB; ++i) {
      const int x = 4 * (kNB * wn + i) + 2 * (tr_q & 1) + ((tr_i & 3) >> 1);
      tfrag[i] = kBM * kBK + r * kBN + ((x ^ tr_swizzle(r)) * 8) + 4 * (tr_i & 1);
    }
  }
  bf16x8 xf[2][kMB], wf[2][kNB];
  auto read_frag = [&](int stage, int kk, int i) {   // weight fragments first
    const uint16_t* cur = smem + stage * kStageElems;
    if (kWT && i < kNB) {
      const uint16_t* p = cur + tfrag[i] + kk * (16 * kBN);
      wf[kk & 1][i] = join_tr(lds_read_tr4(p), lds_read_tr4(p + 4 * kBN));
    } else if (i < kNB) wf[kk & 1][i] = lds_read8(cur + wfrag[kk] + i * kWBlock);
    else xf[kk & 1][i - kNB] = lds_read8(cur + xfrag[kk] + (i - kNB) * 32 * kBK);
  };
  constexpr int kFrags = kMB + kNB, kMfma = kMB * kNB;
  f32x16 acc[kNB][kMB];

  // The k steps of all the workgroup's tiles form one sequence; the loads run kStages steps ahead of the products, across
  // the end of a tile, so that the next tile's first steps arrive during this one's last products and its epilogue.
  // (Past the last tile the loads repeat it: their number stays the same and nobody reads them.  With three stages that would
  // be a step's bytes more, so there they load nothing: their descriptors become empty.)
  int f_tile = blockIdx.x, f_kt = 0;
  aim(f_tile);
  auto advance = [&]() {
    if (++f_kt < nk) return;
    f_kt = 0;
    if (f_tile + (int)gridDim.x < total) {
      f_tile += gridDim.x;
      aim(f_tile);
    } else if (kStages == 3) {
#pragma unroll
      for (int i = 0; i < kLoads; ++i) rsrc[i][2] = 0u;
    }
  };
  auto fill = [&](int st) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) fetch_one(i, st, f_kt);
    advance();
  };
  // (a third stage is requested once the first has arrived: in front of it its loads would only hold up the first products)
  constexpr int kFirst = kStages == 3 ? 2 : kStages;
#pragma unroll
  for (int st = 0; st < kFirst; ++st) fill(st);
  stage_ready<(kFirst - 1) * kLoads>();
#pragma unroll
  for (int i = 0; i < kFrags; ++i) read_frag(0, 0, i);
  if (kFirst < kStages) fill(kFirst);

  // store instructions of an epilogue, per wave (they are issued also where every lane is out of range)
  constexpr int kStores = kMode == kPartial ? 0 : kGated ? 2 * kMB : (kMode == kGateBwd ? 4 : 2) * kMB * kNB;
  constexpr int kNewer = (kStages - 2) * kLoads;   // loads of the steps after the next one
  static_assert(kNewer + kStores < 64, "fits the counter");
  bool first = true;
  int stage = 0;
  for (int tile = blockIdx.x; tile < total; tile += gridDim.x) {
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
      for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[nb][mb][v] = 0.f;
    // One step = four quarters of kMfma matrix instructions (k = 16 each); during a quarter the next one's fragments are
    // read.  In front of the last quarter stands the barrier, behind which nobody reads this stage any more and the
    // next one has arrived: the last quarter reads the next stage's first fragments, and this stage is refilled.  The
    // memory instructions are spread over the matrix instructions: the waves share one address unit and one LDS, and a
    // wave that issues its loads in one go waits for everybody's.
    // Loads and stores complete in the order they were issued, and the loads of a tile's second step are issued before
    // the stores of the tile before it: the first barrier of a tile lets those stores (at least kStores) travel on.
#pragma unroll 1
    for (int kt = 0; kt < nk; ++kt) {
      const int next = stage + 1 == kStages ? 0 : stage + 1;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if (kk == 3) {
          if (kt == 0 && !first) stage_ready<kNewer + kStores>();
          else stage_ready<kNewer>();
        }
#pragma unroll
        for (int x = 0; x < kMfma; ++x) {
#pragma unroll
          for (int i = x; i < kFrags; i += kMfma) read_frag(kk == 3 ? next : stage, (kk + 1) & 3, i);
          if (kk == 3) {
#pragma unroll
            for (int i = x; i < kLoads; i += kMfma) fetch_one(i, stage, f_kt);
          }
          __builtin_amdgcn_sched_barrier(0);
          acc[x % kNB][x / kNB] = mfma32(wf[kk & 1][x % kNB], xf[kk & 1][x / kNB], acc[x % kNB][x / kNB]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      advance();
      stage = next;
    }
    first = false;

    int m0, n0, k0;
    locate(tile, m0, n0, k0);
    if (kMode == kPartial) {   // fp32 sums: a lane owns runs of 4 consecutive columns of one token
      float* dst = reinterpret_cast<float*>(out) + (int64_t)(k0 / nk) * T_cap * ldo;
#pragma unroll
      for (int mb = 0; mb < kMB; ++mb) {
        const int row = m0 + wm * (32 * kMB) + mb * 32 + c;
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) {
          const int col = n0 + wn * kWaveCols + nb * 32 + 4 * g;
          if (row < T && col < w_rows) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              *reinterpret_cast<float4*>(dst + (int64_t)row * ldo + col + 8 * j) =
                  make_float4(acc[nb][mb][4 * j], acc[nb][mb][4 * j + 1], acc[nb][mb][4 * j + 2], acc[nb][mb][4 * j + 3]);
          }
        }
      }
      continue;
    }
    // Epilogue: 32 tokens x 32 columns at a time through the wave's own slab, out of which rows leave as 64-byte
    // segments.  (Piece x of a row at position x ^ (row / 4) % 4; the LDS operations of one wave complete in order.)
    uint16_t* slab = smem + kStages * kStageElems + wave * kSlabElems;
    const int e_lane = kMode == kGateBwd ? lane_again() : lane;
    const int orow = e_lane >> 2, opiece = e_lane & 3, ec = e_lane & 31, eg = e_lane >> 5;
    const __amdgpu_buffer_rsrc_t ors = __builtin_amdgcn_make_buffer_rsrc(
        out + (int64_t)m0 * ldo, 0, (uint32_t)min(T - m0, kBM) * (uint32_t)ldo * 2u, 0x00020000);
    // Gate backward: h and g of a pass are requested kAhead passes before it (rows past the last token read the last one;
    // their results are dropped).
    constexpr int kAhead = 2;
    u32x4 hv[kMB * kNB][2], gv[kMB * kNB][2];
    auto request = [&](int p) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int row = m0 + wm * (32 * kMB) + (p / kNB) * 32 + 16 * u + orow;
        const int64_t at = (int64_t)min(row, T - 1) * ldo + n0 + wn * kWaveCols + (p % kNB) * 32 + opiece * 8;
        hv[p][u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(aux + at));
        gv[p][u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(aux + at + gate_col));
      }
    };
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb) {
#pragma unroll
      for (int nb = 0; nb < (kGated ? 1 : kNB); ++nb) {
        const int col = n0 + wn * kWaveCols + nb * 32 + opiece * 8;
        const int row0 = m0 + wm * (32 * kMB) + mb * 32 + orow;
        const bool cols_ok = kGated || col < w_rows;
        const uint32_t off0 = ((uint32_t)(row0 - m0) * (uint32_t)ldo + (uint32_t)col) * 2u;
        const int pass = mb * kNB + nb;
        if (kMode == kGateBwd) {
          if (pass == 0) {
#pragma unroll
            for (int p = 0; p < kAhead; ++p) request(p);
          }
          if (pass + kAhead < kMB * kNB) request(pass + kAhead);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float r[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (kGated) r[i] = gelu_exact(acc[0][mb][4 * j + i]) * acc[1][mb][4 * j + i];
            else r[i] = acc[nb][mb][4 * j + i];
          }
          u32x2 w;
          w[0] = pack_bf16(r[0], r[1]);
          w[1] = pack_bf16(r[2], r[3]);
          *reinterpret_cast<u32x2*>(&slab[ec * 32 + ((j ^ ((ec >> 2) & 3)) * 8) + 4 * eg]) = w;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int r = 16 * u + orow;
          const u32x4 w = *reinterpret_cast<const u32x4*>(&slab[r * 32 + ((opiece ^ ((r >> 2) & 3)) * 8)]);
          // (rows at or beyond T and columns past the matrix: an offset past the descriptor, the store is dropped)
          // (as the vector operand, where all of it is checked)
          const bool ok = row0 + 16 * u < T && cols_ok;
          const uint32_t off = ok ? off0 + (uint32_t)(32 * u) * (uint32_t)ldo : 0xffffffe0u;
          if (kMode == kGateBwd) {
            // w holds 8 values of dA; h and g of the same positions come from aux (columns col and
            // gate_col + col of a row); dh and dg go to the same two places of out
            u32x4 dh, dg;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              float v0, d0, v1, d1;
              gelu_and_grad(__uint_as_float(hv[pass][u][i] << 16), v0, d0);
              gelu_and_grad(__uint_as_float(hv[pass][u][i] & 0xffff0000u), v1, d1);
              const float a0 = __uint_as_float(w[i] << 16), a1 = __uint_as_float(w[i] & 0xffff0000u);
              const float g0 = __uint_as_float(gv[pass][u][i] << 16), g1 = __uint_as_float(gv[pass][u][i] & 0xffff0000u);
              dh[i] = pack_bf16(a0 * g0 * d0, a1 * g1 * d1);
              dg[i] = pack_bf16(a0 * v0, a1 * v1);
            }
            __builtin_amdgcn_raw_buffer_store_b128(dh, ors, off, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b128(dg, ors, ok ? off + (uint32_t)gate_col * 2u : off, 0, 0);
          } else {
            __builtin_amdgcn_raw_buffer_store_b128(w, ors, off, 0, 0);
          }
        }
      }
    }
  }
  stage_ready<0>();   // no load may still be on its way to LDS that the next workgroup owns
}

template <int kMode, bool kWT, int kMB, int kWN, int kNB, int kStages>
__global__ __launch_bounds__(128 * kWN, kWN / 2) void ffn_gemm_kernel(const uint16_t* __restrict__ X,
                                                                      const uint16_t* __restrict__ W, int K, int n_tiles,
                                                                      int splits, int gate_row, int w_rows, int T_cap,
                                                                      const int32_t* __restrict__ meta,
                                                                      uint16_t* __restrict__ out, int ldo,
                                                                      const uint16_t* __restrict__ aux, int gate_col, int ldw) {
  __shared__ __attribute__((aligned(1024))) uint16_t smem[kGemmLds<kMB, kWN, kNB, kStages>];
  // (readfirstlane: tells the compiler the value is wave-uniform, so descriptors built from it stay scalar)
  const int T = __builtin_amdgcn_readfirstlane(meta ? min(meta[0], T_cap) : T_cap);
  gemm_tiles<kMode, kWT, kMB, kWN, kNB, kStages>(X, W, K, ldw, n_tiles, splits, gate_row, w_rows, T, T_cap, out, ldo, aux, gate_col,
                                            smem, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

// The tile height (in 64 tokens, up to 320) with the least estimated time for T tokens, n_tiles weight tiles of 256 rows
// and `splits` shares of the contraction: rounds over the compute units times a k step's hundredths of a microsecond.  A
// k step of a tile took 0.31 (mb + 1) us with all compute units busy (26963 x 768, K = 6144: mb = 1 .. 4 68, 89, 120,
// 152 us a round) and no less than 0.7 us alone, where the loads' latency shows.  A tile count just above a multiple of
// 256 leaves the last round nearly empty (26963 x 768, K = 3072: tiles of 256 tokens 132 us, of 320 tokens 101 us;
// 945 x 6144, K = 768: 256 tokens 20 us, 128 tokens 14 us).
static inline int64_t height_cost(int T, int n_tiles, int splits, int mb) {
  const int64_t tiles = (int64_t)((T + 64 * mb - 1) / (64 * mb)) * n_tiles * splits;
  const int step = 31 * (mb + 1);
  return (tiles + kComputeUnits - 1) / kComputeUnits * (step < 70 ? 70 : step);
}
static inline int tile_height(int T, int n_tiles, int splits) {
  int best = 5;
  int64_t least = height_cost(T, n_tiles, splits, 5);
#pragma unroll
  for (int mb = 4; mb > 0; --mb) {
    const int64_t cost = height_cost(T, n_tiles, splits, mb);
    if (cost < least) {
      least = cost;
      best = mb;
    }
  }
  return best;
}

// The heights for up to 64 stretches of row counts, 1 << shift rows each, that reach up to a capacity: four bits for each
// (made in 0.5 us of host time).
struct TileHeights {
  uint64_t word[4];
  int shift;
};
static TileHeights tile_heights(int T_cap, int n_tiles, int splits) {
  TileHeights h{{0, 0, 0, 0}, 6};
  while ((T_cap - 1) >> h.shift > 63) ++h.shift;
  for (int i = 0; i <= (T_cap - 1) >> h.shift; ++i) {
    const int64_t last = (int64_t)(i + 1) << h.shift;
    h.word[i >> 4] |= (uint64_t)tile_height(last < T_cap ? (int)last : T_cap, n_tiles, splits) << (4 * (i & 15));
  }
  return h;
}

// For a row count that only the device knows: the height that suits that count is chosen here and not for the capacity
// on the host, whose choice is the worse the emptier the buffers are (in 32768 rows: 16384 tokens, K = 3072, 768 columns, 87
// and 69 us; 945 tokens, K = 768, 2304 columns, 21.2 and 9.7 us).  Out of a table and not by the estimates: their code is
// cold and took 1 us in front of every product.
template <int kMode, bool kWT>
__global__ __launch_bounds__(512, 2) void ffn_gemm_counted_kernel(const uint16_t* __restrict__ X,
                                                                  const uint16_t* __restrict__ W, int K, int n_tiles,
                                                                  int splits, int gate_row, int w_rows, int T_cap,
                                                                  const int32_t* __restrict__ meta,
                                                                  uint16_t* __restrict__ out, int ldo,
                                                                  const uint16_t* __restrict__ aux, int gate_col,
                                                                  TileHeights heights, int ldw) {
  __shared__ __attribute__((aligned(1024))) uint16_t smem[kGemmLds<5, 4, 2, 2>];
  const int T = __builtin_amdgcn_readfirstlane(min(meta[0], T_cap));
#define MB_TILE(n, stages) \
  gemm_tiles<kMode, kWT, n, 4, 2, stages>(X, W, K, ldw, n_tiles, splits, gate_row, w_rows, T, T_cap, out, ldo, aux, gate_col, smem, wave)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool third = K >= kThirdStageFrom * kBK * splits;
  const int at = (max(T, 1) - 1) >> heights.shift;
  const uint64_t word = at < 32 ? (at < 16 ? heights.word[0] : heights.word[1])
                                : (at < 48 ? heights.word[2] : heights.word[3]);
  switch ((int)(word >> (4 * (at & 15))) & 7) {
    case 1:
      if (third) MB_TILE(1, 3);
      else MB_TILE(1, 2);
      break;
    case 2:
      if (third) MB_TILE(2, 3);
      else MB_TILE(2, 2);
      break;
    case 3: MB_TILE(3, 2); break;
    case 4: MB_TILE(4, 2); break;
    default: MB_TILE(5, 2);
  }
#undef MB_TILE
}

// a = GeLU(h) (*) g, elementwise over [T, inter]: the separate activation pass of the unfused arrangements
// (the fused path above never runs it).  One 16-byte piece of h and of g per thread; HBM-bound.
__global__ __launch_bounds__(256) void gelu_gate_kernel(const uint16_t* __restrict__ h,
                                                        const uint16_t* __restrict__ gate, int64_t ld, int T_cap,
                                                        const int32_t* __restrict__ meta, int inter,
                                                        uint16_t* __restrict__ act) {
  const int T = meta ? min(meta[0], T_cap) : T_cap;
  const int pieces = inter >> 3;
  const int64_t total = (int64_t)T * pieces;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = idx / pieces;
    const int col = (int)(idx - row * pieces) * 8;
    const u32x4 hv = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(h + row * ld + col));
    const u32x4 gv = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(gate + row * ld + col));
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float h0 = __uint_as_float(hv[i] << 16), h1 = __uint_as_float(hv[i] & 0xffff0000u);
      const float g0 = __uint_as_float(gv[i] << 16), g1 = __uint_as_float(gv[i] & 0xffff0000u);
      r[i] = pack_bf16(gelu_exact(h0) * g0, gelu_exact(h1) * g1);
    }
    *reinterpret_cast<u32x4*>(act + row * (int64_t)inter + col) = r;
  }
}

// ------------------------------------------------------------------------------------------------ weight gradients
// out[m, n] = sum over tokens t of P[t, m] * Q[t, n]: both operands are stored token-major, so the contraction runs over
// ROWS.  Rows of 256 columns go to LDS as they are and the matrix-core operands (8 consecutive tokens of one column per
// lane) come out of transposing LDS reads (ds_read_b64_tr_b16).  The accumulator has m along registers and n along lanes,
// so a store instruction writes 128 contiguous bytes of two output rows: fp32 tiles need no staging.  Same shape as
// the projection kernel: 256 x 256 tiles, 8 waves of 128 x 64, steps of 64 tokens through two LDS stages (or 128 x 256, three
// stages) that are filled straight from global memory.  Both weight gradients of the sublayer are one launch (its few tiles fill the compute
// units better together); the tokens are split over `splits` workgroups per tile, and a second kernel adds the partial
// tiles in a fixed order, so the result is deterministic.
// Bound like the projections by the loads into LDS and the power limit.  At 26963 tokens, 768 x 3072 (381 GFLOP, two
// splits) 380 us and 13 us for adding up, where two launches of seven splits each, staged through registers, took 430 and
// 40 us (means of 20 passes); at 945 tokens (one split, no adding up) 23 us, in 256 x 256 tiles 30.
constexpr int kWgRows = 64;                         // tokens per k step
// Tiles are 64 kMB x 256: 256 (two stages) or, where those are too few to occupy the compute units, 128 (three stages).
template <int kMB>
constexpr int kWgStage = kWgRows * (64 * kMB + 256);   // elements: P rows, then Q rows

struct WgradProblem {
  const uint16_t* P;
  const uint16_t* Q;
  int ldp, ldq;
  int n_tiles, tiles;   // 256-column tiles of Q, tiles in all (of the height at hand)
  float* out;           // its [M, N] floats of the first split
};

template <int kMB, int kStages>
__global__ __launch_bounds__(512, 2) void ffn_wgrad_kernel(WgradProblem a, WgradProblem b, int splits, int T_cap,
                                                           const int32_t* __restrict__ meta, int64_t split_pitch) {
  __shared__ __attribute__((aligned(1024))) uint16_t smem[kStages * kWgStage<kMB>];
  const int T = __builtin_amdgcn_readfirstlane(meta ? min(meta[0], T_cap) : T_cap);
  // workgroup -> split and tile, every XCD a contiguous run: its compute units stream the same token rows
  const int tiles = a.tiles + b.tiles, total = tiles * splits, run = total >> 3;
  int lin = blockIdx.x;
  if (lin < (run << 3)) lin = (lin & 7) * run + (lin >> 3);
  const int split = __builtin_amdgcn_readfirstlane(lin / tiles);
  const int at = lin - split * tiles;
  const bool second = at >= a.tiles;
  const WgradProblem& pr = second ? b : a;
  const int tile = second ? at - a.tiles : at;
  const int n_tiles = pr.n_tiles, ldp = pr.ldp, ldq = pr.ldq;
  const int tile_m = __builtin_amdgcn_readfirstlane(tile / n_tiles);
  constexpr int kM = 64 * kMB, kLoads = kMB + 4, kMfma = 2 * kMB, kFrags = kMB + 2;
  const int m0 = tile_m * kM, n0 = (tile - tile_m * n_tiles) * 256, N = n_tiles * 256;
  // steps of this split; steps past the last token read zeros and add nothing
  const int steps_total = (T + kWgRows - 1) / kWgRows;
  const int per = (steps_total + splits - 1) / splits;
  const int s_begin = split * per;
  const int nsteps = max(min(steps_total - s_begin, per), 0);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, g = lane >> 5;
  const int wm = wave >> 2, wn = wave & 3;

  // A load carries 1024 bytes, 512 / kM rows of P or two of Q.  Load i of wave w: i < kMB the (w + 8 i)-th of P, else the
  // (w + 8 (i - kMB))-th of Q.  Piece x (8 columns) of row r sits at position x ^ 4 (r % 4): the four rows a transposing read
  // touches lie in different banks.  The descriptor ends with the last token row, so that rows past T deposit zeros.
  constexpr int kPRows = 512 / kM;
  const int prow = lane / (kM / 8), qrow = lane >> 5;
  const int ppiece = (lane % (kM / 8)) ^ (4 * ((kPRows * (wave & 1) + prow) & 3));
  const int qpiece = (lane & 31) ^ (4 * (2 * (wave & 1) + qrow));
  const uint32_t plane = ((uint32_t)prow * (uint32_t)ldp + ppiece * 8) * 2u;
  const uint32_t qlane = ((uint32_t)qrow * (uint32_t)ldq + qpiece * 8) * 2u;
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint16_t*)smem);
  auto fetch_one = [&](int i, int stage, int step) {
    const bool is_p = i < kMB;
    const int per_load = is_p ? kPRows : 2, at = per_load * (wave + 8 * (is_p ? i : i - kMB));
    const int first = (s_begin + step) * kWgRows + at;
    int rows = min(T - first, per_load);
    asm("" : "+s"(rows));   // (else both bounds are one vector instruction, and the descriptor comes out of it too late)
    rows = max(rows, 0);
    const int ld = is_p ? ldp : ldq, cols = is_p ? kM : 256;
    const uint16_t* base = (is_p ? pr.P + m0 : pr.Q + n0) + (int64_t)min(first, T) * ld;
    load_to_lds(lds0 + (stage * kWgStage<kMB> + (is_p ? 0 : kWgRows * kM) + at * cols) * 2, is_p ? plane : qlane,
                raw_rsrc(base, rows > 0 ? (uint32_t)((rows - 1) * ld + cols) * 2u : 0u), 0);
  };

  // Fragment reads: lane -> row tr_row (+ 8) and 4 columns of a 16 x 32 patch; P columns 32 (kMB wm + mb), Q columns
  // 64 wn + 32 nb.
  const int tr_i = lane & 15, tr_q = lane >> 4;
  const int tr_row = (tr_i >> 2) + 4 * (tr_q >> 1);
  const int tr_piece = 2 * (tr_q & 1) + ((tr_i & 3) >> 1), tr_sub = 4 * (tr_i & 1);
  uint32_t foff[kFrags];
#pragma unroll
  for (int i = 0; i < kFrags; ++i) {
    const int x = (i < kMB ? 4 * (kMB * wm + i) : 8 * wn + 4 * (i - kMB)) + tr_piece;
    foff[i] = (i < kMB ? 0 : kWgRows * kM) + tr_row * (i < kMB ? kM : 256) + ((x ^ (4 * (tr_i >> 2))) * 8) + tr_sub;
  }
  bf16x8 pf[2][kMB], qf[2][2];
  auto read_frag = [&](int stage, int kk, int i) {
    const int cols = i < kMB ? kM : 256;
    const uint16_t* p = smem + stage * kWgStage<kMB> + foff[i] + kk * (16 * cols);
    const bf16x8 f = join_tr(lds_read_tr4(p), lds_read_tr4(p + 8 * cols));
    if (i < kMB) pf[kk & 1][i] = f;
    else qf[kk & 1][i - kMB] = f;
  };
  f32x16 acc[kMB][2];   // [m block][n block]
#pragma unroll
  for (int x = 0; x < kMB; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[x][y][v] = 0.f;

#pragma unroll
  for (int st = 0; st < kStages; ++st)
#pragma unroll
    for (int i = 0; i < kLoads; ++i) fetch_one(i, st, st);
  stage_ready<(kStages - 1) * kLoads>();
#pragma unroll
  for (int i = 0; i < kFrags; ++i) read_frag(0, 0, i);
  int stage = 0;
  // (the order within a step is that of the projection kernel)
#pragma unroll 1
  for (int st = 0; st < nsteps; ++st) {
    const int next = stage + 1 == kStages ? 0 : stage + 1;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk == 3) stage_ready<(kStages - 2) * kLoads>();
#pragma unroll
      for (int x = 0; x < kMfma; ++x) {
#pragma unroll
        for (int i = x; i < kFrags; i += kMfma) read_frag(kk == 3 ? next : stage, (kk + 1) & 3, i);
        if (kk == 3) {
#pragma unroll
          for (int i = x; i < kLoads; i += kMfma) fetch_one(i, stage, st + kStages);
        }
        __builtin_amdgcn_sched_barrier(0);
        acc[x >> 1][x & 1] = mfma32(pf[kk & 1][x >> 1], qf[kk & 1][x & 1], acc[x >> 1][x & 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    stage = next;
  }
  // fp32 tile: register v of block (x, y) is row 8 (v / 4) + 4 g + v % 4, lane c is the column
  float* dst = pr.out + split * split_pitch + (int64_t)(m0 + wm * (32 * kMB)) * N + n0 + wn * 64 + c;
#pragma unroll
  for (int x = 0; x < kMB; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        dst[(int64_t)(x * 32 + 8 * (v >> 2) + 4 * g + (v & 3)) * N + y * 32] = acc[x][y][v];
  stage_ready<0>();   // no load may still be on its way to LDS that the next workgroup owns
}

// The two gradients from their partial tiles: out[i] = sum over splits of partial[s][i], in order; the first count_a
// groups of four go to out_a, the others to out_b.
__global__ __launch_bounds__(256) void ffn_wgrad_reduce_kernel(const float* __restrict__ partial, int splits,
                                                               int64_t count_a, int64_t count_b,
                                                               float* __restrict__ out_a, float* __restrict__ out_b) {
  const float4* src = reinterpret_cast<const float4*>(partial);
  const int64_t count4 = count_a + count_b;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count4; i += (int64_t)gridDim.x * blockDim.x) {
    float4 a = src[i];
    for (int s = 1; s < splits; ++s) {
      const float4 b = src[(int64_t)s * count4 + i];
      a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    (i < count_a ? reinterpret_cast<float4*>(out_a)[i] : reinterpret_cast<float4*>(out_b)[i - count_a]) = a;
  }
}

// out[t, :] = sum over splits of partial[s][t, :], in order, for t < T (rows of N floats, N a multiple of 4).
__global__ __launch_bounds__(256) void add_splits_kernel(const float* __restrict__ partial, int splits, int T_cap,
                                                         const int32_t* __restrict__ meta, int N,
                                                         uint16_t* __restrict__ out) {
  const int T = meta ? min(meta[0], T_cap) : T_cap;
  const int64_t pitch = (int64_t)T_cap * N / 4, count = (int64_t)T * N / 4;
  const float4* src = reinterpret_cast<const float4*>(partial);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x) {
    float4 a = src[i];
    for (int s = 1; s < splits; ++s) {
      const float4 b = src[s * pitch + i];
      a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    u32x2 w;
    w[0] = pack_bf16(a.x, a.y);
    w[1] = pack_bf16(a.z, a.w);
    reinterpret_cast<u32x2*>(out)[i] = w;
  }
}

}  // namespace

template <int kMode, bool kWT, int kMB, int kWN, int kNB, int kStages>
static void launch_gemm_tile(const void* x, const void* wt, int K, int n_cols, int splits, int gate_row, int w_rows,
                             int T_cap, const int32_t* meta, void* out, int ldo, const uint16_t* aux, int gate_col,
                             hipStream_t stream) {
  constexpr int kBN = 32 * kWN * kNB;
  const int m_tiles = (T_cap + 64 * kMB - 1) / (64 * kMB), n_tiles = (n_cols + kBN - 1) / kBN;
  const int64_t total = (int64_t)m_tiles * n_tiles * splits;
  ffn_gemm_kernel<kMode, kWT, kMB, kWN, kNB, kStages>
      <<<dim3((unsigned)(total < kComputeUnits ? total : kComputeUnits)), dim3(128 * kWN), 0, stream>>>(
          static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(wt), K, n_tiles, splits, gate_row, w_rows, T_cap,
          meta, static_cast<uint16_t*>(out), ldo, aux, gate_col, n_cols);
}

// Estimated microseconds of a product in tiles of the best height, `splits` shares of the contraction.
static double gemm_cost(int T_cap, int n_cols, int K, int splits) {
  const int n_tiles = (n_cols + 255) / 256;
  return 0.01 * (double)height_cost(T_cap, n_tiles, splits, tile_height(T_cap, n_tiles, splits)) * (K / (kBK * splits));
}

template <int kMode, bool kWT = false>
static void launch_gemm(const void* x, const void* wt, int K, int n_cols, int splits, int gate_row, int w_rows, int T_cap,
                        const int32_t* meta, void* out, int ldo, const uint16_t* aux, int gate_col, hipStream_t stream) {
  const int n_tiles = (n_cols + 255) / 256;
  if (meta) {
    // as many workgroups as the lowest tiles of a full buffer would take, one per compute unit at most
    const int64_t most = (int64_t)((T_cap + 63) / 64) * n_tiles * splits;
    ffn_gemm_counted_kernel<kMode, kWT><<<dim3((unsigned)(most < kComputeUnits ? most : kComputeUnits)), dim3(512), 0, stream>>>(
        static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(wt), K, n_tiles, splits, gate_row, w_rows, T_cap,
        meta, static_cast<uint16_t*>(out), ldo, aux, gate_col, tile_heights(T_cap, n_tiles, splits), n_cols);
    return;
  }
#define MB_TILE(n, stages) \
  launch_gemm_tile<kMode, kWT, n, 4, 2, stages>(x, wt, K, n_cols, splits, gate_row, w_rows, T_cap, meta, out, ldo, aux, gate_col, stream)
  const bool third = K >= kThirdStageFrom * kBK * splits;
  switch (tile_height(T_cap, n_tiles, splits)) {
    case 1:
      if (third) MB_TILE(1, 3);
      else MB_TILE(1, 2);
      break;
    case 2:
      if (third) MB_TILE(2, 3);
      else MB_TILE(2, 2);
      break;
    case 3: MB_TILE(3, 2); break;
    case 4: MB_TILE(4, 2); break;
    default: MB_TILE(5, 2);
  }
#undef MB_TILE
}

// The same in narrow tiles: 0.23 us a step, 1.5 us a tile.
static double narrow_cost(int T_cap, int n_cols, int K) {
  const int64_t tiles = (int64_t)((T_cap + 63) / 64) * (n_cols / 64);
  return (double)((tiles + kComputeUnits - 1) / kComputeUnits) * (0.23 * (K / kBK) + 1.5);
}

// out[t, n] = sum_k x[t, k] * wt[n, k] with the plain epilogue; in narrow tiles where their estimate is less: 945 x 768, K = 3072: 37 us in tiles of 64 x 256, 14 us in 64 x 64; 300 x 768, K = 768: 8.0 and 6.0 us;
// 2000 x 768, K = 768 (two rounds of narrow tiles): 8.7 and 9.9 us.
template <bool kWT = false>
static void launch_plain(const void* x, const void* wt, int T_cap, const int32_t* meta, int n_in, int n_out, void* y,
                         hipStream_t stream) {
  if (narrow_cost(T_cap, n_out, n_in) < gemm_cost(T_cap, n_out, n_in, 1)) {
    launch_gemm_tile<kPlain, kWT, 1, 2, 1, 8>(x, wt, n_in, n_out, 1, 0, n_out, T_cap, meta, y, n_out, nullptr, 0, stream);
    return;
  }
  launch_gemm<kPlain, kWT>(x, wt, n_in, n_out, 1, 0, n_out, T_cap, meta, y, n_out, nullptr, 0, stream);
}

mb_status launch_geglu_fwd(const void* x, const void* w1v, const void* w2, int T_cap, const int32_t* meta,
                           int hidden, int inter, void* act, void* y, hipStream_t stream) {
  if (T_cap == 0) return MB_OK;
  launch_gemm<kGatedFwd>(x, w1v, hidden, 2 * inter, 1, inter, 2 * inter, T_cap, meta, act, inter, nullptr, 0, stream);
  launch_plain(act, w2, T_cap, meta, inter, hidden, y, stream);
  return check_launch("ffn_gemm_kernel");
}

mb_status launch_linear_fwd(const void* x, const void* wt, int T_cap, const int32_t* meta, int n_in, int n_out,
                            void* y, hipStream_t stream) {
  if (T_cap == 0) return MB_OK;
  launch_plain(x, wt, T_cap, meta, n_in, n_out, y, stream);
  return check_launch("ffn_gemm_kernel");
}

mb_status launch_gelu_gate(const void* h, const void* gate, int64_t ld, int T_cap, const int32_t* meta, int inter,
                           void* act, hipStream_t stream) {
  if (T_cap == 0) return MB_OK;
  const int64_t pieces = (int64_t)T_cap * (inter >> 3);
  const int blocks = (int)((pieces + 255) / 256 < 8192 ? (pieces + 255) / 256 : 8192);
  gelu_gate_kernel<<<dim3(blocks), dim3(256), 0, stream>>>(static_cast<const uint16_t*>(h),
                                                           static_cast<const uint16_t*>(gate), ld, T_cap, meta, inter,
                                                           static_cast<uint16_t*>(act));
  return check_launch("gelu_gate_kernel");
}

// Workspace of the backward: h|g recomputed, dh|dg, the partial weight-gradient tiles.
static constexpr int kWgradSplits = 7;
static size_t bwd_ws_layout(int T_cap, int hidden, int inter, size_t off[3]) {
  size_t at = 0;
  const size_t rows = (size_t)T_cap * 2 * inter * 2;
  off[0] = at; at += align_up(rows, 256);                                   // hg   [T_cap, 2 inter] bf16
  off[1] = at; at += align_up(rows, 256);                                   // dhg  [T_cap, 2 inter] bf16
  off[2] = at; at += align_up((size_t)kWgradSplits * 2 * inter * hidden * 4, 256);   // partial tiles, fp32
  return at;
}

size_t geglu_bwd_workspace_bytes(int T_cap, int hidden, int inter) {
  size_t off[3];
  return bwd_ws_layout(T_cap, hidden, inter, off);
}

// dw2[c, j] = sum_t dy[t, c] act[t, j] and dw1v[j, c] = sum_t dhg[t, j] x[t, c], [hidden, inter] and [2 inter, hidden].
// `room`: floats that `partial` holds.
static void launch_wgrad(const void* dy, const void* act, const void* dhg, const void* x, int hidden, int inter,
                         int T_cap, const int32_t* meta, float* partial, size_t room, float* dw2, float* dw1v,
                         hipStream_t stream) {
  const int64_t size_a = (int64_t)hidden * inter, size_b = 2 * size_a;
  // The tile height and the split with the least estimated time: rounds over the compute units (about 1.5 us a step of 64
  // tokens and 6 us before and after, 1.1 us a step in tiles of half the height), and the partial tiles' way through memory
  // at 4.5 TB/s.  (The whole backward at 26963 tokens with 1, 2, 3, 4 splits: 1354, 1165, 1239, 1185 us; at 945 tokens 92,
  // 105, 116, 121 us.)  Half the height occupies the compute units where the tiles are few: one split, 256 and 128 rows,
  // 768 x 3072 (108 and 216 tiles) 200 tokens 14.2 and 11.8 us, 945 tokens 29.9 and 22.9, 2500 tokens 67.6 and 47.6; 8000 tokens
  // in two splits 137 and 167; 256 x 1024 (12 and 24 tiles), 945 tokens in three splits 20.5 and 16.7.
  // Fewer splits are longer chains of fp32 additions, T / (16 splits) of them: against 64 bits on its own bf16 operands dW2
  // is off by 1.8e-7 (945 tokens, one split) and 7.4e-7 (26963, two) where seven splits gave 0.9e-7 and 3.9e-7.  Both are a
  // thousandth and less of the 2^-9 that the operands were rounded by.  So half the height comes with as many splits at
  // least (4000 tokens in one split would be 73 us instead of 81).
  const int tiles_a = hidden / 256 * (inter / 256), steps = (T_cap + kWgRows - 1) / kWgRows;
  int splits = 1, height = 4;
  double least = 1e300;
  for (int mb = 4; mb >= 2; mb -= 2) {
    const int tiles = 3 * tiles_a * (4 / mb);
    for (int s = splits; s <= kWgradSplits && (size_t)s * (size_t)(size_a + size_b) <= room; ++s) {
      const double cost =
          (double)((tiles * s + kComputeUnits - 1) / kComputeUnits) * ((mb == 4 ? 1.5 : 1.1) * ((steps + s - 1) / s) + 6.0) +
          (s > 1 ? 4.0 + 4.0 * (2 * s + 1) * (size_a + size_b) / 4.5e6 : 0.0);
      if (cost < least) {
        least = cost;
        splits = s;
        height = mb;
      }
    }
  }
  const bool whole = splits == 1;   // the tiles are the result
  const int per_256 = 4 / height, tiles = 3 * tiles_a * per_256;
  const WgradProblem a{static_cast<const uint16_t*>(dy), static_cast<const uint16_t*>(act), hidden, inter, inter / 256,
                       tiles_a * per_256, whole ? dw2 : partial};
  const WgradProblem b{static_cast<const uint16_t*>(dhg), static_cast<const uint16_t*>(x), 2 * inter, hidden,
                       hidden / 256, 2 * tiles_a * per_256, whole ? dw1v : partial + size_a};
  if (height == 4)
    ffn_wgrad_kernel<4, 2><<<dim3(tiles * splits), dim3(512), 0, stream>>>(a, b, splits, T_cap, meta, size_a + size_b);
  else
    ffn_wgrad_kernel<2, 3><<<dim3(tiles * splits), dim3(512), 0, stream>>>(a, b, splits, T_cap, meta, size_a + size_b);
  if (!whole)
    ffn_wgrad_reduce_kernel<<<dim3(2048), dim3(256), 0, stream>>>(partial, splits, size_a / 4, size_b / 4, dw2, dw1v);
}

mb_status launch_geglu_bwd(const void* dy, const void* x, const void* w1v, const void* w2, const void* act,
                           const void* hg_saved, int T_cap, const int32_t* meta, int hidden, int inter, void* dx,
                           float* dw1v, float* dw2, void* workspace, hipStream_t stream) {
  size_t off[3];
  bwd_ws_layout(T_cap, hidden, inter, off);
  char* ws = static_cast<char*>(workspace);
  const uint16_t* hg = hg_saved ? static_cast<const uint16_t*>(hg_saved) : reinterpret_cast<uint16_t*>(ws + off[0]);
  uint16_t* dhg = reinterpret_cast<uint16_t*>(ws + off[1]);
  float* partial = reinterpret_cast<float*>(ws + off[2]);
  if (T_cap > 0) {
    // h | g = x (W1 | V): handed over by a caller that stored it, else computed again
    if (!hg_saved) launch_plain(x, w1v, T_cap, meta, hidden, 2 * inter, ws + off[0], stream);
    // dA = dy W2^T, and on its way out  dh = dA g GeLU'(h),  dg = dA GeLU(h)
    launch_gemm<kGateBwd, true>(dy, w2, hidden, inter, 1, 0, inter, T_cap, meta, dhg, 2 * inter, hg, inter, stream);
    // dx = dh W1^T + dg V^T = (dh | dg) (W1 | V)^T: the longest contraction onto the fewest columns.  With few tokens its
    // tiles leave most compute units idle, so it is taken in narrow tiles, or the contraction is split where that pays for
    // a second launch and for adding up the shares (the partial sums lie where the weight gradients' partial tiles come
    // later).  768 x 3072, one piece in narrow tiles and 8 shares with the adding up: 60 tokens 21.6 and 14.8 us, 400 tokens
    // 22.6 and 16.6, 945 tokens 24.0 and 24.5 and the gap between two launches; 256 x 1024: 945 tokens 10.1 and 14.6.
    int splits = 1;
    double least = narrow_cost(T_cap, hidden, 2 * inter) + 1.0;   // (weights by k: 2 us more than the estimate at 100 steps)
    for (int s = 1; s <= 8; s *= 2) {   // (2 inter / 64 is a multiple of 8)
      if ((size_t)s * T_cap > (size_t)kWgradSplits * 2 * inter) break;
      const double cost = gemm_cost(T_cap, hidden, 2 * inter, s) +
                          (s > 1 ? 7.0 + 8.0 * s * T_cap * hidden / 6.0e6 : 0.0);   // launch, write and read
      if (cost < least) {
        least = cost;
        splits = s;
      }
    }
    if (splits == 1) {
      launch_plain<true>(dhg, w1v, T_cap, meta, 2 * inter, hidden, dx, stream);
    } else {
      launch_gemm<kPartial, true>(dhg, w1v, 2 * inter, hidden, splits, 0, hidden, T_cap, meta, partial, hidden, nullptr, 0,
                            stream);
      const int64_t pieces = (int64_t)T_cap * hidden / 4;
      add_splits_kernel<<<dim3((unsigned)(pieces < 256 * 1024 ? (pieces + 255) / 256 : 1024)), dim3(256), 0, stream>>>(
          partial, splits, T_cap, meta, hidden, static_cast<uint16_t*>(dx));
    }
  }
  // the weight gradients; h | g has been read, so their partial tiles may lie over it where that is the larger place
  float* wpart = partial;
  size_t room = (size_t)kWgradSplits * 2 * inter * hidden;
  if (off[1] - off[0] > room * sizeof(float)) {
    wpart = reinterpret_cast<float*>(ws + off[0]);
    room = (off[1] - off[0]) / sizeof(float);
  }
  launch_wgrad(dy, act, dhg, x, hidden, inter, T_cap, meta, wpart, room, dw2, dw1v, stream);
  return check_launch("geglu backward");
}

}  // namespace mb
