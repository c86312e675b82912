// Attention in fp32 arithmetic: fp32 storage, bf16 storage with a head size other than 64, or softmax_scale <= 0;
// head sizes up to 128.  The products run on the matrix cores' fp32 instruction (v_mfma_f32_16x16x4_f32: fp32
// operands, fp32 fused multiply-adds, no rounding of the inputs), everything else is plain fp32; the bias of the
// paper's Eq. 1, -m_h*|i-j|, is evaluated on the fly.
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s, a sixteenth of bf16) and, for small batches, how evenly the
// waves fill the 1024 SIMDs.  Hence the small blocks: a wave owns 16 queries (or keys), a workgroup 64, and the
// other operand is streamed in tiles of 32 rows through two LDS buffers.  The 16x16x4 instruction has the rate of
// the 32x32x2 one with half the rows per wave, so a batch makes twice as many waves.
// Forward + backward, fp32, 16 sequences of up to 256 tokens, 12 heads of 64 (9.6 GFLOP): 206 us (50 + 62 + 88), of
// which the matrix cores are busy a third; one wave per (token, head) on the vector unit takes 3239 us (and is kept for
// sequences of a few tokens, below).
//
// Instruction layout (lane l, c = l % 16, g = l / 16):  A: row c, k = g.  B: column c, k = g.  D: column c, rows
// 4 g + v for register v = 0..3.  k is summed away, so it may be numbered freely as long as A and B agree:
//   * a row operand is read four consecutive floats at a time, instruction e of a group of four taking k = 4 g + e;
//   * an accumulator tile is the B operand of the next product as it stands: instruction v takes rows 4 g + v.
#include "common.h"

namespace mb {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kGThreads = 256;
constexpr int kGOwn = 64;     // queries (keys) per workgroup: 16 per wave
constexpr int kGTile = 32;    // rows of a streamed tile

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Four consecutive elements of a row, as they are stored (16-byte or 8-byte accesses; every row starts 16-byte
// aligned), and as floats.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f32x4 raw4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ u32x2 raw4(const uint16_t* p) { return *reinterpret_cast<const u32x2*>(p); }
__device__ __forceinline__ f32x4 floats(f32x4 r) { return r; }
__device__ __forceinline__ f32x4 floats(u32x2 r) {
  return f32x4{__uint_as_float(r[0] << 16), __uint_as_float(r[0] & 0xffff0000u), __uint_as_float(r[1] << 16),
               __uint_as_float(r[1] & 0xffff0000u)};
}
__device__ __forceinline__ void store4(float* p, f32x4 x) { *reinterpret_cast<f32x4*>(p) = x; }
__device__ __forceinline__ uint32_t bf16_rne(float x) {
  const uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;   // NaN stays NaN
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;                   // nearest even
}
__device__ __forceinline__ void store4(uint16_t* p, f32x4 x) {
  *reinterpret_cast<uint2*>(p) =
      make_uint2(bf16_rne(x[0]) | (bf16_rne(x[1]) << 16), bf16_rne(x[2]) | (bf16_rne(x[3]) << 16));
}

// e^x for the exponents of a softmax: 2^y for y = x log2(e) rounded, times 1 + ln2 (x log2(e) - y), the rounding of
// the product put back (a weight e^-5 of 256 equal ones would otherwise be off by 2e-7 of itself).  Seven instructions
// instead of expf's twelve or more.
// (x = -inf gives 0: the correction is then NaN or infinite, and is left out.)
__device__ __forceinline__ float exp_neg(float x) {
  constexpr float kL = 1.4426950408889634f, kLlo = (float)(1.4426950408889634074 - (double)kL);
  const float y = x * kL;
  const float r = fmaf(x, kLlo, fmaf(x, kL, -y)) * 0.6931471805599453f;
  const float e = __builtin_amdgcn_exp2f(y);
  return x < -104.f ? e : fmaf(e, r, e);   // below the smallest denormal the correction has nothing to add
}

// Sum / maximum over the four lanes that hold one column of an accumulator tile.
__device__ __forceinline__ float column_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}
__device__ __forceinline__ float column_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return fmaxf(x, __shfl_xor(x, 32, 64));
}

// Work slots.  Sequence b owns the slots from first_slot(b) = cu[b] / 64 + b to first_slot(b + 1) - 1, at least as
// many as it has blocks of 64 tokens, so a launch of T / 64 + B slots per head covers any cu_seqlens with no table
// and no host round trip; at most one slot per sequence stays empty.
__device__ __forceinline__ int64_t first_slot(const int32_t* __restrict__ cu, int b) {
  return (int64_t)(cu[b] / kGOwn) + b;
}
__device__ __forceinline__ int find_seq(const int32_t* __restrict__ cu, int B, int64_t slot) {
  int lo = 0, hi = B;   // first_slot(lo) <= slot; b >= hi starts behind it (or does not exist)
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (first_slot(cu, mid) <= slot) lo = mid; else hi = mid;
  }
  return lo;
}
static int64_t slots_of(const AttnShape& s) { return (int64_t)(s.T / kGOwn) + s.B; }

// Rows r0 .. r0 + 31 of one head of a sequence -> registers (as stored: nothing waits for the loads before the tile
// is deposited) -> LDS as floats, zeros past row n and column D.  Rows and columns that do not exist are fetched from
// the last row and the first columns instead of under a branch: a branch per load made every load wait for the one
// before it, a memory round trip per 16 bytes (4 per tile and thread).
// NB: blocks of 16 columns the head is padded to.
template <typename E, int NB>
struct Tile {
  static constexpr int kPitch = 16 * NB + 4;   // floats; a row then starts 4 banks after the one before
  static constexpr int kFloats = kGTile * kPitch;
  static constexpr int kPieces = kGTile * 4 * NB;
  static constexpr int kPerThread = (kPieces + kGThreads - 1) / kGThreads;
  decltype(raw4((const E*)nullptr)) r[kPerThread];
  __device__ __forceinline__ void fetch(const E* __restrict__ base, int64_t stride, const int32_t* __restrict__ rows,
                                        int start, int r0, int n, int D) {
    int at[kPerThread];
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) at[u] = start + min(r0 + ((int)threadIdx.x + u * kGThreads) / (4 * NB), n - 1);
    if (rows) {
#pragma unroll
      for (int u = 0; u < kPerThread; ++u) at[u] = rows[at[u]];
    }
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) {
      const int col = ((int)threadIdx.x + u * kGThreads) % (4 * NB) * 4;
      r[u] = raw4(base + (uint64_t)(uint32_t)at[u] * (uint32_t)stride + (col < D ? col : 0));   // stride < 2^24
    }
  }
  __device__ __forceinline__ void deposit(float* __restrict__ lds, int r0, int n, int D) const {
    const bool full = r0 + kGTile <= n && D == 16 * NB;
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) {
      const int idx = threadIdx.x + u * kGThreads;
      const int row = idx / (4 * NB), col = idx % (4 * NB) * 4;
      f32x4 x = floats(r[u]);
      if (!full) x = r0 + row < n && col < D ? x : f32x4{0.f, 0.f, 0.f, 0.f};
      if (kPieces % kGThreads == 0 || idx < kPieces) *reinterpret_cast<f32x4*>(&lds[row * kPitch + col]) = x;
    }
  }
};

// A wave's own 16 rows (lane column c) as B operand fragments: register 4 s + e holds element 16 s + 4 g + e.  (All loads
// first, as stored: converted where it is loaded, each bf16 piece would wait for the one before it, as in Tile.)
template <typename E, int NB>
__device__ __forceinline__ void own_rows(f32x4 (&f)[NB], const E* __restrict__ row, bool ok, int g, int D) {
  decltype(raw4(row)) r[NB];
#pragma unroll
  for (int s = 0; s < NB; ++s) {
    r[s] = decltype(raw4(row)){};
    if (ok && 16 * s + 4 * g < D) r[s] = raw4(row + 16 * s + 4 * g);
  }
#pragma unroll
  for (int s = 0; s < NB; ++s) f[s] = floats(r[s]);
}

// 16 rows of an LDS tile (from `rowp` = its first row, this lane's row c and column 4 g) times the wave's own rows, in
// two sums (shorter chains of dependent instructions and of roundings).
template <int NB>
__device__ __forceinline__ f32x4 rows_times_own(const float* __restrict__ rowp, const f32x4 (&own)[NB]) {
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}}, a[NB];
#pragma unroll
  for (int s = 0; s < NB; ++s) a[s] = *reinterpret_cast<const f32x4*>(rowp + 16 * s);
#pragma unroll
  for (int s = 0; s < NB; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e & 1] = mfma_f32(a[s][e], own[s][e], acc[e & 1]);
  return acc[0] + acc[1];
}

// Four rows of an LDS tile, this lane's column of every block: A operands of a product with the tile's transpose.
// `colp` points at this lane's row 4 g and column c.  They are read ahead of the exponentials that make the other
// operand (the fence keeps the compiler from sinking each read to its use, where its latency would show).
template <int NB>
struct Columns {
  float f[4][NB];
  __device__ __forceinline__ void read(const float* __restrict__ colp) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int db = 0; db < NB; ++db) f[v][db] = colp[v * (16 * NB + 4) + 16 * db];
  }
  // acc[db] += (those rows)^T x
  __device__ __forceinline__ void multiply(f32x4 (&acc)[NB], f32x4 x) const {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int db = 0; db < NB; ++db) acc[db] = mfma_f32(f[v][db], x[v], acc[db]);
  }
};

template <typename E, int NB>
__device__ __forceinline__ void store_own(E* __restrict__ row, const f32x4 (&acc)[NB], float mul, int g, int D) {
#pragma unroll
  for (int db = 0; db < NB; ++db)
    if (16 * db + 4 * g < D) store4(row + 16 * db + 4 * g, acc[db] * mul);
}

// Workgroups that share a compute unit (what their LDS tiles allow; the dK/dV kernel holds more registers and gets one
// fewer): bounds the registers the compiler may use.
template <int NB>
constexpr int kGWaves = NB <= 4 ? 3 : 2;

// Forward: a workgroup per (64 queries, head); S^T = K Q^T (keys along accumulator rows, queries along lanes), online
// softmax over tiles of 32 keys, O^T += V^T P^T.
template <typename E, int NB>
__global__ __launch_bounds__(kGThreads, kGWaves<NB>) void fwd_f32_kernel(
    const E* __restrict__ q, const E* __restrict__ k, const E* __restrict__ v, int64_t qs, int64_t ks, int64_t vs,
    const int32_t* __restrict__ cu, int B, int T, int D, const float* __restrict__ slopes, float scale,
    E* __restrict__ o, int64_t os, float* __restrict__ lse, const int32_t* __restrict__ rows, int max_seqlen,
    int32_t* __restrict__ misuse, int64_t slots) {
  using Tl = Tile<E, NB>;
  __shared__ __attribute__((aligned(16))) float smem[2][2][Tl::kFloats];   // [buffer][K, V]
  const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float slope = slopes[h];
  for (int64_t slot = blockIdx.x; slot < slots; slot += gridDim.x) {
    const int b = find_seq(cu, B, slot);
    const int start = cu[b], n = cu[b + 1] - start;
    const int64_t q0_ = (slot - first_slot(cu, b)) * kGOwn;
    if (q0_ >= n) continue;
    const int q0 = (int)q0_;
    if (n > max_seqlen) {   // longer than the caller promised: skipped, never computed on a guess
      raise_misuse(misuse);
      if (tid < kGOwn && q0 + tid < n) lse[(int64_t)h * T + start + q0 + tid] = __builtin_nanf("");
      continue;
    }
    const int qi = q0 + 16 * wave + c;
    const bool active = q0 + 16 * wave < n, q_ok = qi < n;
    const int64_t qrow = q_ok ? tok_row(rows, start + qi) : 0;
    const E* kh = k + (int64_t)h * D;
    const E* vh = v + (int64_t)h * D;
    Tl tk, tv;
    f32x4 bq[NB], acc[2][NB];   // two sums each (even and odd blocks of 16 keys): half as many roundings in a row
    own_rows<E, NB>(bq, q + qrow * qs + (int64_t)h * D, q_ok, g, D);
    tk.fetch(kh, ks, rows, start, 0, n, D);
    tv.fetch(vh, vs, rows, start, 0, n, D);
#pragma unroll
    for (int db = 0; db < NB; ++db) acc[0][db] = acc[1][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l[2] = {0.f, 0.f};   // l: this lane's share of the row sum
    __syncthreads();                // the previous slot's tiles are no longer read
    tk.deposit(smem[0][0], 0, n, D);
    tv.deposit(smem[0][1], 0, n, D);
    for (int j0 = 0, buf = 0; j0 < n; j0 += kGTile, buf ^= 1) {
      __syncthreads();   // this tile is complete; the other buffer is no longer read
      const bool more = j0 + kGTile < n;
      if (more) {
        tk.fetch(kh, ks, rows, start, j0 + kGTile, n, D);
        tv.fetch(vh, vs, rows, start, j0 + kGTile, n, D);
      }
      if (active) {
        f32x4 s[2];
        const float far = (float)(qi - j0 - 4 * g);   // i - j = far - (16 jb + x)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
          s[jb] = rows_times_own<NB>(&smem[buf][0][(16 * jb + c) * Tl::kPitch + 4 * g], bq);
#pragma unroll
          for (int x = 0; x < 4; ++x) s[jb][x] = fmaf(scale, s[jb][x], -slope * fabsf(far - (float)(16 * jb + x)));
        }
        if (!more) {   // keys past the end
          const int lim = n - j0 - 4 * g;
#pragma unroll
          for (int x = 0; x < 8; ++x) s[x / 4][x % 4] = 16 * (x / 4) + x % 4 < lim ? s[x / 4][x % 4] : -INFINITY;
        }
        float mt = m;
#pragma unroll
        for (int x = 0; x < 8; ++x) mt = fmaxf(mt, s[x / 4][x % 4]);
        Columns<NB> cv[2];
        cv[0].read(&smem[buf][1][4 * g * Tl::kPitch + c]);
        cv[1].read(&smem[buf][1][(16 + 4 * g) * Tl::kPitch + c]);
        __builtin_amdgcn_sched_barrier(0);
        mt = column_max(mt);
        const float mu = mt == -INFINITY ? 0.f : mt;   // nothing but -inf so far: every weight is an exact zero
        if (__any(mt > m)) {
          const float alpha = exp_neg(m - mu);
          l[0] *= alpha;
          l[1] *= alpha;
#pragma unroll
          for (int db = 0; db < NB; ++db) {
            acc[0][db] *= alpha;
            acc[1][db] *= alpha;
          }
        }
        m = mt;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            s[jb][x] = exp_neg(s[jb][x] - mu);
            l[jb] += s[jb][x];
          }
          cv[jb].multiply(acc[jb], s[jb]);
        }
      }
      if (more) {
        tk.deposit(smem[buf ^ 1][0], j0 + kGTile, n, D);
        tv.deposit(smem[buf ^ 1][1], j0 + kGTile, n, D);
      }
    }
    if (active) {
      const float sum = column_sum(l[0] + l[1]);
#pragma unroll
      for (int db = 0; db < NB; ++db) acc[0][db] += acc[1][db];
      if (q_ok) {
        store_own<E, NB>(o + qrow * os + (int64_t)h * D, acc[0], 1.f / sum, g, D);
        if (g == 0) lse[(int64_t)h * T + start + qi] = m + logf(sum);
      }
    }
  }
}

// Backward, query side: Delta of the workgroup's 64 queries (also left in `delta` for the key side), then
// dQ^T += K^T dS^T over tiles of 32 keys.
template <typename E, int NB>
__global__ __launch_bounds__(kGThreads, kGWaves<NB>) void bwd_f32_dq_kernel(
    const E* __restrict__ dout, const E* __restrict__ q, const E* __restrict__ k, const E* __restrict__ v,
    const E* __restrict__ o, const float* __restrict__ lse, int64_t dos, int64_t qs, int64_t ks, int64_t vs,
    int64_t os, const int32_t* __restrict__ cu, int B, int T, int D, const float* __restrict__ slopes, float scale,
    E* __restrict__ dq, int64_t dqs, float* __restrict__ delta, const int32_t* __restrict__ rows, int max_seqlen,
    int32_t* __restrict__ misuse, int64_t slots) {
  using Tl = Tile<E, NB>;
  __shared__ __attribute__((aligned(16))) float smem[2][2][Tl::kFloats];   // [buffer][K, V]
  const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float slope = slopes[h];
  for (int64_t slot = blockIdx.x; slot < slots; slot += gridDim.x) {
    const int b = find_seq(cu, B, slot);
    const int start = cu[b], n = cu[b + 1] - start;
    const int64_t q0_ = (slot - first_slot(cu, b)) * kGOwn;
    if (q0_ >= n) continue;
    const int q0 = (int)q0_;
    if (n > max_seqlen) {
      raise_misuse(misuse);
      continue;
    }
    const int qi = q0 + 16 * wave + c;
    const bool active = q0 + 16 * wave < n, q_ok = qi < n;
    const int64_t qrow = q_ok ? tok_row(rows, start + qi) : 0;
    const E* kh = k + (int64_t)h * D;
    const E* vh = v + (int64_t)h * D;
    Tl tk, tv;
    f32x4 bq[NB], bg[NB], acc[NB];
    own_rows<E, NB>(bq, q + qrow * qs + (int64_t)h * D, q_ok, g, D);
    own_rows<E, NB>(bg, dout + qrow * dos + (int64_t)h * D, q_ok, g, D);
    own_rows<E, NB>(acc, o + qrow * os + (int64_t)h * D, q_ok, g, D);   // O, for Delta only
    const float lq = q_ok ? lse[(int64_t)h * T + start + qi] : INFINITY;
    tk.fetch(kh, ks, rows, start, 0, n, D);
    tv.fetch(vh, vs, rows, start, 0, n, D);
    float dlt = 0.f;
#pragma unroll
    for (int s = 0; s < NB; ++s) {
#pragma unroll
      for (int e = 0; e < 4; ++e) dlt = fmaf(bg[s][e], acc[s][e], dlt);
      acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    dlt = column_sum(dlt);
    if (q_ok && g == 0) delta[(int64_t)h * T + start + qi] = dlt;
    __syncthreads();
    tk.deposit(smem[0][0], 0, n, D);
    tv.deposit(smem[0][1], 0, n, D);
    for (int j0 = 0, buf = 0; j0 < n; j0 += kGTile, buf ^= 1) {
      __syncthreads();
      const bool more = j0 + kGTile < n;
      if (more) {
        tk.fetch(kh, ks, rows, start, j0 + kGTile, n, D);
        tv.fetch(vh, vs, rows, start, j0 + kGTile, n, D);
      }
      if (active) {
        const float far = (float)(qi - j0 - 4 * g);   // i - j = far - (16 jb + x)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
          const int off = (16 * jb + c) * Tl::kPitch + 4 * g;
          const f32x4 s = rows_times_own<NB>(&smem[buf][0][off], bq);
          f32x4 ds = rows_times_own<NB>(&smem[buf][1][off], bg);
          Columns<NB> ck;
          ck.read(&smem[buf][0][(16 * jb + 4 * g) * Tl::kPitch + c]);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const float p = exp_neg(fmaf(scale, s[x], -slope * fabsf(far - (float)(16 * jb + x))) - lq);
            ds[x] = p * (ds[x] - dlt);
          }
          if (!more) {   // a key past the end has a zero K row but was never part of lse: its p may overflow
#pragma unroll
            for (int x = 0; x < 4; ++x) ds[x] = 16 * jb + x < n - j0 - 4 * g ? ds[x] : 0.f;
          }
          ck.multiply(acc, ds);
        }
      }
      if (more) {
        tk.deposit(smem[buf ^ 1][0], j0 + kGTile, n, D);
        tv.deposit(smem[buf ^ 1][1], j0 + kGTile, n, D);
      }
    }
    if (q_ok) store_own<E, NB>(dq + qrow * dqs + (int64_t)h * D, acc, scale, g, D);
  }
}

// Backward, key side: a workgroup per (64 keys, head), S = Q K^T (queries along accumulator rows, keys along lanes),
// dV^T += dO^T P and dK^T += Q^T dS over tiles of 32 queries.
template <typename E, int NB>
__global__ __launch_bounds__(kGThreads, kGWaves<NB> - 1) void bwd_f32_dkv_kernel(
    const E* __restrict__ dout, const E* __restrict__ q, const E* __restrict__ k, const E* __restrict__ v,
    const float* __restrict__ lse, const float* __restrict__ delta, int64_t dos, int64_t qs, int64_t ks, int64_t vs,
    const int32_t* __restrict__ cu, int B, int T, int D, int max_seqlen, const float* __restrict__ slopes,
    float scale, E* __restrict__ dk, E* __restrict__ dv, int64_t dks, int64_t dvs,
    const int32_t* __restrict__ rows, int32_t* __restrict__ misuse, int64_t slots) {
  using Tl = Tile<E, NB>;
  __shared__ __attribute__((aligned(16))) float smem[2][2][Tl::kFloats];   // [buffer][Q, dO]
  __shared__ __attribute__((aligned(16))) float srow[2][2][kGTile];        // [buffer][lse, Delta]
  const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float slope = slopes[h];
  for (int64_t slot = blockIdx.x; slot < slots; slot += gridDim.x) {
    const int b = find_seq(cu, B, slot);
    const int start = cu[b], n = cu[b + 1] - start;
    const int64_t k0_ = (slot - first_slot(cu, b)) * kGOwn;
    if (k0_ >= n) continue;
    const int k0 = (int)k0_;
    if (n > max_seqlen) {
      raise_misuse(misuse);
      continue;
    }
    const int kj = k0 + 16 * wave + c;
    const bool active = k0 + 16 * wave < n, k_ok = kj < n;
    const int64_t krow = k_ok ? tok_row(rows, start + kj) : 0;
    const E* qh = q + (int64_t)h * D;
    const E* gh = dout + (int64_t)h * D;
    Tl tq, tg;
    float tr = 0.f;
    auto fetch = [&](int i0) {
      tq.fetch(qh, qs, rows, start, i0, n, D);
      tg.fetch(gh, dos, rows, start, i0, n, D);
      // threads 0..31 carry lse (+inf past the end: P = 0), threads 32..63 Delta
      const int i = i0 + (tid & (kGTile - 1));
      if (tid < 2 * kGTile)
        tr = i < n ? (tid < kGTile ? lse : delta)[(int64_t)h * T + start + i] : (tid < kGTile ? INFINITY : 0.f);
    };
    auto deposit = [&](int buf, int i0) {
      tq.deposit(smem[buf][0], i0, n, D);
      tg.deposit(smem[buf][1], i0, n, D);
      if (tid < 2 * kGTile) srow[buf][tid / kGTile][tid & (kGTile - 1)] = tr;
    };
    f32x4 bk[NB], bv[NB], ak[NB], av[2][NB];   // dV in two sums, as O in the forward
    own_rows<E, NB>(bk, k + krow * ks + (int64_t)h * D, k_ok, g, D);
    own_rows<E, NB>(bv, v + krow * vs + (int64_t)h * D, k_ok, g, D);
    fetch(0);
#pragma unroll
    for (int db = 0; db < NB; ++db) ak[db] = av[0][db] = av[1][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
    deposit(0, 0);
    for (int i0 = 0, buf = 0; i0 < n; i0 += kGTile, buf ^= 1) {
      __syncthreads();
      const bool more = i0 + kGTile < n;
      if (more) fetch(i0 + kGTile);
      if (active) {
        const float far = (float)(kj - i0 - 4 * g);   // j - i = far - (16 ib + x)
#pragma unroll
        for (int ib = 0; ib < 2; ++ib) {
          const int off = (16 * ib + c) * Tl::kPitch + 4 * g;
          f32x4 p = rows_times_own<NB>(&smem[buf][0][off], bk);
          f32x4 ds = rows_times_own<NB>(&smem[buf][1][off], bv);
          const f32x4 lq = *reinterpret_cast<const f32x4*>(&srow[buf][0][16 * ib + 4 * g]);
          const f32x4 dl = *reinterpret_cast<const f32x4*>(&srow[buf][1][16 * ib + 4 * g]);
          const int cof = (16 * ib + 4 * g) * Tl::kPitch + c;
          Columns<NB> cg, cq;
          cg.read(&smem[buf][1][cof]);
          cq.read(&smem[buf][0][cof]);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            p[x] = exp_neg(fmaf(scale, p[x], -slope * fabsf(far - (float)(16 * ib + x))) - lq[x]);
            ds[x] = p[x] * (ds[x] - dl[x]);
          }
          cg.multiply(av[ib], p);
          cq.multiply(ak, ds);
        }
      }
      if (more) deposit(buf ^ 1, i0 + kGTile);
    }
#pragma unroll
    for (int db = 0; db < NB; ++db) av[0][db] += av[1][db];
    if (k_ok) {
      store_own<E, NB>(dv + krow * dvs + (int64_t)h * D, av[0], 1.f, g, D);
      store_own<E, NB>(dk + krow * dks + (int64_t)h * D, ak, scale, g, D);
    }
  }
}

// Workgroups per head: one per slot, up to a bound that any slot count fits under (the kernels walk on from there).
dim3 grid_of(const AttnShape& s) {
  const int64_t slots = slots_of(s);
  return dim3((unsigned)(slots < (1 << 20) ? slots : (1 << 20)), s.H);
}

template <typename E, int NB>
mb_status fwd_t(const AttnShape& s, const void* q, const void* k, const void* v, int64_t qs, int64_t ks, int64_t vs,
                void* o, int64_t os, float* lse, hipStream_t stream) {
  fwd_f32_kernel<E, NB><<<grid_of(s), dim3(kGThreads), 0, stream>>>(
      (const E*)q, (const E*)k, (const E*)v, qs, ks, vs, s.cu_seqlens, s.B, s.T, s.D, s.slopes, s.scale, (E*)o, os,
      lse, s.token_rows, s.max_seqlen, s.misuse, slots_of(s));
  return check_launch("fwd_f32_kernel");
}

template <typename E, int NB>
mb_status bwd_t(const AttnShape& s, const void* dout, const void* q, const void* k, const void* v, const void* o,
                const float* lse, int64_t dos, int64_t qs, int64_t ks, int64_t vs, int64_t os, void* dq, void* dk,
                void* dv, int64_t dqs, int64_t dks, int64_t dvs, float* delta, hipStream_t stream) {
  bwd_f32_dq_kernel<E, NB><<<grid_of(s), dim3(kGThreads), 0, stream>>>(
      (const E*)dout, (const E*)q, (const E*)k, (const E*)v, (const E*)o, lse, dos, qs, ks, vs, os, s.cu_seqlens, s.B,
      s.T, s.D, s.slopes, s.scale, (E*)dq, dqs, delta, s.token_rows, s.max_seqlen, s.misuse, slots_of(s));
  const mb_status st = check_launch("bwd_f32_dq_kernel");
  if (st != MB_OK) return st;
  bwd_f32_dkv_kernel<E, NB><<<grid_of(s), dim3(kGThreads), 0, stream>>>(
      (const E*)dout, (const E*)q, (const E*)k, (const E*)v, lse, delta, dos, qs, ks, vs, s.cu_seqlens, s.B, s.T, s.D,
      s.max_seqlen, s.slopes, s.scale, (E*)dk, (E*)dv, dks, dvs, s.token_rows, s.misuse, slots_of(s));
  return check_launch("bwd_f32_dkv_kernel");
}

// ------------------------------------------------------------------------------------------------ very short sequences
// One wave per (token, head) on the vector unit.  The kernels above give a sequence at least one workgroup and a whole
// tile of products however short it is: with a handful of tokens per sequence most of that is padding, and a workgroup's
// chain of loads, products and barriers is longer than the work.  Here every token is its own wave with nothing in front
// of it but its rows.  `limit` <= kTokenMax bounds the sequences' lengths.
constexpr int kTokenMax = 16;

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(uint16_t x) { return __uint_as_float((uint32_t)x << 16); }
__device__ __forceinline__ void from_f32(float* p, float x) { *p = x; }
__device__ __forceinline__ void from_f32(uint16_t* p, float x) { *p = (uint16_t)bf16_rne(x); }
__device__ __forceinline__ float wave_sum(float x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}
__device__ __forceinline__ float wave_max(float x) {
  for (int off = 32; off > 0; off >>= 1) x = fmaxf(x, __shfl_xor(x, off, 64));
  return x;
}
// Sequence that owns packed token t: the b with cu[b] <= t < cu[b+1] (empty sequences are skipped).
__device__ __forceinline__ int seq_of_token(const int32_t* __restrict__ cu, int B, int t) {
  int lo = 0, hi = B;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cu[mid] <= t) lo = mid; else hi = mid;
  }
  return lo;
}

template <typename E>
__global__ __launch_bounds__(64) void fwd_token_kernel(
    const E* __restrict__ q, const E* __restrict__ k, const E* __restrict__ v, int64_t qs, int64_t ks, int64_t vs,
    const int32_t* __restrict__ cu, int B, int T, int D, const float* __restrict__ slopes, float scale,
    E* __restrict__ o, int64_t os, float* __restrict__ lse, const int32_t* __restrict__ rows, int limit,
    int32_t* __restrict__ misuse) {
  __shared__ float sq[128], ss[kTokenMax];
  const int t = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
  if (t >= cu[B]) return;   // T may be a capacity: rows past the last real token are not touched
  const int b = seq_of_token(cu, B, t);
  const int start = cu[b], n = cu[b + 1] - start, i = t - start;
  if (n > limit) {   // longer than the caller promised: skipped
    raise_misuse(misuse);
    if (lane == 0) lse[(int64_t)h * T + t] = __builtin_nanf("");
    return;
  }
  const float slope = slopes[h];
  for (int d = lane; d < D; d += 64) sq[d] = to_f32(q[tok_row(rows, t) * qs + h * D + d]);
  __syncthreads();
  float s = -INFINITY;
  if (lane < n) {
    const E* kr = k + tok_row(rows, start + lane) * ks + h * D;
    float dot = 0.f;
    for (int d = 0; d < D; ++d) dot = fmaf(sq[d], to_f32(kr[d]), dot);
    s = scale * dot - slope * fabsf((float)(i - lane));
  }
  const float m = wave_max(s);
  const float e = lane < n ? expf(s - m) : 0.f;
  if (lane < n) ss[lane] = e;
  const float z = wave_sum(e);
  __syncthreads();
  const float inv = 1.f / z;
  for (int d = lane; d < D; d += 64) {
    float acc = 0.f;
    for (int j = 0; j < n; ++j) acc = fmaf(ss[j], to_f32(v[tok_row(rows, start + j) * vs + h * D + d]), acc);
    from_f32(&o[tok_row(rows, t) * os + h * D + d], acc * inv);
  }
  if (lane == 0) lse[(int64_t)h * T + t] = m + logf(z);
}

// Query side: Delta_i, dS_ij for all j, dQ_i.
template <typename E>
__global__ __launch_bounds__(64) void bwd_token_dq_kernel(
    const E* __restrict__ dout, const E* __restrict__ q, const E* __restrict__ k, const E* __restrict__ v,
    const E* __restrict__ o, const float* __restrict__ lse, int64_t dos, int64_t qs, int64_t ks, int64_t vs,
    int64_t os, const int32_t* __restrict__ cu, int B, int T, int D, const float* __restrict__ slopes, float scale,
    E* __restrict__ dq, int64_t dqs, float* __restrict__ delta, const int32_t* __restrict__ rows, int limit,
    int32_t* __restrict__ misuse) {
  __shared__ float sq[128], sg[128], sds[kTokenMax];
  const int t = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
  if (t >= cu[B]) return;
  const int b = seq_of_token(cu, B, t);
  const int start = cu[b], n = cu[b + 1] - start, i = t - start;
  if (n > limit) {
    raise_misuse(misuse);
    return;
  }
  const float slope = slopes[h];
  float part = 0.f;
  for (int d = lane; d < D; d += 64) {
    const float g = to_f32(dout[tok_row(rows, t) * dos + h * D + d]);
    sq[d] = to_f32(q[tok_row(rows, t) * qs + h * D + d]);
    sg[d] = g;
    part = fmaf(g, to_f32(o[tok_row(rows, t) * os + h * D + d]), part);
  }
  const float dlt = wave_sum(part);
  if (lane == 0) delta[(int64_t)h * T + t] = dlt;
  __syncthreads();
  const float l = lse[(int64_t)h * T + t];
  if (lane < n) {
    const E* kr = k + tok_row(rows, start + lane) * ks + h * D;
    const E* vr = v + tok_row(rows, start + lane) * vs + h * D;
    float dot = 0.f, dp = 0.f;
    for (int d = 0; d < D; ++d) {
      dot = fmaf(sq[d], to_f32(kr[d]), dot);
      dp = fmaf(sg[d], to_f32(vr[d]), dp);
    }
    sds[lane] = expf(scale * dot - slope * fabsf((float)(i - lane)) - l) * (dp - dlt);
  }
  __syncthreads();
  for (int d = lane; d < D; d += 64) {
    float acc = 0.f;
    for (int j = 0; j < n; ++j) acc = fmaf(sds[j], to_f32(k[tok_row(rows, start + j) * ks + h * D + d]), acc);
    from_f32(&dq[tok_row(rows, t) * dqs + h * D + d], scale * acc);
  }
}

// Key side: P_ij and dS_ij for all i, dV_j and dK_j.
template <typename E>
__global__ __launch_bounds__(64) void bwd_token_dkv_kernel(
    const E* __restrict__ dout, const E* __restrict__ q, const E* __restrict__ k, const E* __restrict__ v,
    const float* __restrict__ lse, const float* __restrict__ delta, int64_t dos, int64_t qs, int64_t ks, int64_t vs,
    const int32_t* __restrict__ cu, int B, int T, int D, int limit, const float* __restrict__ slopes, float scale,
    E* __restrict__ dk, E* __restrict__ dv, int64_t dks, int64_t dvs, const int32_t* __restrict__ rows,
    int32_t* __restrict__ misuse) {
  __shared__ float sk[128], sv[128], sp[kTokenMax], sds[kTokenMax];
  const int t = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
  if (t >= cu[B]) return;
  const int b = seq_of_token(cu, B, t);
  const int start = cu[b], n = cu[b + 1] - start, j = t - start;
  if (n > limit) {
    raise_misuse(misuse);
    return;
  }
  const float slope = slopes[h];
  for (int d = lane; d < D; d += 64) {
    sk[d] = to_f32(k[tok_row(rows, t) * ks + h * D + d]);
    sv[d] = to_f32(v[tok_row(rows, t) * vs + h * D + d]);
  }
  __syncthreads();
  if (lane < n) {
    const E* qr = q + tok_row(rows, start + lane) * qs + h * D;
    const E* gr = dout + tok_row(rows, start + lane) * dos + h * D;
    float dot = 0.f, dp = 0.f;
    for (int d = 0; d < D; ++d) {
      dot = fmaf(to_f32(qr[d]), sk[d], dot);
      dp = fmaf(to_f32(gr[d]), sv[d], dp);
    }
    const float p = expf(scale * dot - slope * fabsf((float)(lane - j)) - lse[(int64_t)h * T + start + lane]);
    sp[lane] = p;
    sds[lane] = p * (dp - delta[(int64_t)h * T + start + lane]);
  }
  __syncthreads();
  for (int d = lane; d < D; d += 64) {
    float av = 0.f, ak = 0.f;
    for (int i = 0; i < n; ++i) {
      av = fmaf(sp[i], to_f32(dout[tok_row(rows, start + i) * dos + h * D + d]), av);
      ak = fmaf(sds[i], to_f32(q[tok_row(rows, start + i) * qs + h * D + d]), ak);
    }
    from_f32(&dv[tok_row(rows, t) * dvs + h * D + d], av);
    from_f32(&dk[tok_row(rows, t) * dks + h * D + d], scale * ak);
  }
}

// Longest sequence the launch has to expect, and whether the per-token kernels are the faster ones for it.
int longest_of(const AttnShape& s) { return s.max_seqlen < s.T ? s.max_seqlen : s.T; }
// The line is drawn where neither forward nor backward loses by taking the tile kernels; T * H waves is what the token
// kernels start.  Replayed, us, token kernels | tile kernels.  fp32, D = 64, 4 heads, forward; backward:
//   2048 sequences of 1 token 8.6; 24 | 48; 157     of 6 tokens 52; 133 | 55; 167        of 8 tokens 70; 192 | 56; 169
//   4 sequences of 8 tokens 4.6; 9.1 | 4.7; 10.4    of 12 tokens 4.9; 10.0 | 4.7; 10.7   of 16 tokens 5.1; 10.8 | 4.8; 10.5
// bf16, D = 128: 2048 sequences of 12 tokens 171; 490 | 140; 549    of 16 tokens 260; 765 | 135; 514.
bool per_token(const AttnShape& s, mb_dtype dt) {
  const int n = longest_of(s);
  const int64_t waves = (int64_t)s.T * s.H;
  if (s.T > (1 << 25)) return false;   // a launch holds fewer than 2^32 threads per dimension: T waves of 64
  const bool wide_bf16 = dt == MB_BF16 && s.D > 64;   // where the tile kernels have one workgroup per compute unit
  if (n <= 4) return true;
  if (n > kTokenMax || s.D <= 16) return false;
  if (n <= 6) return true;
  if (n <= 8) return s.D > 64 || waves <= 8192;
  if (n <= 12) return wide_bf16 || (s.D > 32 && waves <= 2048);
  return wide_bf16 && waves <= 512;
}

template <typename E>
mb_status fwd_token_t(const AttnShape& s, const void* q, const void* k, const void* v, int64_t qs, int64_t ks, int64_t vs,
                      void* o, int64_t os, float* lse, hipStream_t stream) {
  fwd_token_kernel<E><<<dim3(s.T, s.H), dim3(64), 0, stream>>>((const E*)q, (const E*)k, (const E*)v, qs, ks, vs,
                                                             s.cu_seqlens, s.B, s.T, s.D, s.slopes, s.scale, (E*)o, os,
                                                             lse, s.token_rows, longest_of(s), s.misuse);
  return check_launch("fwd_token_kernel");
}

template <typename E>
mb_status bwd_token_t(const AttnShape& s, const void* dout, const void* q, const void* k, const void* v, const void* o,
                      const float* lse, int64_t dos, int64_t qs, int64_t ks, int64_t vs, int64_t os, void* dq, void* dk,
                      void* dv, int64_t dqs, int64_t dks, int64_t dvs, float* delta, hipStream_t stream) {
  bwd_token_dq_kernel<E><<<dim3(s.T, s.H), dim3(64), 0, stream>>>(
      (const E*)dout, (const E*)q, (const E*)k, (const E*)v, (const E*)o, lse, dos, qs, ks, vs, os, s.cu_seqlens, s.B,
      s.T, s.D, s.slopes, s.scale, (E*)dq, dqs, delta, s.token_rows, longest_of(s), s.misuse);
  const mb_status st = check_launch("bwd_token_dq_kernel");
  if (st != MB_OK) return st;
  bwd_token_dkv_kernel<E><<<dim3(s.T, s.H), dim3(64), 0, stream>>>(
      (const E*)dout, (const E*)q, (const E*)k, (const E*)v, lse, delta, dos, qs, ks, vs, s.cu_seqlens, s.B, s.T, s.D,
      longest_of(s), s.slopes, s.scale, (E*)dk, (E*)dv, dks, dvs, s.token_rows, s.misuse);
  return check_launch("bwd_token_dkv_kernel");
}

// fn<E, NB>(args...) with the head size rounded up to the next instantiated number of 16-column blocks.
#define MB_BY_HEAD_SIZE(fn, E, ...)                       \
  ((s.D <= 16)   ? fn<E, 1>(s, __VA_ARGS__)               \
   : (s.D <= 32) ? fn<E, 2>(s, __VA_ARGS__)               \
   : (s.D <= 48) ? fn<E, 3>(s, __VA_ARGS__)               \
   : (s.D <= 64) ? fn<E, 4>(s, __VA_ARGS__)               \
   : (s.D <= 96) ? fn<E, 6>(s, __VA_ARGS__)               \
                 : fn<E, 8>(s, __VA_ARGS__))

}  // namespace

mb_status launch_attn_fwd_generic(const AttnShape& s, mb_dtype dt, const void* q, const void* k, const void* v,
                                  int64_t qs, int64_t ks, int64_t vs, void* o, int64_t os, float* lse,
                                  hipStream_t stream) {
  if (per_token(s, dt))
    return dt == MB_F32 ? fwd_token_t<float>(s, q, k, v, qs, ks, vs, o, os, lse, stream)
                        : fwd_token_t<uint16_t>(s, q, k, v, qs, ks, vs, o, os, lse, stream);
  return dt == MB_F32 ? MB_BY_HEAD_SIZE(fwd_t, float, q, k, v, qs, ks, vs, o, os, lse, stream)
                      : MB_BY_HEAD_SIZE(fwd_t, uint16_t, q, k, v, qs, ks, vs, o, os, lse, stream);
}

mb_status launch_attn_bwd_generic(const AttnShape& s, mb_dtype dt, const void* dout, const void* q, const void* k,
                                  const void* v, const void* o, const float* lse, int64_t dos, int64_t qs,
                                  int64_t ks, int64_t vs, int64_t os, void* dq, void* dk, void* dv, int64_t dqs,
                                  int64_t dks, int64_t dvs, float* delta_ws, hipStream_t stream) {
  if (per_token(s, dt))
    return dt == MB_F32 ? bwd_token_t<float>(s, dout, q, k, v, o, lse, dos, qs, ks, vs, os, dq, dk, dv, dqs, dks, dvs,
                                             delta_ws, stream)
                        : bwd_token_t<uint16_t>(s, dout, q, k, v, o, lse, dos, qs, ks, vs, os, dq, dk, dv, dqs, dks, dvs,
                                                delta_ws, stream);
  return dt == MB_F32 ? MB_BY_HEAD_SIZE(bwd_t, float, dout, q, k, v, o, lse, dos, qs, ks, vs, os, dq, dk, dv, dqs, dks,
                                        dvs, delta_ws, stream)
                      : MB_BY_HEAD_SIZE(bwd_t, uint16_t, dout, q, k, v, o, lse, dos, qs, ks, vs, os, dq, dk, dv, dqs,
                                        dks, dvs, delta_ws, stream);
}

}  // namespace mb
