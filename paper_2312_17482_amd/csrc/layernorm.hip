// Add & LayerNorm over packed token rows with bf16 (or fp32) storage: the "Low Precision LayerNorm" of the
// paper (LayerNorm reads and writes 2-byte elements because it is bandwidth-bound) together with the
// residual add in front of it ("Add & Norm" in Figure 1A).  Statistics and normalisation are fp32.
//
//   forward :  s = x + r (stored, rounded once),  y = (s - mean) * rstd * gamma + beta
//   backward:  xhat = (s - mean) rstd, g = dy * gamma,
//              ds = rstd * (g - mean(g) - xhat * mean(g * xhat)),  dgamma = sum_t dy * xhat,  dbeta = sum_t dy
//
// One wave per row, 16-byte pieces, every tensor crosses HBM once.  Forward at 26963 x 768 bf16: 30.7 -> 26.1 us (6.3 TB/s)
// since all loads of a row, gamma and beta included, go out together.  The column sums of the backward are
// reduced in a fixed order (per-workgroup partials in the workspace, then one pass over them): no atomics.
#include "common.h"
#include "mfma_util.h"

namespace mb {
namespace {

// 16-byte pieces per lane: 1 for rows up to 1 KB (a load that no lane needs still takes its turn: the forward of 26963 x 64
// floats 12.6 us with two), 2 up to 2 KB (fewer registers, four waves per SIMD), 3 up to 3 KB (with four: 5447 x 520 floats,
// scattered, forward 6.9 us, with three 6.05; 8000 x 1536 bf16 forward and backward 15.9 and 24.4, with three 15.4 and 21.8),
// else 4 (up to 4 KB)
constexpr int kLnThreads = 256;
constexpr int kLnWaves = kLnThreads / 64;

__device__ __forceinline__ float wsum(float x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// Rows move with buffer instructions whose descriptor ends with the row: a lane without a piece reads zeros and stores
// nothing, without a branch that would make its loads wait for the ones before.
template <typename E>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const E* base, int row, int W, bool there = true) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<E*>(base) + (size_t)row * W, 0, there ? W * (int)sizeof(E) : 0, 0x00020000);
}
__device__ __forceinline__ u32x4 get_words(__amdgpu_buffer_rsrc_t r, int piece, u32x4) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, piece * 16, 0, 0);
}
__device__ __forceinline__ u32x2 get_words(__amdgpu_buffer_rsrc_t r, int piece, u32x2) {
  return __builtin_amdgcn_raw_buffer_load_b64(r, piece * 8, 0, 0);
}
__device__ __forceinline__ void put_words(__amdgpu_buffer_rsrc_t r, int piece, u32x4 w) {
  __builtin_amdgcn_raw_buffer_store_b128(w, r, piece * 16, 0, 0);
}
__device__ __forceinline__ void put_words(__amdgpu_buffer_rsrc_t r, int piece, u32x2 w) {
  __builtin_amdgcn_raw_buffer_store_b64(w, r, piece * 8, 0, 0);
}

template <typename E> struct Piece;      // one 16-byte piece of a row <-> floats
template <> struct Piece<uint16_t> {
  static constexpr int kN = 8;
  using Words = u32x4;
  static __device__ __forceinline__ void unpack(Words w, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(w[i] << 16);
      f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ Words pack(const float* f) {   // nearest even; NaN stays NaN
    return Words{pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]), pack_bf16(f[4], f[5]), pack_bf16(f[6], f[7])};
  }
};
// 8-byte pieces of a bf16 row of 256 columns: 64 of them, one per lane, where 16-byte pieces leave half the lanes idle.  Used by
// the forward (26963 x 256: 12.2 -> 11.7 us; 768 columns are 3 x 64 of them, but no faster so since the loads go out
// together: 25.5 against 25.4); the backward was slower with them.
struct HalfPiece {
  static constexpr int kN = 4;
  using Words = u32x2;
  static __device__ __forceinline__ void unpack(Words w, float* f) {
    f[0] = __uint_as_float(w[0] << 16); f[1] = __uint_as_float(w[0] & 0xffff0000u);
    f[2] = __uint_as_float(w[1] << 16); f[3] = __uint_as_float(w[1] & 0xffff0000u);
  }
  static __device__ __forceinline__ Words pack(const float* f) { return Words{pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3])}; }
};
template <> struct Piece<float> {
  static constexpr int kN = 4;
  using Words = u32x4;
  static __device__ __forceinline__ void unpack(Words w, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(w[i]);
  }
  static __device__ __forceinline__ Words pack(const float* f) {
    return Words{__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])};
  }
};

template <typename E, int kMaxPieces, typename PT = Piece<E>>
__global__ __launch_bounds__(kLnThreads) void add_layernorm_fwd_kernel(
    const E* __restrict__ x, const E* __restrict__ r, const E* __restrict__ gamma, const E* __restrict__ beta,
    int T_cap, const int32_t* __restrict__ meta, int W, float eps, E* __restrict__ y, E* __restrict__ s,
    float* __restrict__ mean, float* __restrict__ rstd, const int32_t* __restrict__ y_rows) {
  using Words = typename PT::Words;
  constexpr int N = PT::kN;
  const int T = meta ? min(meta[0], T_cap) : T_cap;
  const int row = blockIdx.x * kLnWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= T) return;
  const int lane = threadIdx.x & 63;
  const int pieces = W / N;
  Words wx[kMaxPieces], wr[kMaxPieces], wg[kMaxPieces], wb[kMaxPieces];   // every load of the row, in one go
  const __amdgpu_buffer_rsrc_t xr = row_rsrc(x, row, W), rr = row_rsrc(r, row, W, r != nullptr);
#pragma unroll
  for (int c = 0; c < kMaxPieces; ++c) {
    wx[c] = get_words(xr, lane + 64 * c, Words{});
    wr[c] = get_words(rr, lane + 64 * c, Words{});
  }
#pragma unroll
  for (int c = 0; c < kMaxPieces; ++c) {
    wg[c] = get_words(row_rsrc(gamma, 0, W), lane + 64 * c, Words{});
    wb[c] = get_words(row_rsrc(beta, 0, W), lane + 64 * c, Words{});
  }
  float v[kMaxPieces][N];
  float sum = 0.f;
#pragma unroll
  for (int c = 0; c < kMaxPieces; ++c) {
    PT::unpack(wx[c], v[c]);
    if (r) {
      float t[N];
      PT::unpack(wr[c], t);
#pragma unroll
      for (int i = 0; i < N; ++i) v[c][i] += t[i];
      const Words w = PT::pack(v[c]);
      put_words(row_rsrc(s, row, W), lane + 64 * c, w);
      PT::unpack(w, v[c]);   // the stored sum is what is normalised
    }
#pragma unroll
    for (int i = 0; i < N; ++i) sum += v[c][i];
  }
  const float mu = wsum(sum) / (float)W;
  float sq = 0.f;
#pragma unroll
  for (int c = 0; c < kMaxPieces; ++c) {
    if (lane + 64 * c < pieces) {
#pragma unroll
      for (int i = 0; i < N; ++i) { const float d = v[c][i] - mu; sq = fmaf(d, d, sq); }
    }
  }
  const float rs = rsqrtf(wsum(sq) / (float)W + eps);
  const __amdgpu_buffer_rsrc_t yr = row_rsrc(y, tok_row(y_rows, row), W);   // packed row, or the token's in the padded batch
#pragma unroll
  for (int c = 0; c < kMaxPieces; ++c) {
    float g[N], b[N], out[N];
    PT::unpack(wg[c], g);
    PT::unpack(wb[c], b);
#pragma unroll
    for (int i = 0; i < N; ++i) out[i] = fmaf((v[c][i] - mu) * rs, g[i], b[i]);
    put_words(yr, lane + 64 * c, PT::pack(out));
  }
  if (lane == 0) { mean[row] = mu; rstd[row] = rs; }
}

// Each wave walks rows  blockIdx*4 + wave, + 4*gridDim, ...: writes ds and keeps per-lane partial column
// sums; the four waves of a block are then added in a fixed order and written to part[block][2][W].
//
// Bound by memory, so the requests must not wait for one another: all loads of a row go out before the first is used, and
// with one or two pieces per lane, where the registers allow it at four waves per SIMD, the next row's go out before this
// row's arithmetic.  26963 x 768: 27.5 -> 23.2 us (5.4 TB/s); with a branch and a conversion behind each load every piece waited
// for the one before it.
template <typename E, int kMaxPieces>
__global__ __launch_bounds__(kLnThreads, kMaxPieces <= 2 ? 4 : 2) void add_layernorm_bwd_kernel(
    const E* __restrict__ dy, const E* __restrict__ s, const E* __restrict__ gamma, const float* __restrict__ mean,
    const float* __restrict__ rstd, int T_cap, const int32_t* __restrict__ meta, int W, E* __restrict__ ds,
    float* __restrict__ part, const int32_t* __restrict__ dy_rows) {
  using PT = Piece<E>;
  using Words = typename PT::Words;
  constexpr int N = PT::kN;
  constexpr bool kAhead = kMaxPieces <= 2;
  extern __shared__ float lds[];   // [kLnWaves][2][W]
  const int T = meta ? min(meta[0], T_cap) : T_cap;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pieces = W / N;
  float g[kMaxPieces][N], ag[kMaxPieces][N], ab[kMaxPieces][N];
#pragma unroll
  for (int c = 0; c < kMaxPieces; ++c) {
#pragma unroll
    for (int i = 0; i < N; ++i) { ag[c][i] = 0.f; ab[c][i] = 0.f; }
    PT::unpack(get_words(row_rsrc(gamma, 0, W), lane + 64 * c, Words{}), g[c]);
  }
  const int stride = gridDim.x * kLnWaves;
  Words ws[kMaxPieces], wd[kMaxPieces];
  float mu = 0.f, rs = 0.f;
  auto request = [&](int row, bool there) {   // packed row of dy, or the token's row in the padded batch
    const __amdgpu_buffer_rsrc_t sr = row_rsrc(s, row, W, there), dr = row_rsrc(dy, tok_row(dy_rows, row), W, there);
#pragma unroll
    for (int c = 0; c < kMaxPieces; ++c) {
      ws[c] = get_words(sr, lane + 64 * c, Words{});
      wd[c] = get_words(dr, lane + 64 * c, Words{});
    }
    mu = mean[row];
    rs = rstd[row];
  };
  int row = blockIdx.x * kLnWaves + wave;
  if (row < T) {
    if (kAhead) {
      request(row, true);
      // as many stores behind the first row's loads as behind every other's (these go nowhere): the wait for a row's loads
      // then never includes the stores of the row before
#pragma unroll
      for (int c = 0; c < kMaxPieces; ++c) put_words(row_rsrc(ds, row, W, false), lane + 64 * c, Words{});
    }
#pragma unroll 1
    for (; row < T; row += stride) {
      if (!kAhead) request(row, true);
      float xh[kMaxPieces][N], gy[kMaxPieces][N];
      float c1 = 0.f, c2 = 0.f;
      const float m = mu, r = rs;
#pragma unroll
      for (int c = 0; c < kMaxPieces; ++c) {
        PT::unpack(ws[c], xh[c]);
        PT::unpack(wd[c], gy[c]);
      }
      if (kAhead) request(row + stride < T ? row + stride : row, row + stride < T);
#pragma unroll
      for (int c = 0; c < kMaxPieces; ++c) {
        const bool in = lane + 64 * c < pieces;   // (a lane without a piece adds zeros whatever the statistics are)
        const float mc = in ? m : 0.f, rc = in ? r : 0.f;
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const float d = gy[c][i];
          xh[c][i] = (xh[c][i] - mc) * rc;
          ag[c][i] = fmaf(d, xh[c][i], ag[c][i]);
          ab[c][i] += d;
          gy[c][i] = d * g[c][i];
          c1 += gy[c][i];
          c2 = fmaf(gy[c][i], xh[c][i], c2);
        }
      }
      c1 = wsum(c1) / (float)W;
      c2 = wsum(c2) / (float)W;
#pragma unroll
      for (int c = 0; c < kMaxPieces; ++c) {
        float out[N];
#pragma unroll
        for (int i = 0; i < N; ++i) out[i] = r * (gy[c][i] - c1 - xh[c][i] * c2);
        put_words(row_rsrc(ds, row, W), lane + 64 * c, PT::pack(out));
      }
    }
  }
#pragma unroll
  for (int c = 0; c < kMaxPieces; ++c) {
    const int pc = lane + 64 * c;
    if (pc < pieces) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        lds[(wave * 2 + 0) * W + pc * N + i] = ag[c][i];
        lds[(wave * 2 + 1) * W + pc * N + i] = ab[c][i];
      }
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < 2 * W; idx += kLnThreads) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < kLnWaves; ++w) t += lds[w * 2 * W + idx];
    part[(size_t)blockIdx.x * 2 * W + idx] = t;
  }
}

// dgamma[w], dbeta[w] = sum over the `nparts` partial rows, in a fixed order.  32 columns (a cache line) per block; the partial
// rows are dealt to 32 half waves x 16 independent accumulators: the kernel is a chain of memory round trips, nothing else, so it
// wants many loads in flight and many blocks (1024 rows of 2 x 768: 4.4 us, 24 blocks of 64 columns 5.3; 237 rows 2.5 times as
// fast as with single loads for the rest of 256).  Rows past the end read as zeros.
constexpr int kColsumSlices = 32, kColsumColumns = 32;
__global__ __launch_bounds__(kColsumSlices * kColsumColumns) void add_layernorm_colsum_kernel(
    const float* __restrict__ part, int nparts, int W, float* __restrict__ dgamma, float* __restrict__ dbeta) {
  __shared__ float red[kColsumSlices][kColsumColumns];
  const int l = threadIdx.x % kColsumColumns;
  const int idx = blockIdx.x * kColsumColumns + l;
  const int slice = threadIdx.x / kColsumColumns;
  constexpr int kAcc = 16;
  const uint32_t pitch = 2u * (uint32_t)W * 4u;   // at most 1024 partial rows of 16 KB
  const __amdgpu_buffer_rsrc_t rows =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(part), 0, (int)((uint32_t)nparts * pitch), 0x00020000);
  float acc[kAcc];
#pragma unroll
  for (int u = 0; u < kAcc; ++u) acc[u] = 0.f;
  for (int p = slice; p < nparts; p += kAcc * kColsumSlices) {
    float x[kAcc];
#pragma unroll
    for (int u = 0; u < kAcc; ++u)
      x[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows, (uint32_t)(p + kColsumSlices * u) * pitch + idx * 4u, 0, 0));
#pragma unroll
    for (int u = 0; u < kAcc; ++u) acc[u] += x[u];
  }
#pragma unroll
  for (int w = kAcc / 2; w > 0; w >>= 1)
#pragma unroll
    for (int u = 0; u < w; ++u) acc[u] += acc[u + w];
  red[slice][l] = acc[0];
  __syncthreads();
  if (slice == 0 && idx < 2 * W) {
    float t = 0.f;
#pragma unroll
    for (int sl = 0; sl < kColsumSlices; ++sl) t += red[sl][l];
    if (idx < W) dgamma[idx] = t; else dbeta[idx - W] = t;
  }
}

int bwd_blocks(int T_cap) { return max(1, min((T_cap + kLnWaves - 1) / kLnWaves, kLayerNormMaxParts)); }

}  // namespace

#define MB_LN_PIECES(LAUNCH, E)       \
  if (bytes <= 1024) LAUNCH(E, 1);      \
  else if (bytes <= 2048) LAUNCH(E, 2); \
  else if (bytes <= 3072) LAUNCH(E, 3); \
  else LAUNCH(E, 4)

mb_status launch_add_layernorm_fwd(mb_dtype dt, const void* x, const void* r, const void* gamma, const void* beta,
                                   int T_cap, const int32_t* meta, int W, float eps, void* y, void* s, float* mean,
                                   float* rstd, const int32_t* y_rows, hipStream_t stream) {
  const int blocks = (T_cap + kLnWaves - 1) / kLnWaves;
  const size_t bytes = (size_t)W * elem_size(dt);
#define MB_LN_FWD(E, P)                                                                                           \
  hipLaunchKernelGGL((add_layernorm_fwd_kernel<E, P>), dim3(blocks), dim3(kLnThreads), 0, stream, (const E*)x,    \
                     (const E*)r, (const E*)gamma, (const E*)beta, T_cap, meta, W, eps, (E*)y, (E*)s, mean, rstd,  \
                     y_rows)
  if (dt == MB_BF16 && W == 256) {   // (HalfPiece)
    hipLaunchKernelGGL((add_layernorm_fwd_kernel<uint16_t, 1, HalfPiece>), dim3(blocks), dim3(kLnThreads), 0, stream,
                       (const uint16_t*)x, (const uint16_t*)r, (const uint16_t*)gamma, (const uint16_t*)beta, T_cap, meta, W,
                       eps, (uint16_t*)y, (uint16_t*)s, mean, rstd, y_rows);
  } else if (dt == MB_BF16) {
    MB_LN_PIECES(MB_LN_FWD, uint16_t);
  } else {
    MB_LN_PIECES(MB_LN_FWD, float);
  }
#undef MB_LN_FWD
  return check_launch("add_layernorm_fwd_kernel");
}

mb_status launch_add_layernorm_bwd(mb_dtype dt, const void* dy, const void* s, const void* gamma, const float* mean,
                                   const float* rstd, int T_cap, const int32_t* meta, int W, void* ds, float* dgamma,
                                   float* dbeta, float* part, const int32_t* dy_rows, hipStream_t stream) {
  if (T_cap == 0) {
    // no rows (dy, s, gamma, ... may be NULL): nothing to read, the column sums are zeros
    hipLaunchKernelGGL(add_layernorm_colsum_kernel, dim3((2 * W + kColsumColumns - 1) / kColsumColumns),
                       dim3(kColsumSlices * kColsumColumns), 0, stream, part, 0, W,
                       dgamma, dbeta);
    return check_launch("add_layernorm_colsum_kernel");
  }
  const int blocks = bwd_blocks(T_cap);
  const size_t smem = sizeof(float) * kLnWaves * 2 * (size_t)W;
  const size_t bytes = (size_t)W * elem_size(dt);
#define MB_LN_BWD(E, P)                                                                                          \
  hipLaunchKernelGGL((add_layernorm_bwd_kernel<E, P>), dim3(blocks), dim3(kLnThreads), smem, stream,             \
                     (const E*)dy, (const E*)s, (const E*)gamma, mean, rstd, T_cap, meta, W, (E*)ds, part, dy_rows)
  if (dt == MB_BF16) {
    MB_LN_PIECES(MB_LN_BWD, uint16_t);
  } else {
    MB_LN_PIECES(MB_LN_BWD, float);
  }
#undef MB_LN_BWD
  mb_status st = check_launch("add_layernorm_bwd_kernel");
  if (st != MB_OK) return st;
  hipLaunchKernelGGL(add_layernorm_colsum_kernel, dim3((2 * W + kColsumColumns - 1) / kColsumColumns),
                       dim3(kColsumSlices * kColsumColumns), 0, stream, part, blocks, W,
                     dgamma, dbeta);
  return check_launch("add_layernorm_colsum_kernel");
}

}  // namespace mb
