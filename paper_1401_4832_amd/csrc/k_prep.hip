// k_prep.hip -- everything an evaluation needs before its first forward, in one
// launch: the alignment's internal copies (chunk-major, position-major and by
// position triples), the residual rows no forward tile writes, the check of the
// weights and the scale of path 0's residual digits, and, for a standalone
// evaluation, the work tables.  The parts are independent of each other and
// take different blocks.
// Bound: HBM (the symbols read once, written two or three times) for large
// alignments, one launch's latency for small ones: N = 500, B = 50 000
// 130 us in three passes -> 36 us, N = 40, B = 500 8 us where six
// launches took 19.
#include "plm_internal.h"

namespace plm {

constexpr int kPrThreads = 256;
constexpr int kPrRows = 256;            // rows of a tile: one gradient chunk
constexpr int kPrCols = 48;             // columns: three chunks of sixteen, sixteen triples
constexpr int kPrPitch = kPrCols + 4;   // LDS bytes per row: an odd number of words
static_assert(kPrPitch % 4 == 0 && kFwdChunk % 4 == 0, "rows and chunks are read as words");
constexpr int kPrZeroBlocks = 64;

// The symbols of one tile, zeros past B and N; symbols >= q become zero and
// raise bit 1 of *flag.
__device__ inline void prep_tile(const PrepArgs& a, int rt, int ct, uint8_t* sh) {
  const int tid = threadIdx.x, b0 = rt * kPrRows, i0 = ct * kPrCols;
  constexpr int kPer = kPrRows * kPrCols / kPrThreads, kBatch = 16;
  static_assert(kPer % kBatch == 0, "whole batches");
  bool bad = false;
  for (int k0 = 0; k0 < kPer; k0 += kBatch) {
    uint32_t v[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int e = tid + (k0 + k) * kPrThreads, b = b0 + e / kPrCols, i = i0 + e % kPrCols;
      v[k] = b < a.B && i < a.N ? a.msa[(size_t)b * a.N + i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int e = tid + (k0 + k) * kPrThreads;
      const bool over = v[k] >= (uint32_t)a.q;
      bad |= over;
      sh[(e / kPrCols) * kPrPitch + e % kPrCols] = (uint8_t)(over ? 0u : v[k]);
    }
  }
  if (bad && a.flag) atomicOr(a.flag, 1);
  __syncthreads();
  // chunk-major: symbol (b, i) at ((i / 16) * B_pad + b) * 16 + i % 16
  const int b = b0 + tid;
  const uint8_t* row = sh + tid * kPrPitch;
#pragma unroll
  for (int c = 0; c < kPrCols / kFwdChunk; ++c) {
    const int i = i0 + c * kFwdChunk;
    if (i >= a.N_pad) break;
    const uint32_t* p = reinterpret_cast<const uint32_t*>(row + c * kFwdChunk);
    *reinterpret_cast<uint4*>(a.msa_cm + ((size_t)(i / kFwdChunk) * a.B_pad + b) * kFwdChunk) =
        make_uint4(p[0], p[1], p[2], p[3]);
  }
  if (a.msaT) {
    // position-major: (b, i) at i * B_pad + b, sixteen rows of a column per store
#pragma unroll
    for (int k = 0; k < kPrCols * (kPrRows / 16) / kPrThreads; ++k) {
      const int e = tid + k * kPrThreads, g = e & 15, c = e >> 4, i = i0 + c;
      if (i >= a.N_pad) continue;
      uint32_t w[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        w[t] = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) w[t] |= (uint32_t)sh[(16 * g + 4 * t + u) * kPrPitch + c] << (8 * u);
      }
      *reinterpret_cast<uint4*>(a.msaT + (size_t)i * a.B_pad + b0 + 16 * g) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
  if (a.sym3) {
#pragma unroll 4
    for (int t = 0; t < kPrCols / 3; ++t) {
      const int G = ct * (kPrCols / 3) + t;
      if (G >= a.NG) break;
      a.sym3[(size_t)G * a.B_pad + b] =
          (uint32_t)row[3 * t] | ((uint32_t)row[3 * t + 1] << 8) | ((uint32_t)row[3 * t + 2] << 16);
    }
  }
}

// Zeros in the residual rows [B rounded down to 256, B3 rounded up to 256) of
// every site (grouped gradients): the forward writes only the rows of its
// tiles, and the last gradient chunk may reach past them.
__device__ inline void prep_zero(const PrepArgs& a, int blk) {
  const int64_t per = (int64_t)(a.zc1 - a.zc0) * a.chunk16, total = per * a.N;
  for (int64_t e = (int64_t)blk * kPrThreads + threadIdx.x; e < total; e += (int64_t)kPrZeroBlocks * kPrThreads) {
    const int64_t r = e / per, k = e - r * per;
    const int64_t at = (r * (a.B_pad >> 8) + a.zc0) * a.chunk16 + k;
    a.zero0[at] = make_uint4(0, 0, 0, 0);
    if (a.zero1) a.zero1[at] = make_uint4(0, 0, 0, 0);
  }
}

// Raises bit 2 of *flag for a non-finite weight; wexp (if any) receives the
// smallest exponent e with every |w_b| <= 2^e (0 for all-zero weights), and
// whether a weight that is not zero lies below 2^(e - kR4RangeLog2), which goes
// to *wide too.
__device__ inline void prep_weights(const PrepArgs& a) {
  __shared__ double red[2][kPrThreads / 64];
  double mx = 0.0, mn = INFINITY;
  bool bad = false;
#pragma unroll 16
  for (int b = threadIdx.x; b < a.B; b += kPrThreads) {
    const double v = fabs(a.w[b]);
    bad |= !isfinite(v);
    mx = fmax(mx, v);
    mn = fmin(mn, v > 0.0 ? v : INFINITY);
  }
  if (bad && a.flag) atomicOr(a.flag, 2);
  if (!a.wexp) {
    if (threadIdx.x == 0) *a.wide = 0;
    return;
  }
  for (int o = 32; o > 0; o >>= 1) {
    mx = fmax(mx, __shfl_xor(mx, o, 64));
    mn = fmin(mn, __shfl_xor(mn, o, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = mx;
    red[1][threadIdx.x >> 6] = mn;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kPrThreads / 64; ++k) {
      mx = fmax(mx, red[0][k]);
      mn = fmin(mn, red[1][k]);
    }
    int e = 0;
    if (mx > 0.0 && isfinite(mx)) {
      const double m = frexp(mx, &e);  // m in [0.5, 1)
      if (m == 0.5) --e;
    }
    a.wexp[0] = e;
    a.wexp[1] = *a.wide = mn < ldexp(1.0, e - kR4RangeLog2);
  }
}

// Blocks: [0] the tables (table = 1), then [1] the weights, kPrZeroBlocks of
// zeros (if there are any to write), and one per tile, columns first.
__global__ __launch_bounds__(kPrThreads) void prep_kernel(PrepArgs a, TableArgs t, int32_t table, int32_t nzero,
                                                          int32_t col_tiles) {
  __shared__ __attribute__((aligned(16))) uint8_t sh[kPrRows * kPrPitch];
  int blk = blockIdx.x;
  if (table) {
    if (blk == 0) {
      write_eval_tables(t, a.flag);
      if (a.tables_only && threadIdx.x == 0) *a.wide = a.wexp ? a.wexp[1] : 0;  // (the weights' block is not run)
      return;
    }
    --blk;
  }
  if (blk == 0) {
    prep_weights(a);
    return;
  }
  --blk;
  if (blk < nzero) {
    prep_zero(a, blk);
    return;
  }
  blk -= nzero;
  prep_tile(a, blk / col_tiles, blk % col_tiles, sh);
}

hipError_t launch_prepare(const PrepArgs& a, const TableArgs* t, hipStream_t st) {
  const int col_tiles = (a.N_pad + kPrCols - 1) / kPrCols;
  const int64_t tiles = (int64_t)(a.B_pad / kPrRows) * col_tiles;
  const int nzero = a.zero0 && a.zc0 < a.zc1 ? kPrZeroBlocks : 0;
  const int64_t grid = a.tables_only ? 1 : tiles + nzero + 1 + (t ? 1 : 0);
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(prep_kernel, dim3((unsigned)grid), dim3(kPrThreads), 0, st, a, t ? *t : TableArgs{}, t ? 1 : 0,
                     nzero, col_tiles);
  return hipGetLastError();
}

}  // namespace plm
