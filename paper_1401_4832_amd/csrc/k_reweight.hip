// k_reweight.hip -- sequence reweighting (sec. 3.1, eq. inverse_weights;
// sec. 3.4 step 2, eq. inverse_weights2).
//
// id(a,b) = number of columns where rows a and b hold the same symbol (gap =
// gap counts).  Symbols take five bits (q <= 21), so 32 columns of a row are
// five bit planes of one 32-bit word each, and the columns where two rows
// differ are the OR over the planes of the XOR of their words: five
// three-operand bit operations and one accumulating popcount per pair and 32
// columns.  Bound: integer ALU, 6 operations per 32 columns (four-symbol byte
// compares take 5 per 4 columns).  Each block compares a square tile of row
// pairs (upper triangle only); counts m_b are integer atomics, so the result
// does not depend on scheduling.  Measured: identity counts of N = 500,
// B = 50 000 26.3 -> 3.2 ms (all columns at the full integer rate would take
// 3.1 ms; a part is skipped, see identity_kernel), of N = 120, B = 5000
// 87 -> 23 us; B_eff (beff_kernel) 3820 -> 57 us and 336 -> 20 us.
#include "plm_internal.h"

namespace plm {

constexpr int kRwThreads = 256;
constexpr int kRwWords = 4;   // plane words (32 columns each) staged per chunk
constexpr int kRwPlanes = 5;  // bits of a symbol
static_assert(kQMax <= (1 << kRwPlanes), "symbols fit the planes");

__global__ void fill_i32_kernel(int32_t* p, int32_t v, int32_t n) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) p[e] = v;
}

// x where the mask has ones, y elsewhere
__device__ inline uint32_t bit_select(uint32_t mask, uint32_t x, uint32_t y) { return (mask & x) | (~mask & y); }

// 32 symbols (eight words of four) to their five bit planes: the 8 x 8 bit
// matrix of every byte column over the eight words, transposed by three
// rounds of masked swaps (planes 5..7, all zero, left out).  The order of the
// columns within a plane word is the same for every row.
__device__ inline void bit_planes(const uint32_t (&d)[8], uint32_t (&pl)[kRwPlanes]) {
  uint32_t ev[4], od[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    ev[j] = bit_select(0x55555555u, d[2 * j], d[2 * j + 1] << 1);
    od[j] = bit_select(0x55555555u, d[2 * j] >> 1, d[2 * j + 1]);
  }
  uint32_t p04[2], p26[2], p15[2], p37[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    p04[j] = bit_select(0x33333333u, ev[2 * j], ev[2 * j + 1] << 2);
    p26[j] = bit_select(0x33333333u, ev[2 * j] >> 2, ev[2 * j + 1]);
    p15[j] = bit_select(0x33333333u, od[2 * j], od[2 * j + 1] << 2);
    p37[j] = bit_select(0x33333333u, od[2 * j] >> 2, od[2 * j + 1]);
  }
  pl[0] = bit_select(0x0f0f0f0fu, p04[0], p04[1] << 4);
  pl[1] = bit_select(0x0f0f0f0fu, p15[0], p15[1] << 4);
  pl[2] = bit_select(0x0f0f0f0fu, p26[0], p26[1] << 4);
  pl[3] = bit_select(0x0f0f0f0fu, p37[0], p37[1] << 4);
  pl[4] = bit_select(0x0f0f0f0fu, p04[0] >> 4, p04[1]);
}

// One block: a tile of 16 U x 16 U row pairs, U x U pairs per thread in
// registers.  Chunks of kRwWords plane words are double-buffered in LDS: the
// next chunk's symbols are loaded while the current chunk is compared.  A wave
// whose pairs all differ in more than maxdiff columns already skips the
// remaining compares, and the block ends once every wave has: unrelated rows
// are settled after a fraction of their columns.
template <int U>
__global__ __launch_bounds__(kRwThreads, U == 8 ? 2 : 4) void identity_kernel(const uint8_t* __restrict__ msa, int32_t B, int32_t N,
                                                              int32_t q, int32_t maxdiff, int32_t* __restrict__ m,
                                                              int32_t* flag) {
  constexpr int kTile = 16 * U;
  // row pitch: 16-byte aligned, and the words a wave converts together fall into different banks
  constexpr int kPitch = kTile + 4;
  constexpr int kUnits = 2 * kTile * kRwWords / kRwThreads;  // (side, row, word) units per thread and chunk
  __shared__ __attribute__((aligned(16))) uint32_t S[2][2][kRwWords * kRwPlanes * kPitch];
  __shared__ int32_t cntA[kTile], cntB[kTile];
  __shared__ int32_t live[3];
  const int ta = blockIdx.y, tb = blockIdx.x;
  if (tb < ta) return;
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  for (int e = tid; e < kTile; e += kRwThreads) {
    cntA[e] = 0;
    cntB[e] = 0;
  }
  if (tid < 3) live[tid] = 0;
  uint32_t nz[U][U];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int v = 0; v < U; ++v) nz[u][v] = 0;
  const int W = (N + 31) / 32, nchunks = (W + kRwWords - 1) / kRwWords;
  uint32_t raw[kUnits][8];
  // unit k of this thread: side (0: rows of ta, 1: rows of tb), row of the tile, word of the chunk
  auto unit = [&](int k, int& side, int& row, int& wd) {
    const int e = tid + k * kRwThreads;
    wd = e % kRwWords;
    const int sr = e / kRwWords;
    side = sr / kTile;
    row = sr - side * kTile;
  };
  auto load = [&](int c) {
#pragma unroll
    for (int k = 0; k < kUnits; ++k) {
      int side, row, wd;
      unit(k, side, row, wd);
      const int rr = (side ? tb : ta) * kTile + row, col = 32 * (c * kRwWords + wd);
#pragma unroll
      for (int j = 0; j < 8; ++j) raw[k][j] = 0;
      if (rr < B && col < N) {
        if (N >= 32) {
          // the row's last word is read as its last 32 columns, with the
          // columns of earlier words cleared (zero on both sides: they agree)
          const int skip = max(0, col + 32 - N);
          __builtin_memcpy(raw[k], msa + (size_t)rr * N + col - skip, 32);  // rows start at any byte
          if (skip) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const int n = min(max(skip - 4 * j, 0), 4);
              raw[k][j] = n == 4 ? 0u : raw[k][j] & (~0u << (8 * n));
            }
          }
        } else {
#pragma unroll
          for (int j = 0; j < 32; ++j)
            if (j < N) raw[k][j >> 2] |= (uint32_t)msa[(size_t)rr * N + j] << (8 * (j & 3));
        }
      }
    }
  };
  uint32_t bad = 0;
  auto store = [&](int buf) {
#pragma unroll
    for (int k = 0; k < kUnits; ++k) {
      int side, row, wd;
      unit(k, side, row, wd);
      if (ta == tb) {  // every row is on one diagonal tile: symbols >= q are found there
#pragma unroll
        for (int j = 0; j < 8; ++j)
          bad |= ((raw[k][j] & 0x7f7f7f7fu) + (0x80u - (uint32_t)q) * 0x01010101u) | raw[k][j];
      }
      uint32_t pl[kRwPlanes];
      bit_planes(raw[k], pl);
#pragma unroll
      for (int p = 0; p < kRwPlanes; ++p) S[buf][side][(wd * kRwPlanes + p) * kPitch + row] = pl[p];
    }
  };
  load(0);
  store(0);
  __syncthreads();
  bool open = true;  // some pair of this wave may still reach the threshold
  for (int c = 0; c < nchunks; ++c) {
    const int buf = c & 1;
    const bool more = c + 1 < nchunks;
    if (more) load(c + 1);
    if (open) {
      const int nw = min(kRwWords, W - c * kRwWords);
      for (int wd = 0; wd < nw; ++wd) {
        uint32_t x[U][U];
#pragma unroll
        for (int p = 0; p < kRwPlanes; ++p) {
          const uint32_t* A = &S[buf][0][(wd * kRwPlanes + p) * kPitch];
          const uint32_t* Bp = &S[buf][1][(wd * kRwPlanes + p) * kPitch];
          uint32_t a[U], b[U];
          // rows 4 ty + u (+ 64 for u >= 4): sixteen lanes read contiguous 16-byte words
#pragma unroll
          for (int g = 0; g < U / 4; ++g) {
            const uint4 av = *reinterpret_cast<const uint4*>(A + g * 64 + ty * 4);
            const uint4 bv = *reinterpret_cast<const uint4*>(Bp + g * 64 + tx * 4);
            a[4 * g] = av.x; a[4 * g + 1] = av.y; a[4 * g + 2] = av.z; a[4 * g + 3] = av.w;
            b[4 * g] = bv.x; b[4 * g + 1] = bv.y; b[4 * g + 2] = bv.z; b[4 * g + 3] = bv.w;
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < U; ++v)
              x[u][v] = p == 0 ? a[u] ^ b[v] : __builtin_amdgcn_bitop3_b32(a[u], b[v], x[u][v], 0xbe);  // (a ^ b) | x
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int v = 0; v < U; ++v) nz[u][v] += __popc(x[u][v]);
      }
      uint32_t lo = nz[0][0];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < U; ++v) lo = min(lo, nz[u][v]);
      open = __any((int)lo <= maxdiff);
    }
    if (!more) break;
    // three flags in turn: one is set, one read, one cleared between two barriers
    if (open && (tid & 63) == 0) live[c % 3] = 1;
    store(buf ^ 1);
    __syncthreads();
    if (!live[c % 3] && ta != tb) break;  // (a diagonal tile goes on: it checks every symbol)
    if (tid == 0) live[(c + 2) % 3] = 0;
  }
  if (__any(bad & 0x80808080u) && (tid & 63) == 0 && flag) atomicOr(flag, 1);
  if (open) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int v = 0; v < U; ++v) {
        const int la = (u >> 2) * 64 + ty * 4 + (u & 3), lb = (v >> 2) * 64 + tx * 4 + (v & 3);
        const int a = ta * kTile + la, b = tb * kTile + lb;
        if ((int)nz[u][v] <= maxdiff && a < B && b < B && a <= b) {
          atomicAdd(&cntA[la], 1);
          if (a != b) atomicAdd(&cntB[lb], 1);
        }
      }
  }
  __syncthreads();
  for (int e = tid; e < kTile; e += kRwThreads) {
    const int a = ta * kTile + e, b = tb * kTile + e;
    if (a < B && cntA[e]) atomicAdd(&m[a], cntA[e]);
    if (b < B && cntB[e]) atomicAdd(&m[b], cntB[e]);
  }
}

// w_b = 1/m_b (IEEE division, correctly rounded)
__global__ void weights_kernel(const int32_t* m, int32_t B, int32_t uniform, double* w) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) w[b] = uniform ? 1.0 : 1.0 / (double)m[b];
}

// B_eff: the weights added in index order, each sum rounded, bit for bit what
// one thread adding them one by one gets.  While the running sum t stays
// within one binade (t in [2^k, 2^(k+1)), spacing u = 2^(k-52)), adding w
// rounds w to a multiple of u -- the same multiple whatever t is, unless w
// lies halfway between two -- so the sum of a run of weights is a sum of
// integers w/u, exact in any order.  One wave takes runs of 64 * kSumWide
// weights that way (t, the run's integers and their sum below 2^53, no
// halfway case); a run that fails is cut into runs of 64 * kSumRun, and one of
// those that fails is added one by one.  Bound: latency of one wave (the
// one-by-one loop over global memory took 80 cycles a weight).
constexpr int kSumThreads = 256;
constexpr int kSumWide = 32;
constexpr int kSumRun = 4;
constexpr int kSumTile = 64 * kSumWide;  // weights staged in LDS at a time

// adds the integers of V * 64 weights at x to t where that is exact; false leaves t as it was
template <int V>
__device__ inline bool sum_run(const double* x, int lane, double& t) {
  if (!(t >= 1.0)) return false;
  const uint64_t ex = (uint64_t)__double_as_longlong(t) >> 52;            // biased exponent, 1023 + k
  const double sc = __longlong_as_double((long long)((1023 + 1023 + 52 - ex) << 52));  // 1/u
  double sum = 0.0;
  bool half = false;
#pragma unroll
  for (int j = 0; j < V; ++j) {
    const double y = x[j * 64 + lane] * sc, n = rint(y);
    half |= fabs(y - n) == 0.5;
    sum += n;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  const double T = t * sc + sum;
  if (__any(half) || !(T < 9007199254740992.0)) return false;
  t = T / sc;  // a power of two: exact
  return true;
}

__global__ __launch_bounds__(kSumThreads) void beff_kernel(const double* __restrict__ w, int32_t B,
                                                           double* __restrict__ beff) {
  __shared__ double buf[2][kSumTile];
  constexpr int kPer = kSumTile / kSumThreads;
  const int tid = threadIdx.x, lane = tid & 63;
  const int ntile = (B + kSumTile - 1) / kSumTile;
  double r[kPer];
  auto load = [&](int c) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int b = c * kSumTile + tid + k * kSumThreads;
      r[k] = b < B ? w[b] : 0.0;
    }
  };
  auto store = [&](int c) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) buf[c & 1][tid + k * kSumThreads] = r[k];
  };
  load(0);
  store(0);
  double t = 0.0;
  for (int c = 0; c < ntile; ++c) {
    __syncthreads();
    if (c + 1 < ntile) load(c + 1);
    if (tid < 64) {
      const double* x = buf[c & 1];
      if (!sum_run<kSumWide>(x, lane, t)) {
        for (int g = 0; g < kSumTile; g += 64 * kSumRun) {
          if (sum_run<kSumRun>(x + g, lane, t)) continue;
#pragma unroll 16
          for (int j = 0; j < 64 * kSumRun; ++j) t += x[g + j];  // (zeros past B change nothing)
        }
      }
    }
    if (c + 1 < ntile) store(c + 1);
  }
  if (tid == 0) *beff = t;
}

int32_t identity_threshold(int32_t N, double theta) {
  // smallest integer id with (double)id / (double)N >= theta: the comparison the
  // definition makes, evaluated once per id on the host
  for (int32_t t = 0; t <= N; ++t)
    if ((double)t / (double)N >= theta) return t;
  return N + 1;
}

// Tiles of 128 rows (64 pairs per thread in registers: two LDS operands per
// eight compares) once they make several per CU; smaller alignments take
// 64-row tiles, four times as many.
constexpr int kRwWideRows = 8192;

hipError_t launch_reweight(const uint8_t* msa, int32_t B, int32_t N, int32_t q, double theta,
                           int32_t uniform, int32_t* m, double* w, double* beff, int32_t* flag,
                           hipStream_t st) {
  const int fb = (B + 255) / 256 < 4096 ? (B + 255) / 256 : 4096;
  hipLaunchKernelGGL(fill_i32_kernel, dim3(fb), dim3(256), 0, st, m, uniform ? 1 : 0, B);
  if (!uniform) {
    const int maxdiff = N - identity_threshold(N, theta);
    const int tile = B >= kRwWideRows ? 128 : 64;
    const int ntile = (B + tile - 1) / tile;
    if ((int64_t)ntile * (ntile + 1) / 2 > 0x7fffffff || ntile > 65535) return hipErrorInvalidValue;
    const dim3 grid(ntile, ntile);
    if (tile == 128)
      hipLaunchKernelGGL(identity_kernel<8>, grid, dim3(kRwThreads), 0, st, msa, B, N, q, maxdiff, m, flag);
    else
      hipLaunchKernelGGL(identity_kernel<4>, grid, dim3(kRwThreads), 0, st, msa, B, N, q, maxdiff, m, flag);
  }
  hipLaunchKernelGGL(weights_kernel, dim3((B + 255) / 256), dim3(256), 0, st, m, B, uniform, w);
  hipLaunchKernelGGL(beff_kernel, dim3(1), dim3(kSumThreads), 0, st, w, B, beff);
  return hipGetLastError();
}

}  // namespace plm
