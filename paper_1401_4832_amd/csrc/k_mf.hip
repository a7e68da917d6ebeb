// k_mf.hip -- mean-field starting guess (sec. 2 and sec. 7): couplings from
// the inverse of the connected correlation matrix
//   c_ij(k,l) = f_ij(k,l) - f_i(k) f_j(l),   k, l < q - 1,
// built from reweighted frequencies mixed with a uniform pseudocount of
// weight lam (f_i = (1-lam) F_i/B_eff + lam/q, f_ij = (1-lam) F_ij/B_eff +
// lam/q^2 for i != j, f_ii(k,l) = f_i(k)[k = l]); J_ij(k,l) = -(C^-1)_(i,k),(j,l)
// with the last state (the gap) as reference, and the fields of the
// mean-field equations in that gauge,
//   h_i(k) = ln(f_i(k)/f_i(q-1)) - sum_{j != i} sum_{l < q-1} J_ij(k,l) f_j(l).
//
// Steps (all FP64, every sum in a fixed order):
//   sort    per column, a stable counting sort of the sequence indices by
//           state (one block per column)
//   single  f_i(k): the weights of one state's run summed in sorted order
//   pair    for one (i, k): the weights of the rows with state k at i,
//           histogrammed by the state of every column j; each thread owns
//           the bins of one column in LDS, so no two threads touch a bin;
//           writes row (i, k) of C up to the diagonal's unit
//   invert  in-place block sweep of the SPD matrix C (128 x 128 pivot blocks,
//           no pivoting: every pivot block is a Schur complement of an SPD
//           matrix), which keeps it symmetric, so that only the tiles on and
//           below the diagonal are formed: per pivot block, sweep it, multiply
//           its panel, rank-128 update of every other tile (FP64 matrix
//           products); ends with -C^-1
//   output  J in the asymmetric layout J[r][i][k][s] = J_ri(s, k) (both
//           estimates equal) and the fields
#include <math.h>

#include "plm_internal.h"

namespace plm {

constexpr int kMfThreads = 256;
constexpr int kGjTile = 64;              // tile size

// ---- sort ------------------------------------------------------------------
// order[i*B + t] = the t-th sequence (by index) among those sorted by state
// at column i; start[i*(q+1) + k] = first position of state k.  Symbols >= q
// raise bit 1 of *flag and are counted as state q - 1.
__global__ __launch_bounds__(kMfThreads) void mf_sort_kernel(const uint8_t* msa, int32_t B, int32_t N,
                                                             int32_t q, int32_t* order, int32_t* start,
                                                             int32_t* flag) {
  __shared__ int32_t cnt[kQMax][kMfThreads];
  __shared__ int32_t base[kQMax + 1];
  const int i = blockIdx.x, t = threadIdx.x;
  const int chunk = (B + kMfThreads - 1) / kMfThreads;
  const int b0 = min(B, t * chunk), b1 = min(B, b0 + chunk);
  for (int k = 0; k < q; ++k) cnt[k][t] = 0;
  bool bad = false;
  for (int b = b0; b < b1; ++b) {
    int s = msa[(size_t)b * N + i];
    if (s >= q) {
      bad = true;
      s = q - 1;
    }
    cnt[s][t] += 1;
  }
  if (bad && flag) atomicOr(flag, 1);
  __syncthreads();
  // exclusive prefix over (state, thread): state-major so that each state's
  // run is in sequence order
  if (t < q) {
    int acc = 0;
    for (int u = 0; u < kMfThreads; ++u) {
      const int c = cnt[t][u];
      cnt[t][u] = acc;
      acc += c;
    }
    base[t + 1] = acc;  // the run length of state t
  }
  __syncthreads();
  if (t == 0) {
    base[0] = 0;
    for (int k = 0; k < q; ++k) base[k + 1] += base[k];
    for (int k = 0; k <= q; ++k) start[(size_t)i * (q + 1) + k] = base[k];
  }
  __syncthreads();
  int pos[kQMax];
#pragma unroll
  for (int k = 0; k < kQMax; ++k) pos[k] = k < q ? base[k] + cnt[k][t] : 0;
  for (int b = b0; b < b1; ++b) {
    int s = msa[(size_t)b * N + i];
    if (s >= q) s = q - 1;
    int p = 0;
#pragma unroll
    for (int k = 0; k < kQMax; ++k)
      if (k == s) p = pos[k]++;
    order[(size_t)i * B + p] = b;
  }
}

// ---- single-site frequencies -------------------------------------------------
// One wave per (i, k): the weights of the state's run, lane by lane, then a
// shuffle tree (one thread per (i, k) waited for every load: 3.3 ms at
// N = 300, B = 30 000).
__global__ __launch_bounds__(kMfThreads) void mf_single_kernel(const int32_t* order, const int32_t* start,
                                                               const double* w, const double* beff, int32_t B,
                                                               int32_t N, int32_t q, double lam, double* fi) {
  const int e = blockIdx.x * (kMfThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (e >= N * q) return;
  const int i = e / q, k = e - i * q;
  const int32_t* o = order + (size_t)i * B;
  const int a = start[(size_t)i * (q + 1) + k], z = start[(size_t)i * (q + 1) + k + 1];
  double t = 0.0;
#pragma unroll 4
  for (int p = a + lane; p < z; p += 64) t += w[o[p]];
  for (int d = 32; d > 0; d >>= 1) t += __shfl_xor(t, d, 64);
  if (lane == 0) fi[e] = (1.0 - lam) * t / *beff + lam / q;
}

// ---- pair frequencies -> rows of C -------------------------------------------
// Block (i, k, jb): row (i, k) of C over the columns of sites jb*64 .. +63, one
// wave, one site per lane; rows of C are needed up to the end of their 64-index
// unit (the inversion reads tiles on and below the diagonal only), so the
// blocks past it have nothing to do.  C is n_pad x n_pad row-major, n = N (q - 1),
// entry ((i,k), (j,l)) at (i (q-1) + k) * ld + j (q-1) + l.  Bound: LDS, one
// FP64 read and write per (sequence, site pair); N = 300, B = 30 000: 2617 -> 1502 us
// (blocks of 256 sites, both triangles).
constexpr int kMfCols = 64;
__global__ __launch_bounds__(kMfCols) void mf_pair_kernel(const uint8_t* msa, const int32_t* order,
                                                          const int32_t* start, const double* w, const double* beff,
                                                          const double* fi, int32_t B, int32_t N, int32_t q,
                                                          double lam, double* C, int64_t ld) {
  __shared__ double bins[kQMax][kMfCols];
  __shared__ int32_t rows[kMfCols];
  __shared__ double wts[kMfCols];
  const int i = blockIdx.x, k = blockIdx.y, t = threadIdx.x;
  const int j0 = blockIdx.z * kMfCols, j = j0 + t;
  const int r = q - 1;
  if (j0 * r >= ((i * r + k) / kGjTile + 1) * kGjTile) return;
  for (int l = 0; l < q; ++l) bins[l][t] = 0.0;
  const int32_t* o = order + (size_t)i * B;
  const int a = start[(size_t)i * (q + 1) + k], z = start[(size_t)i * (q + 1) + k + 1];
  const int jc = min(j, N - 1);
  for (int c0 = a; c0 < z; c0 += kMfCols) {
    const int nc = min(kMfCols, z - c0);
    __syncthreads();
    if (t < nc) {
      const int b = o[c0 + t];
      rows[t] = b;
      wts[t] = w[b];
    }
    __syncthreads();
    int c = 0;
    for (; c + 16 <= nc; c += 16) {
      uint8_t s[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) s[u] = msa[(size_t)rows[c + u] * N + jc];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int su = s[u] < q ? s[u] : q - 1;
        bins[su][t] += wts[c + u];
      }
    }
    for (; c < nc; ++c) {
      const uint8_t s = msa[(size_t)rows[c] * N + jc];
      bins[s < q ? s : q - 1][t] += wts[c];
    }
  }
  __syncthreads();
  // row (i, k) of C over columns (j, l), j in [j0, j0 + 64), l < q - 1, written contiguously
  const double ib = 1.0 / *beff, fik = fi[(size_t)i * q + k];
  const int jn = min(kMfCols, N - j0);
  double* row = C + (size_t)(i * r + k) * ld + (size_t)j0 * r;
  for (int e = t; e < jn * r; e += kMfCols) {
    const int jl = e / r, l = e - jl * r, jj = j0 + jl;
    const double fjl = fi[(size_t)jj * q + l];
    double v;
    if (jj == i)
      v = (l == k ? fik : 0.0) - fik * fjl;
    else
      v = (1.0 - lam) * bins[l][jl] * ib + lam / ((double)q * q) - fik * fjl;
    row[e] = v;
  }
}

// identity on the padded rows and columns [n, n_pad)
__global__ void mf_pad_kernel(double* C, int64_t ld, int32_t n, int32_t n_pad) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t npad = n_pad - n;
  if (npad <= 0) return;
  // region 1: rows [n, n_pad) x all columns; region 2: rows [0, n) x columns [n, n_pad)
  const int64_t r1 = npad * n_pad, r2 = (int64_t)n * npad;
  if (e < r1) {
    const int64_t rr = n + e / n_pad, cc = e % n_pad;
    C[rr * ld + cc] = rr == cc ? 1.0 : 0.0;
  } else if (e < r1 + r2) {
    const int64_t f = e - r1, rr = f / npad, cc = n + f % npad;
    C[rr * ld + cc] = 0.0;
  }
}

// ---- block sweep ----------------------------------------------------------------
// Sweeping a set S of indices of a symmetric A: A_SS -> -P with P = A_SS^-1,
// A_iS -> W_i = A_iS P, A_ij -> A_ij - W_i A_jS^T (i, j outside S).  The matrix
// stays symmetric and ends, every index swept, as -A^-1.  Units of 64 indices;
// a pivot block is two units (the last one may be a single unit).  Tiles (I, J),
// I >= J, hold the matrix; the mirror tiles above the diagonal hold scratch: of
// a sweep, the panel before it, as [k][index] within each 64 x 64 tile.
typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int kPv = 2 * kGjTile;  // pivot block width

// 1 / a to the last bit or so: the hardware's reciprocal and two Newton steps
// (a division is a chain twice as long, and every step of a sweep waits for it)
__device__ inline double recip(double a) {
  double r = __builtin_amdgcn_rcp(a);
  r = fma(fma(-a, r, 1.0), r, r);
  return fma(fma(-a, r, 1.0), r, r);
}

// Sweep of 64 indices of the pivot block in LDS (M: the block's corner), by one
// block of four waves: a thread holds one row of sixteen columns.  Two
// indices k, k + 1 at a time: their columns, which are also their rows, go
// round through LDS, and with the 2 x 2 inverse p of their block every row
// subtracts f0 c0 + f1 c1.  Rows k and k + 1, which hold c0 and c1, come out as
// p c with f0, f1 changed by one; columns k and k + 1 come out as zero (of rows
// k, k + 1 as one) and get their values added, so that no register is written
// by a part of the lanes only.
constexpr int kPvPitch = kPv + 2;  // LDS row pitch of the pivot block: products read it without bank conflicts
__device__ inline void sweep_unit(double* M, double (*col)[2][kGjTile], bool& bad) {
  const int i = threadIdx.x & 63, g = threadIdx.x >> 6, j0 = 16 * g;
  double m[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) m[j] = M[i * kPvPitch + j0 + j];
#pragma unroll 1
  for (int gk = 0; gk < 4; ++gk) {
#pragma unroll
    for (int kk = 0; kk < 16; kk += 2) {
      const int k = 16 * gk + kk;
      double(*c)[kGjTile] = col[(kk >> 1) & 1];
      if (g == gk) {
        c[0][i] = m[kk];
        c[1][i] = m[kk + 1];
      }
      __syncthreads();
      const double a0 = c[0][k], a01 = c[0][k + 1], a1 = c[1][k + 1], r0 = c[0][i], r1 = c[1][i];
      double c0[16], c1[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        c0[j] = c[0][j0 + j];
        c1[j] = c[1][j0 + j];
      }
      __builtin_amdgcn_sched_barrier(0);  // every read is issued before the chain below
      const double i0 = recip(a0), x = a01 * i0, sc = fma(-a01, x, a1);
      if (!(a0 > 0.0) || !(sc > 0.0)) bad = true;
      const double p11 = recip(sc), p01 = -x * p11, p00 = fma(-x, p01, i0);
      const double f0 = fma(r0, p00, r1 * p01), f1 = fma(r0, p01, r1 * p11);
      const bool is0 = i == k, is1 = i == k + 1, here = g == gk;
      const double e0 = is0 ? 1.0 - p00 : is1 ? -p01 : f0;
      const double e1 = is0 ? -p01 : is1 ? 1.0 - p11 : f1;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        m[j] = fma(-e1, c1[j], fma(-e0, c0[j], m[j]));
        asm volatile("" : "+v"(m[j]));  // formed here: put off, the steps' operands would pile up in registers
      }
      m[kk] += !here ? 0.0 : is0 ? -1.0 - p00 : is1 ? -p01 : f0;
      m[kk + 1] += !here ? 0.0 : is0 ? -p01 : is1 ? -1.0 - p11 : f1;
    }
  }
#pragma unroll
  for (int j = 0; j < 16; ++j) M[i * kPvPitch + j0 + j] = m[j];
  __syncthreads();
}

// Sweep of a pivot block of one or two units (nu) from unit u0 on, in LDS: each
// unit in turn, the other unit's panel and tile by matrix products.  A pivot
// that is not positive raises bit 8 of *flag (A is not positive definite).
// Bound: the chain of 32 steps per unit (barrier, LDS, two reciprocals); 44 us for
// two units.  All 128 indices in registers took 80 us (four rows a thread) and
// 104 us (one row a thread, one index a step): LDS reads and spills.
__device__ __forceinline__ void pivot_block(double* A, int64_t ld, int32_t u0, int32_t nu, int32_t* flag, double* M,
                                   double (&col)[2][2][kGjTile]) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, l16 = lane & 15, lk = lane >> 4;
  const size_t o = (size_t)u0 * kGjTile;
  const int w = nu * kGjTile;
  // (the tile above the diagonal holds scratch: its values come from below)
  for (int i0 = 0; i0 < w; i0 += kGjTile)
    for (int j0 = 0; j0 <= i0; j0 += kGjTile) {
      double v[kGjTile * kGjTile / kMfThreads];
#pragma unroll
      for (int k = 0; k < kGjTile * kGjTile / kMfThreads; ++k)
        v[k] = A[(o + i0 + wid + 4 * k) * ld + o + j0 + lane];
#pragma unroll
      for (int k = 0; k < kGjTile * kGjTile / kMfThreads; ++k) {
        const int i = i0 + wid + 4 * k, j = j0 + lane;
        M[i * kPvPitch + j] = v[k];
        if (j0 < i0) M[j * kPvPitch + i] = v[k];
      }
    }
  __syncthreads();
  bool bad = false;
  for (int u = 0; u < nu; ++u) {
    const int b = u * kGjTile, r = (1 - u) * kGjTile;  // swept unit, other unit
    sweep_unit(M + b * kPvPitch + b, col, bad);
    if (nu == 1) break;
    // W = X P = -X M_bb (X = M_rb), put at M_br transposed; wave wid: rows 16 wid ..
    d4 acc[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) acc[n] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int k = 0; k < kGjTile; k += 4) {
      const double av = M[(r + 16 * wid + l16) * kPvPitch + b + k + lk];
#pragma unroll
      for (int n = 0; n < 4; ++n)
        acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, M[(b + k + lk) * kPvPitch + b + 16 * n + l16], acc[n], 0, 0, 0);
    }
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int q = 0; q < 4; ++q) M[(b + 16 * n + l16) * kPvPitch + r + 16 * wid + 4 * q + lk] = -acc[n][q];
    __syncthreads();
    // M_rr -= W X^T
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[n][q] = M[(r + 16 * wid + 4 * q + lk) * kPvPitch + r + 16 * n + l16];
#pragma unroll 4
    for (int k = 0; k < kGjTile; k += 4) {
      const double av = -M[(b + k + lk) * kPvPitch + r + 16 * wid + l16];
#pragma unroll
      for (int n = 0; n < 4; ++n)
        acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, M[(r + 16 * n + l16) * kPvPitch + b + k + lk], acc[n], 0, 0, 0);
    }
    __syncthreads();  // every wave has read X
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int q = 0; q < 4; ++q) M[(r + 16 * wid + 4 * q + lk) * kPvPitch + r + 16 * n + l16] = acc[n][q];
#pragma unroll
    for (int k = 0; k < kGjTile * kGjTile / kMfThreads; ++k)
      M[(r + wid + 4 * k) * kPvPitch + b + lane] = M[(b + lane) * kPvPitch + r + wid + 4 * k];
    __syncthreads();
  }
  if (bad && tid == 0 && flag) atomicOr(flag, 8);
  for (int i0 = 0; i0 < w; i0 += kGjTile)
    for (int j0 = 0; j0 < w; j0 += kGjTile)
#pragma unroll
      for (int k = 0; k < kGjTile * kGjTile / kMfThreads; ++k) {
        const int i = i0 + wid + 4 * k, j = j0 + lane;
        A[(o + i) * ld + o + j] = M[i * kPvPitch + j];
      }
}

// LDS pitch (doubles) of a staged [k][128] panel: rows k and k + 1 start 32 banks apart
constexpr int kGjPitch = 2 * kGjTile + 16;
constexpr int kGjK = 16;  // panel indices per staged chunk

// Sixteen panel values of a 64-index unit per lane, from a tile stored
// [index][k] (kmajor = false: lane = index) or [k][index] (two k at a time, 32
// lanes across the indices), and their way into a staged [k][index] panel; both
// keep the lanes of a write on consecutive banks.
__device__ inline void load_panel(const double* t, int64_t ld, int k0, bool kmajor, int lane, double (&v)[16]) {
  const double* p = kmajor ? t + (size_t)(k0 + (lane >> 5)) * ld + (lane & 31) * 2 : t + (size_t)lane * ld + k0;
  const int64_t st = kmajor ? 2 * ld : 2;
#pragma unroll
  for (int e = 0; e < 16; e += 2) {
    const double2 x = *reinterpret_cast<const double2*>(p + (e >> 1) * st);
    v[e] = x.x;
    v[e + 1] = x.y;
  }
}
__device__ inline void store_panel(double* L, bool kmajor, int lane, double sign, const double (&v)[16]) {
  if (kmajor) {
    double* p = L + (lane >> 5) * kGjPitch + (lane & 31) * 2;
#pragma unroll
    for (int e = 0; e < 16; e += 2)
      *reinterpret_cast<double2*>(p + e * kGjPitch) = make_double2(sign * v[e], sign * v[e + 1]);
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) L[lane + e * kGjPitch] = sign * v[e];
  }
}

// Panel of half a unit (outside the pivot block): X = A_iS is copied to the
// scratch tiles as [k][index], and W = X P = -X (-P) takes its place in the
// matrix.  One block per 32 rows; each wave forms 32 rows x w / 4 columns, its
// part of P in registers from the start.  Bound: latency (a few microseconds of
// loads, products and stores in turn).
constexpr int kPnRows = kGjTile / 2;
__global__ __launch_bounds__(kMfThreads, 2) void gj_panel_kernel(double* A, int64_t ld, int32_t u0, int32_t nu) {
  constexpr int kXp = kPnRows + 16;
  __shared__ __attribute__((aligned(16))) double X[kPv * kXp];
  const int unit = blockIdx.x >> 1, hf = blockIdx.x & 1;
  const int i = unit < u0 ? unit : unit + nu;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, l16 = lane & 15, lk = lane >> 4;
  const int w = nu * kGjTile;
  const size_t oi = (size_t)i * kGjTile, op = (size_t)u0 * kGjTile;
  const int x0 = hf * kPnRows;    // this block's rows of the unit
  const bool below = i > u0;  // the panel is a tile row (matrix tiles (i, S)) or tile column ((S, i))
  // -P, symmetric: this lane's operands of every product (columns wid * w/4 ..: two tiles of 16, or one)
  const int nc = w / 64;
  const double* P = A + op * ld + op + wid * (w / 4) + l16;
  double bv[kPv / 4][2];
#pragma unroll
  for (int k = 0; k < kPv / 4; ++k)
#pragma unroll
    for (int c = 0; c < 2; ++c) bv[k][c] = P[(size_t)(k < w / 4 ? 4 * k + lk : 0) * ld + (c < nc ? 16 * c : 0)];
  // X to LDS as [k][index] and to the scratch tiles
  constexpr int kPer = kPv * kPnRows / kMfThreads;
  double xv[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int id = min(tid + e * kMfThreads, w * kPnRows - 1);
    // below: consecutive threads along k (the tile's rows), else along the index
    const int k = below ? id % w : id / kPnRows, x = below ? id / w : id % kPnRows;
    xv[e] = below ? A[(oi + x0 + x) * ld + op + k] : A[(op + k) * ld + oi + x0 + x];
  }
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int id = min(tid + e * kMfThreads, w * kPnRows - 1);
    const int k = below ? id % w : id / kPnRows, x = below ? id / w : id % kPnRows;
    X[k * kXp + x] = xv[e];
  }
  __syncthreads();
  for (int e = tid; e < w * kPnRows; e += kMfThreads) {
    const int k = e / kPnRows, x = e % kPnRows;
    const size_t at = below ? (op + k) * ld + oi + x0 + x
                            : (oi + k % kGjTile) * ld + op + (k / kGjTile) * kGjTile + x0 + x;
    A[at] = X[k * kXp + x];
  }
  d4 acc[2][2];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[m][c] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < kPv / 4; ++k) {
    if (k < w / 4)
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const double av = X[(4 * k + lk) * kXp + 16 * m + l16];
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[m][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[k][c], acc[m][c], 0, 0, 0);
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if (c >= nc) continue;
    const int k = wid * (w / 4) + 16 * c + l16;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int x = x0 + 16 * m + 4 * r + lk;  // row of the result (D: row 4 r + lane / 16, column lane % 16)
        if (below) A[(oi + x) * ld + op + k] = -acc[m][c][r];
        else A[(op + k) * ld + oi + x] = -acc[m][c][r];
      }
  }
}

// Update of the tiles outside pivot block ps: A_ij -= W_i X_j^T, tile t a 2 x 2 of
// units (a, b), a >= b, one unit per wave (64 x 64 in registers, sixteen
// FP64 products per four panel indices); chunks of kGjK panel indices are
// double-buffered in LDS, each wave staging one of the block's four panel units.
using UpdateLds = double[2][2][kGjK * kGjPitch];
__device__ __forceinline__ void update_tile(double* A, int64_t ld, int32_t nt, int32_t ps, int32_t u0, int32_t nu, int32_t t,
                                   UpdateLds& L) {
  int a = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
  while (a * (a + 1) / 2 > t) --a;
  while ((a + 1) * (a + 2) / 2 <= t) ++a;
  int b = t - a * (a + 1) / 2;
  a += a >= ps;
  b += b >= ps;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lk = lane >> 4;
  const int I = 2 * a + (wid >> 1), J = 2 * b + (wid & 1);
  const bool live = I < nt && J <= I;
  // the panel unit this wave stages: W of 2a, 2a + 1, X of 2b, 2b + 1
  const int su = (wid < 2 ? 2 * a : 2 * b) + (wid & 1);
  const bool sok = su < nt;
  const bool after = su > u0;  // below or right of the pivot block
  // W sits in the matrix: [index][k] in tiles (su, S), or [k][index] in tiles (S, su);
  // X in the scratch tiles, [k][index] always
  const bool km = wid >= 2 || !after;
  double v0[16], v1[16];  // chunks in flight: even and odd ones
  auto load = [&](int c, double (&v)[16]) {
    const int s = u0 + c / (kGjTile / kGjK), k0 = (c % (kGjTile / kGjK)) * kGjK;
    const int row = wid < 2 ? (after ? su : s) : (after ? s : su), cl = wid < 2 ? (after ? s : su) : (after ? su : s);
    if (sok) load_panel(A + (size_t)row * kGjTile * ld + (size_t)cl * kGjTile, ld, k0, km, lane, v);
  };
  auto store = [&](int buf, const double (&v)[16]) {
    double* dst = L[buf][wid >> 1] + (wid & 1) * kGjTile;
    if (sok) store_panel(dst, km, lane, wid < 2 ? -1.0 : 1.0, v);
  };
  const int nch = nu * (kGjTile / kGjK);  // at least four, and even
  load(0, v0);
  load(1, v1);
  d4 acc[4][4];
  double* C = A + (size_t)I * kGjTile * ld + (size_t)J * kGjTile + (size_t)lk * ld + l16;
  if (live) {
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[m][n][r] = C[(size_t)(16 * m + 4 * r) * ld + 16 * n];
  }
  store(0, v0);
  // the tile has arrived here: no wait for it inside the loop, where it would
  // cover the panel loads in flight too
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) asm volatile("" : "+v"(acc[m][n]));
  __syncthreads();
  auto products = [&](int buf) {
    if (!live) return;
    const double* W = L[buf][0] + (wid >> 1) * kGjTile + lk * kGjPitch + l16;
    const double* X = L[buf][1] + (wid & 1) * kGjTile + lk * kGjPitch + l16;
#pragma unroll
    for (int k = 0; k < kGjK; k += 4) {
      double av[4], bv[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        av[m] = W[k * kGjPitch + 16 * m];
        bv[m] = X[k * kGjPitch + 16 * m];
      }
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n)
          acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[m], bv[n], acc[m][n], 0, 0, 0);
    }
  };
  // two chunks in flight: the panel loads take longer than one chunk's products
  for (int c = 0; c < nch; c += 2) {
    if (c + 2 < nch) load(c + 2, v0);
    products(0);
    store(1, v1);
    __syncthreads();
    if (c + 3 < nch) load(c + 3, v1);
    products(1);
    if (c + 2 < nch) store(0, v0);
    __syncthreads();
  }
  if (live)
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) C[(size_t)(16 * m + 4 * r) * ld + 16 * n] = acc[m][n][r];
}

// Whole rounds of the update's tiles over the chip, dealt to the XCDs in runs, so
// that a run's panels stay in one L2.  The tile that holds the next pivot block
// (index tp) is one of them: it takes the place of the last.
// Bound: the FP64 matrix cores (43 TFLOP/s of the 69 they reach alone); n = 6000:
// 50 us a round of 512 blocks, where 64-index updates of both triangles in vector
// FP64 took 328 us each.
__global__ __launch_bounds__(kMfThreads, 2) void gj_update_kernel(double* A, int64_t ld, int32_t nt, int32_t ps,
                                                                  int32_t u0, int32_t nu, int32_t ntile, int32_t tp) {
  __shared__ __attribute__((aligned(16))) UpdateLds L;
  const int per = (ntile + kQueues - 1) / kQueues;
  int t = (blockIdx.x % kQueues) * per + blockIdx.x / kQueues;
  if (t >= ntile) return;
  if (t == ntile - 1 && tp >= ntile) t = tp;
  update_tile(A, ld, nt, ps, u0, nu, t, L);
}

// The rest of the tiles, from first on, beside the sweep of the next pivot block
// (block 0), which took 44 us alone after an update whose last round left most of
// the chip idle: n = 6000, 117 + 44 -> 100 + 45 us (with 255 or 510 of
// its 1081 tiles here instead of what whole rounds leave, 96 + 48 and 73 + 73 us).  With no whole round (first = 0)
// block 0 updates its own tile (index tp) before the sweep.
// Bound: the sweep's chain, or with few blocks a tile's.
__global__ __launch_bounds__(kMfThreads) void gj_sweep_kernel(double* A, int64_t ld, int32_t nt, int32_t ps, int32_t u0,
                                                              int32_t nu, int32_t first, int32_t tp, int32_t un,
                                                              int32_t nun, int32_t* flag) {
  __shared__ __attribute__((aligned(16))) double M[kPv * kPvPitch];
  __shared__ __attribute__((aligned(16))) double col[2][2][kGjTile];
  static_assert(sizeof(UpdateLds) <= sizeof(M), "a tile's panels take the pivot block's place");
  UpdateLds& L = *reinterpret_cast<UpdateLds*>(M);
  if (blockIdx.x > 0) {
    int t = first + (int)blockIdx.x - 1;
    if (first == 0) t += t >= tp;                       // tp is block 0's
    else if (t == tp) t = first - 1;                    // tp took the place of this one
    update_tile(A, ld, nt, ps, u0, nu, t, L);
    return;
  }
  if (first == 0 && tp >= 0) {
    update_tile(A, ld, nt, ps, u0, nu, tp, L);
    __syncthreads();  // the tile is written, its panels are done with
  }
  pivot_block(A, ld, un, nun, flag, M, col);
}

// ---- output ------------------------------------------------------------------
// S = -C^-1 (tiles on and below the diagonal).  J[a][i][k][s] = S[(a,s),(i,k)]
// and J[i][a][k][s] = S[(a,k),(i,s)] for s, k < q - 1 from the one stored block
// of a pair a > i (q - 1 values per row); 0 for the reference state and a = i.
__global__ __launch_bounds__(kMfThreads) void mf_couplings_kernel(const double* S, int64_t ld, int32_t N, int32_t q,
                                                                  float* J) {
  __shared__ float T[kQMax * kQMax];
  const int a = blockIdx.y, i = blockIdx.x, r = q - 1, qq = q * q;
  if (i > a) return;
  float* out = J + ((size_t)a * N + i) * qq;
  if (a == i) {
    for (int e = threadIdx.x; e < qq; e += blockDim.x) out[e] = 0.f;
    return;
  }
  // T[k][s]: state s of a, k of i
  for (int e = threadIdx.x; e < r * r; e += blockDim.x) {
    const int s = e / r, k = e - s * r;
    T[k * q + s] = (float)S[(size_t)(a * r + s) * ld + i * r + k];
  }
  __syncthreads();
  float* out2 = J + ((size_t)i * N + a) * qq;
  for (int e = threadIdx.x; e < qq; e += blockDim.x) {
    const int k = e / q, s = e - k * q;
    const bool in = k < r && s < r;
    out[e] = in ? T[k * q + s] : 0.f;
    out2[e] = in ? T[s * q + k] : 0.f;
  }
}

// h_a(s) = ln(f_a(s)/f_a(q-1)) - sum_{i != a} sum_{k < q-1} S[(a,s),(i,k)] f_i(k);
// a zero reference frequency (possible only without pseudocounts) raises bit 8.
// Sites before a: row (a, s) of S, one wave per state; sites after a: the q - 1
// columns (a, .) of their rows, 16 rows at a time.
constexpr int kMfRows = kMfThreads / 16;
__global__ __launch_bounds__(kMfThreads) void mf_fields_kernel(const double* S, int64_t ld, const double* fi, int32_t N,
                                                               int32_t q, float* h, int32_t* flag) {
  __shared__ double row[kQMax], col[kMfThreads];
  const int a = blockIdx.x, r = q - 1, tid = threadIdx.x, lane = tid & 63;
  if (tid == 0 && !(fi[(size_t)a * q + r] > 0.0) && flag) atomicOr(flag, 8);
  for (int s = tid >> 6; s < r; s += kMfThreads / 64) {
    const double* p = S + (size_t)(a * r + s) * ld;
    double t = 0.0;
#pragma unroll 4
    for (int e = lane; e < a * r; e += 64) t += p[e] * fi[(size_t)(e / r) * q + e % r];
    for (int d = 32; d > 0; d >>= 1) t += __shfl_xor(t, d, 64);
    if (lane == 0) row[s] = t;
  }
  // states sixteen at a time: thread (g, u) takes state s0 + u of rows g, g + 16, ...
  const int g = tid >> 4, u = tid & 15;
  for (int s0 = 0; s0 < r; s0 += 16) {
    const int s = s0 + u;
    double t = 0.0;
    if (s < r)
#pragma unroll 4
      for (int e = (a + 1) * r + g; e < N * r; e += kMfRows)
        t += S[(size_t)e * ld + a * r + s] * fi[(size_t)(e / r) * q + e % r];
    __syncthreads();
    col[tid] = t;
    __syncthreads();
    if (tid < 16 && s < r) {
      double sum = row[s];
      for (int k = 0; k < kMfRows; ++k) sum += col[k * 16 + tid];
      h[(size_t)a * q + s] = (float)(log(fi[(size_t)a * q + s] / fi[(size_t)a * q + r]) - sum);
    }
  }
  if (tid == 0) h[(size_t)a * q + r] = 0.f;
}

// ---- host side -------------------------------------------------------------------
int32_t mf_tile() { return kGjTile; }

hipError_t launch_mf_frequencies(const uint8_t* msa, int32_t B, int32_t N, int32_t q, const double* w,
                                 const double* beff, double lam, int32_t* order, int32_t* start, double* fi,
                                 int32_t* flag, hipStream_t st) {
  hipLaunchKernelGGL(mf_sort_kernel, dim3(N), dim3(kMfThreads), 0, st, msa, B, N, q, order, start, flag);
  hipLaunchKernelGGL(mf_single_kernel, dim3((N * q + 3) / 4), dim3(kMfThreads), 0, st, order, start, w, beff, B,
                     N, q, lam, fi);
  return hipGetLastError();
}

hipError_t launch_mf_correlation(const uint8_t* msa, const int32_t* order, const int32_t* start, const double* w,
                                 const double* beff, const double* fi, int32_t B, int32_t N, int32_t q,
                                 double lam, double* C, int32_t n_pad, hipStream_t st) {
  const int r = q - 1, n = N * r;
  hipLaunchKernelGGL(mf_pair_kernel, dim3(N, r, (N + kMfCols - 1) / kMfCols), dim3(kMfCols), 0, st,
                     msa, order, start, w, beff, fi, B, N, q, lam, C, (int64_t)n_pad);
  const int64_t npad = n_pad - n;
  if (npad > 0) {
    const int64_t tot = npad * n_pad + (int64_t)n * npad;
    hipLaunchKernelGGL(mf_pad_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, C, (int64_t)n_pad,
                       n, n_pad);
  }
  return hipGetLastError();
}

hipError_t launch_mf_invert(double* C, int32_t n_pad, int32_t ncu, int32_t* flag, hipStream_t st) {
  const int nt = n_pad / kGjTile, ns = (nt + 1) / 2;  // units, pivot blocks
  const int64_t ld = n_pad;
  const int nblk = (ns - 1) * ns / 2;  // pairs a >= b of the blocks besides the pivot
  auto units = [&](int p) { return nt - 2 * p < 2 ? nt - 2 * p : 2; };
  hipLaunchKernelGGL(gj_sweep_kernel, dim3(1), dim3(kMfThreads), 0, st, C, ld, nt, 0, 0, 0, 0, -1, 0, units(0), flag);
  for (int p = 0; p < ns && ns > 1; ++p) {
    const int u0 = 2 * p, nu = units(p);
    hipLaunchKernelGGL(gj_panel_kernel, dim3(2 * (nt - nu)), dim3(kMfThreads), 0, st, C, ld, u0, nu);
    // the next pivot block is pair (p, p) of the others; the last update is followed by no sweep
    const bool last = p + 1 == ns;
    const int tp = last ? -1 : p * (p + 1) / 2 + p;
    const int whole = last ? nblk : nblk / (2 * ncu) * (2 * ncu);  // rounds of two blocks per compute unit
    if (whole > 0)
      hipLaunchKernelGGL(gj_update_kernel, dim3((whole + kQueues - 1) / kQueues * kQueues), dim3(kMfThreads), 0, st, C,
                         ld, nt, p, u0, nu, whole, tp);
    if (!last)
      hipLaunchKernelGGL(gj_sweep_kernel, dim3(1 + nblk - (whole > 0 ? whole : 1)), dim3(kMfThreads), 0, st, C, ld, nt,
                         p, u0, nu, whole, tp, u0 + 2, units(p + 1), flag);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

hipError_t launch_mf_output(const double* Cinv, int32_t n_pad, const double* fi, int32_t N, int32_t q, float* h,
                            float* J, int32_t* flag, hipStream_t st) {
  hipLaunchKernelGGL(mf_couplings_kernel, dim3(N, N), dim3(kMfThreads), 0, st, Cinv, (int64_t)n_pad, N, q, J);
  hipLaunchKernelGGL(mf_fields_kernel, dim3(N), dim3(kMfThreads), 0, st, Cinv, (int64_t)n_pad, fi, N, q, h, flag);
  return hipGetLastError();
}

}  // namespace plm
