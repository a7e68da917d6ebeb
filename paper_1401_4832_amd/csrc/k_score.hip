// k_score.hip -- coupling scores of asymmetric plmDCA (sec. 3.4 steps 4-6).
//
// For every pair (i, j), i < j: both estimates of the pair as q x q
// matrices indexed (state of i, state of j) -- the site-i estimate is
// J[i][j][k][s] read with s the state of i, the site-j estimate J[j][i][k][s]
// with s the state of j, i.e. transposed -- each moved to the Ising gauge by
// subtracting row and column means and adding the grand mean
// (eq. gauge_change2), averaged (eq. average2) and reduced to the Frobenius
// norm (eq. frob_normtrans2).  A second pass applies the average product
// correction (eq. corr_norm2) with means over all N positions.  FP64.  The
// same kernels compute the variants the paper also tried (sec. 7): min/max
// combinations, l_p norms, the Burkoff divergence (eqs. burkoffscore1,
// burkoffscore2), the gap state left out, and the average-sum correction
// (eq. corr_normsum).
#include "plm_internal.h"

namespace plm {

// Each wave scores a run of `per` consecutive pairs (i < j, ordered by i, then
// j): both estimates to the Ising gauge, combined (average, elementwise min or
// max), reduced by the chosen norm over all states or over the non-gap states
// 0..q-2: Frobenius, l_p (sum of |J|^p to
// the power 1/p), or the Burkoff divergence sum P ln(P / (f_i f_j)) with P
// proportional to f_i(k) f_j(l) exp(J(k,l)) (computed with the largest
// exponent factored out).
// Lane 21 h + a holds the elements (state a of i, states h nc + k of j),
// k < nc = ceil(q / 3), in registers: the site-i block is read straight into them (q
// contiguous floats at a time), the site-j block through LDS (transposed);
// the sums over j's states are nc adds and a sum over three lanes, those
// over i's states the same on the matrix written to LDS and read with the
// states exchanged.  Every wave uses its own LDS, so nothing waits for the
// block; the next pair's loads are in flight while the current one is scored.  AVG: the gauge shift is linear, so the average is shifted once; the
// other combinations shift both estimates.
// Bound: HBM, the couplings read once (441 MB at N = 500, 92 us at the copy
// rate); measured there 277 -> 124 us (one wave per block, transposed
// global reads, every sum q serial LDS reads before).
constexpr int kScWaves = 4;
constexpr int kScPer = 7;           // states of j per lane at most
constexpr int kScPitch = kQMax + 2;  // row pitch of the FP64 matrix in LDS (odd)
static_assert(3 * kScPer == kQMax, "three lanes cover the states of j");

template <bool AVG, int NORM>
__global__ __launch_bounds__(64 * kScWaves) void pair_score_kernel(const float* __restrict__ J, int32_t N, int32_t q,
                                                                   int32_t npairs, int32_t per, ScoreOpts o,
                                                                   const double* __restrict__ freq,
                                                                   double* __restrict__ raw) {
  constexpr int NM = AVG ? 1 : 2;  // matrices moved to the Ising gauge
  __shared__ float T[kScWaves][kQMax * kQMax];
  __shared__ double M[kScWaves][kQMax * kScPitch];
  __shared__ double mean[kScWaves][kQMax];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < N; k += gridDim.x * blockDim.x) raw[(size_t)k * N + k] = 0.0;
  const int64_t lo = (int64_t)(blockIdx.x * kScWaves + wid) * per;
  if (lo >= npairs) return;
  const int p0 = (int)lo, p1 = (int)min((int64_t)npairs, lo + per);
  // row i of pair p0: the last i whose first pair i (2 N - 1 - i) / 2 is <= p0
  int i, j;
  {
    const double b = 2.0 * N - 1.0;
    i = (int)(0.5 * (b - sqrt(b * b - 8.0 * (double)p0)));
    auto first = [&](int r) { return (int)((int64_t)r * (2 * (int64_t)N - 1 - r) / 2); };
    while (first(i) > p0) --i;
    while (first(i + 1) <= p0) ++i;
    j = i + 1 + (p0 - first(i));
    i = __builtin_amdgcn_readfirstlane(i);
    j = __builtin_amdgcn_readfirstlane(j);
  }
  const int qq = q * q, qs = o.exclude_gap ? q - 1 : q;  // states summed over
  const int nc = (q + 2) / 3;  // states of j per lane
  const int h = lane / kQMax, a = lane - h * kQMax, c0 = nc * h, cn = min(nc, q - c0);
  const bool act = h < 3 && a < q;
  // the other two lanes of this state
  const int l1 = h < 3 ? (h + 1) % 3 * kQMax + a : lane, l2 = h < 3 ? (h + 2) % 3 * kQMax + a : lane;
  auto sum3 = [&](double v) { return v + (__shfl(v, l1, 64) + __shfl(v, l2, 64)); };
  const double dq = (double)q;
  float xi[kScPer], t[kScPer];
  auto load = [&](int ii, int jj) {
    const float* Jij = J + ((size_t)ii * N + jj) * qq;
    const float* Jji = J + ((size_t)jj * N + ii) * qq;
#pragma unroll
    for (int k = 0; k < kScPer; ++k) {
      xi[k] = act && k < cn ? Jij[(c0 + k) * q + a] : 0.f;
      t[k] = lane + 64 * k < qq ? Jji[lane + 64 * k] : 0.f;
    }
  };
  load(i, j);
  for (int p = p0; p < p1; ++p) {
    const int ci = i, cj = j;
    float xc[kScPer];
    wave_sync();
#pragma unroll
    for (int k = 0; k < kScPer; ++k) {
      xc[k] = xi[k];
      if (lane + 64 * k < qq) T[wid][lane + 64 * k] = t[k];
    }
    if (++j == N) {
      ++i;
      j = i + 1;
    }
    if (p + 1 < p1) load(i, j);
    wave_sync();
    double x[NM][kScPer];
#pragma unroll
    for (int k = 0; k < kScPer; ++k) {
      const double y = act && k < cn ? (double)T[wid][a * q + c0 + k] : 0.0;
      x[0][k] = AVG ? 0.5 * ((double)xc[k] + y) : (double)xc[k];
      if (!AVG) x[NM - 1][k] = y;
    }
#pragma unroll
    for (int z = 0; z < NM; ++z) {
      double r = 0.0, s = 0.0, g = 0.0, cm[kScPer];
      if (z) wave_sync();
#pragma unroll
      for (int k = 0; k < kScPer; ++k) {
        r += x[z][k];
        if (act && k < cn) M[wid][(c0 + k) * kScPitch + a] = x[z][k];
      }
      r = sum3(r) / dq;
      wave_sync();
      // here a is the state of j, c0 + k the states of i
#pragma unroll
      for (int k = 0; k < kScPer; ++k)
        if (act && k < cn) s += M[wid][a * kScPitch + c0 + k];
      s = sum3(s) / dq;
      if (act && h == 0) mean[wid][a] = s;
      wave_sync();
#pragma unroll
      for (int k = 0; k < kScPer; ++k) {
        cm[k] = k < cn && h < 3 ? mean[wid][c0 + k] : 0.0;
        g += cm[k];
      }
      g = sum3(g) / dq;
#pragma unroll
      for (int k = 0; k < kScPer; ++k) x[z][k] = x[z][k] - cm[k] - r + g;
    }
    double v[kScPer];
    bool in[kScPer];
#pragma unroll
    for (int k = 0; k < kScPer; ++k) {
      v[k] = AVG ? x[0][k]
                 : o.combine == PLM_COMBINE_MIN ? fmin(x[0][k], x[NM - 1][k]) : fmax(x[0][k], x[NM - 1][k]);
      in[k] = act && a < qs && k < cn && c0 + k < qs;
    }
    double out = 0.0;
    if constexpr (NORM == PLM_NORM_BURKOFF) {
      double mx = -INFINITY;
#pragma unroll
      for (int k = 0; k < kScPer; ++k)
        if (in[k]) mx = fmax(mx, v[k]);
      for (int d = 32; d > 0; d >>= 1) mx = fmax(mx, __shfl_xor(mx, d, 64));
      double z = 0.0, zv = 0.0;
      const double fi = act ? freq[(size_t)ci * q + a] : 0.0;
#pragma unroll
      for (int k = 0; k < kScPer; ++k)
        if (in[k]) {
          const double w = fi * freq[(size_t)cj * q + c0 + k] * exp(v[k] - mx);
          z += w;
          zv += w * v[k];
        }
      for (int d = 32; d > 0; d >>= 1) {
        z += __shfl_xor(z, d, 64);
        zv += __shfl_xor(zv, d, 64);
      }
      out = z > 0.0 ? zv / z - mx - log(z) : 0.0;
    } else {
      constexpr bool lp = NORM == PLM_NORM_LP;
      double ss = 0.0;
#pragma unroll
      for (int k = 0; k < kScPer; ++k)
        if (in[k]) ss += lp ? pow(fabs(v[k]), o.p) : v[k] * v[k];
      for (int d = 32; d > 0; d >>= 1) ss += __shfl_xor(ss, d, 64);
      out = lp ? pow(ss, 1.0 / o.p) : sqrt(ss);
    }
    if (lane == 0) {
      raw[(size_t)ci * N + cj] = out;
      raw[(size_t)cj * N + ci] = out;
    }
  }
}

// row sums of the raw scores, one wave per row, parked on the diagonal of the
// output until the correction has read them
__global__ __launch_bounds__(64) void rowsum_kernel(const double* __restrict__ fn, int32_t N,
                                                    double* __restrict__ cfn) {
  const int i = blockIdx.x;
  const double* row = fn + (size_t)i * N;
  double s = 0.0;
#pragma unroll 4
  for (int j = threadIdx.x; j < N; j += 64) s += row[j];
  for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
  if (threadIdx.x == 0) cfn[(size_t)i * N + i] = s;
}

// Correction of the symmetric raw scores with means over all N positions:
// average product (eq. corr_norm2), average sum (eq. corr_normsum) or none.
// kCorRows rows per block; every block adds the row sums parked on the
// diagonal in the same order, and leaves the diagonal alone (other blocks
// still read it: diag_zero_kernel clears it).  Measured at N = 500: 333 -> 8 us
// (one block for all pairs before), the row sums 105 -> 5 us (one thread a row).
constexpr int kCorRows = 4;
__global__ __launch_bounds__(256) void correct_kernel(const double* __restrict__ fn, int32_t N, int32_t mode,
                                                      double* __restrict__ cfn) {
  __shared__ double red[4];
  double t = 0.0;
  for (int k = threadIdx.x; k < N; k += blockDim.x) t += cfn[(size_t)k * N + k];
  const double all = block_sum_f64(t, red) / ((double)N * (double)N);
  const int i0 = blockIdx.x * kCorRows, i1 = min(N, i0 + kCorRows);
  for (int j = threadIdx.x; j < N; j += blockDim.x) {
    const double rj = cfn[(size_t)j * N + j] / (double)N;
    for (int i = i0; i < i1; ++i) {
      if (i == j) continue;
      const size_t e = (size_t)i * N + j;
      const double ri = cfn[(size_t)i * N + i] / (double)N;
      cfn[e] = mode == PLM_CORR_NONE ? fn[e]
               : mode == PLM_CORR_ASC ? fn[e] - ri - rj + all
               : all == 0.0           ? 0.0
                                      : fn[e] - ri * rj / all;
    }
  }
}

__global__ void diag_zero_kernel(double* cfn, int32_t N) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < N) cfn[(size_t)i * N + i] = 0.0;
}

// Row sums and correction in one block, the same sums in the same order: for few
// positions, where the launches above take longer than the work (plm_score whole,
// with them and so: N = 2 12.3 / 6.9 us, N = 32 13.2 / 9.3, N = 64 13.5 / 12.9, N = 80
// 15.0 / 17.5; two launches where one for both, one thread a row, took 9.6 and 15.5 us).
constexpr int kCorSmall = 64;
__global__ __launch_bounds__(1024) void correct_small_kernel(const double* __restrict__ fn, int32_t N, int32_t mode,
                                                             double* __restrict__ cfn) {
  __shared__ double rs[kCorSmall], red[16];
  const int tid = threadIdx.x, lane = tid & 63;
  for (int i = tid >> 6; i < N; i += 16) {
    double s = 0.0;
    for (int j = lane; j < N; j += 64) s += fn[(size_t)i * N + j];
    for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
    if (lane == 0) rs[i] = s;
  }
  __syncthreads();
  const double all = block_sum_f64(tid < N ? rs[tid] : 0.0, red) / ((double)N * (double)N);
  for (int e = tid; e < N * N; e += blockDim.x) {
    const int i = e / N, j = e - i * N;
    const double ri = rs[i] / (double)N, rj = rs[j] / (double)N;
    cfn[e] = i == j                   ? 0.0
             : mode == PLM_CORR_NONE ? fn[e]
             : mode == PLM_CORR_ASC  ? fn[e] - ri - rj + all
             : all == 0.0            ? 0.0
                                     : fn[e] - ri * rj / all;
  }
}

constexpr int kScResident = 256 * 6 * kScWaves;  // waves: six blocks (LDS) on each CU

hipError_t launch_score_ex(const float* J, int32_t N, int32_t q, const ScoreOpts& o,
                           const double* freq, double* raw, double* cor, hipStream_t st) {
  // runs of pairs for as many waves as stay resident: a block per four pairs
  // spent as long being dispatched as scoring (198 us at N = 500)
  const int64_t npairs = (int64_t)N * (N - 1) / 2;
  if (npairs > 0x7fffffff - 64) return hipErrorInvalidValue;
  const int64_t per = (npairs + kScResident - 1) / kScResident;
  const dim3 grid((unsigned)((npairs + kScWaves * per - 1) / (kScWaves * per))), block(64 * kScWaves);
  auto launch = [&](auto avg, auto norm) {
    hipLaunchKernelGGL((pair_score_kernel<decltype(avg)::value, decltype(norm)::value>), grid, block, 0, st, J, N, q,
                       (int32_t)npairs, (int32_t)per, o, freq, raw);
  };
  auto launch_norm = [&](auto avg) {
    if (o.norm == PLM_NORM_BURKOFF) launch(avg, std::integral_constant<int, PLM_NORM_BURKOFF>{});
    else if (o.norm == PLM_NORM_LP) launch(avg, std::integral_constant<int, PLM_NORM_LP>{});
    else launch(avg, std::integral_constant<int, PLM_NORM_FROB>{});
  };
  if (o.combine == PLM_COMBINE_AVG) launch_norm(std::true_type{});
  else launch_norm(std::false_type{});
  if (N <= kCorSmall) {
    hipLaunchKernelGGL(correct_small_kernel, dim3(1), dim3(1024), 0, st, raw, N, o.correction, cor);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(rowsum_kernel, dim3(N), dim3(64), 0, st, raw, N, cor);
  hipLaunchKernelGGL(correct_kernel, dim3((N + kCorRows - 1) / kCorRows), dim3(256), 0, st, raw, N, o.correction, cor);
  hipLaunchKernelGGL(diag_zero_kernel, dim3((N + 255) / 256), dim3(256), 0, st, cor, N);
  return hipGetLastError();
}

hipError_t launch_score(const float* J, int32_t N, int32_t q, double* fn, double* cfn,
                        hipStream_t st) {
  ScoreOpts o;
  o.combine = PLM_COMBINE_AVG;
  o.norm = PLM_NORM_FROB;
  o.p = 2.0;
  o.exclude_gap = 0;
  o.correction = PLM_CORR_APC;
  return launch_score_ex(J, N, q, o, nullptr, fn, cfn, st);
}

// Reweighted single-site frequencies f_i(k) = sum_b w_b [sigma_i^b = k] / B_eff:
// one block per column; per-thread FP64 counters in LDS (eight rows' loads in
// flight per thread), then a fixed-order sum over the threads, eight lanes per
// state.  Bound: load latency (N = 200, B = 10 000: 29 -> 16 us; one row in
// flight per thread and 256 serial adds per state before).
__global__ __launch_bounds__(256) void freq_kernel(const uint8_t* __restrict__ msa, int32_t B,
                                                   int32_t N, int32_t q,
                                                   const double* __restrict__ w,
                                                   const double* __restrict__ beff,
                                                   double* __restrict__ f) {
  __shared__ double cnt[256 * kQMax];
  const int i = blockIdx.x, t = threadIdx.x;
  for (int k = 0; k < kQMax; ++k) cnt[t * kQMax + k] = 0.0;
  constexpr int U = 8;
  for (int b0 = t; b0 < B; b0 += 256 * U) {
    int s[U];
    double wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int b = b0 + 256 * u;
      s[u] = b < B ? msa[(size_t)b * N + i] : 255;
      wv[u] = b < B ? w[b] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s[u] < q) cnt[t * kQMax + s[u]] += wv[u];
  }
  __syncthreads();
  const int k = t >> 3, p = t & 7;
  if (k < q) {
    double s = 0.0;
#pragma unroll 8
    for (int u = 0; u < 32; ++u) s += cnt[(8 * u + p) * kQMax + k];
    for (int d = 4; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
    if (p == 0) f[(size_t)i * q + k] = s / *beff;
  }
}

hipError_t launch_frequencies(const uint8_t* msa, int32_t B, int32_t N, int32_t q, const double* w,
                              const double* beff, double* f, hipStream_t st) {
  hipLaunchKernelGGL(freq_kernel, dim3(N), dim3(256), 0, st, msa, B, N, q, w, beff, f);
  return hipGetLastError();
}

}  // namespace plm
