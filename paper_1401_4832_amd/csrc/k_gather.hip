// k_gather.hip -- gather evaluation of the per-site objective and residuals of
// asymmetric plmDCA (sec. 3.4 step 3: eqs. g_regdef2, g_gradh2,
// g_gradJ2) for many sites at once.
//
// Forward (one block = one site r x a tile of sequences): the site's coupling
// slice J_r is streamed through LDS eight columns at a time; each lane adds
// J_ri(s, sigma_i^b) into the energy E_b(s) of its (sequence, state) pair
// (eq. condpfinal); then every lane takes one sequence through its states:
// log Z_b, the objective term w_b (log Z_b - E_b(sigma_r^b)) and the residuals
// R_b(s) = w_b (P_b(s) - [sigma_r^b = s]), which leave in the form the path's
// gradient kernel reads (k_mfma.hip).
// Bound: LDS, one 4-byte word per (row, column, state): 32 a clock and CU,
// with the symbols 25.  Measured, all sites at N = 500, B = 50 000: 24 -> 19 ms
// (the softmax over 21 lanes by shuffles, a row at a time with its loads inside
// the loop and byte stores of the digits, took a third of it), N = 150,
// B = 8000: 830 -> 425 us, N = 40, B = 500: 66 -> 22 us.  A wave's read and its
// two vector instructions take 2.7 clocks a CU at best (a read alone 2.2); the
// loop takes 2.8 at N = 500.
#include "plm_internal.h"

namespace plm {

int32_t forward_tile_seqs(int32_t nb) { return kFwdWaves * kSlots * nb; }

// J chunk of the gather forward: kFwdPos columns of kQMax rows of 64 floats;
// the same LDS later parks the energies of 48 rows per wave.
constexpr int kFwdPos = 8;
constexpr int kPosBytes = kQMax * kRowF * 4;  // 5376
static_assert((kFwdPos - 1) * kPosBytes + 20 * 256 + 255 < 65536, "LDS offsets fit the immediate field");
constexpr int kFwdJFloats = kFwdPos * kQMax * kRowF;
constexpr int kParkRows = 16 * kSlots;  // rows of a wave parked at a time
constexpr int kFwdParkFloats = kFwdWaves * kParkRows * kSlot;
// LDS floats of the forward block: the J chunk (with LO, as the FP64 sums of
// the couplings' high and low words, twice the bytes), or the parked energies
// (AT values)
template <class AT, bool LO>
constexpr int fwd_lds_floats() {
  return kFwdJFloats * (LO ? 2 : 1) > kFwdParkFloats * (int)(sizeof(AT) / 4) ? kFwdJFloats * (LO ? 2 : 1)
                                                                             : kFwdParkFloats * (int)(sizeof(AT) / 4);
}

// One forward work item: site r x sequence tile `tile` of one alignment.
// lds: J_r for kFwdPos columns, 3 copies per row, with a fixed pitch of kQMax
// rows per column so that a column's offset is a compile-time constant (and
// later the parked energies); sgl: the tile's symbols for those columns; red:
// FP64 reduction scratch.  AT is the accumulation type of the energies and of
// the log-softmax and residuals: float, or double (the precise path, whose
// residuals go out as two sets of int8 digits, rfrag = 3).  LO (with double):
// the point is h + h_lo, J + J_lo; the low words are staged and gathered like
// the high ones, and each pair is summed in FP64.
template <int NB, class AT, bool LO>
__device__ inline void fwd_item(const EvalArgs& a, int r, int tile, float* lds, uint2* sgl,
                                double* red) {
  static_assert(!LO || sizeof(AT) == 8, "low-order words only with FP64 accumulation");
  constexpr int tileSeq = kFwdWaves * kSlots * NB;
  const int q = a.q, N = a.N, qq = q * q;
  const int tid = item_tid(), lane = tid & 63, wid = tid >> 6;
  const int slot = lane / kSlot, s = lane - slot * kSlot;
  const int slotA = slot < kSlots ? slot : kSlots - 1;  // lane 63 shadows slot 2 for addressing
  const bool act = (slot < kSlots) && (s < q);
  // the alignment's groups of 48 rows, divided evenly over the tiles; a tile's
  // groups go to its waves in turn, so that tiles and waves are equally loaded
  // (whole tiles first left the last one nearly empty: with N = 120, B = 5000,
  // 3.3 tiles a site, 178 -> 156 us; N = 150, B = 8000 476 -> 425 us with the rows
  // per tile chosen for it)
  const int ngroups = (a.B3 + kParkRows - 1) / kParkRows, tgroups = (ngroups + a.tiles - 1) / a.tiles;
  const int tile0 = tile * tgroups * kParkRows;
  const int tgr = min(tgroups, ngroups - tile * tgroups);  // this tile's groups with rows (none: not positive)
  const int ng = __builtin_amdgcn_readfirstlane(max(0, min(NB / 16, (tgr - wid + kFwdWaves - 1) / kFwdWaves)));  // this wave's
  const int tw = wid * kParkRows + slotA;  // the tile row of the wave's row j: tw + trow(j)
  constexpr auto trow = [](int j) { return (j / 16) * (kFwdWaves * kParkRows) + (j % 16) * kSlots; };

  AT E[NB];
  AT hv = act ? (AT)gmem(a.h)[r * q + s] : (AT)0;
  if (LO && act) hv += (AT)gmem(a.h_lo)[r * q + s];
#pragma unroll
  for (int j = 0; j < NB; ++j) E[j] = hv;

  const size_t Jr = (size_t)r * N * qq;
  const int nchunks = (N + kFwdPos - 1) / kFwdPos;
  // groups that lie past the alignment's rows (padded to three) are left out:
  // no row of them is read by the gradient (the rows of the last gradient chunk
  // past the alignment are zeroed once per alignment)
  const char* L = reinterpret_cast<const char*>(lds);
  // LDS byte address of row (p, sigma), this lane's word: p * kPosBytes (an
  // immediate offset) + sigma * 256 + 4 * lane, where the last two are one
  // byte permute: byte 0 = 4 * lane (< 256), byte 1 = the symbol byte
  const uint32_t lane4 = 4u * lane;
  // the next chunk's couplings and symbols travel in registers while the
  // current chunk is gathered.  Entry e of a chunk (column p, row k, state s)
  // is e values after the chunk's first in J_r, whatever the column
  constexpr int kJPer = (kFwdPos * kQMax * kQMax + kFwdThreads - 1) / kFwdThreads;
  constexpr int kSPer = (tileSeq + kFwdThreads - 1) / kFwdThreads;
  float jv[kJPer], jl[LO ? kJPer : 1];
  uint2 sv[kSPer];
  int jdst[kJPer];  // the entry's word in the staged chunk; -1 past its end
#pragma unroll
  for (int k = 0; k < kJPer; ++k) {
    const int e = tid + k * kFwdThreads;
    const int p = e / qq, rem = e - p * qq, kk = rem / q;
    jdst[k] = e < kFwdPos * qq ? (p * kQMax + kk) * kRowF + rem - kk * q : -1;
  }
  const int Nqq = N * qq, self0 = r * qq;
  auto load = [&](int c) {
    const int c0 = c * kFwdPos * qq;
#pragma unroll
    for (int k = 0; k < kJPer; ++k) {
      const int e = c0 + tid + k * kFwdThreads;
      const bool in = jdst[k] >= 0 && e < Nqq && (unsigned)(e - self0) >= (unsigned)qq;
      jv[k] = in ? gmem(a.J)[Jr + e] : 0.f;
      if (LO) jl[k] = in ? gmem(a.J_lo)[Jr + e] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < kSPer; ++k) {
      const int e = tid + k * kFwdThreads;
      sv[k] = uint2{0, 0};
      if (e < tgr * kParkRows)
        sv[k] = gload_u2(a.msa_cm + ((size_t)(c >> 1) * a.B_pad + tile0 + e) * kFwdChunk + 8 * (c & 1));
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int k = 0; k < kJPer; ++k) {
      if (jdst[k] >= 0) {
        if (LO) {
          // the pair's exact FP64 sum (two 24-bit significands 2^24 apart fit
          // 53 bits), one 8-byte word per entry: the gather then reads one
          // word and adds once per term
          double* row = reinterpret_cast<double*>(lds) + jdst[k];
          const double v = (double)jv[k] + (double)jl[k];
          row[0] = v;
          row[kSlot] = v;
          row[2 * kSlot] = v;
        } else {
          float* row = lds + jdst[k];
          row[0] = jv[k];
          row[kSlot] = jv[k];
          row[2 * kSlot] = jv[k];
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kSPer; ++k) {
      const int e = tid + k * kFwdThreads;
      if (e < tileSeq) sgl[e] = sv[k];
    }
  };
  load(0);
  for (int c = 0; c < nchunks; ++c) {
    __syncthreads();  // every wave is done with the previous chunk
    store();
    __syncthreads();
    if (c + 1 < nchunks) load(c + 1);
    if (ng == 0) continue;
    // row j + 1's words are read while row j's are added, and its symbols one
    // row earlier still: one row at a time left the LDS idle between a row's
    // reads and its sums
    AT v[2][kFwdPos];
    auto gather = [&](uint2 sg, AT (&d)[kFwdPos]) {
#pragma unroll
      for (int p = 0; p < kFwdPos; ++p) {
        const uint32_t word = p < 4 ? sg.x : sg.y;
        const uint32_t addr = __builtin_amdgcn_perm(lane4, word, 0x0c0c0004u | ((uint32_t)(p & 3) << 8));
        if (LO) {
          // 8-byte rows: twice the float row's byte address, from a base per
          // four positions so that the offset fits the immediate field
          const char* L2 = L + (p < 4 ? 0 : 4 * 2 * kPosBytes);
          d[p] = *reinterpret_cast<const double*>(L2 + 2 * addr + (p & 3) * 2 * kPosBytes);
        } else {
          d[p] = (AT)*reinterpret_cast<const float*>(L + addr + p * kPosBytes);
        }
      }
    };
    gather(sgl[tw], v[0]);
    uint2 sn = sgl[tw + kSlots];
#pragma unroll
    for (int g = 0; g < NB / 16; ++g) {
      if (g >= ng) continue;
#pragma unroll
      for (int jj = 0; jj < 16; ++jj) {
        const int j = 16 * g + jj;
        const uint2 sc = sn;
        // (past the wave's last group these reads are of rows that are not used, inside the tile's arrays)
        if (j + 2 < NB) sn = sgl[tw + trow(j + 2)];
        if (j + 1 < NB) gather(sc, v[(j + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        // two accumulation chains (even and odd columns)
        const AT(&d)[kFwdPos] = v[j & 1];
        AT acc0 = E[j], acc1 = d[1];
#pragma unroll
        for (int p = 0; p < kFwdPos; ++p) {
          if (p == 1) continue;
          if (p & 1) acc1 += d[p];
          else acc0 += d[p];
        }
        E[j] = acc0 + acc1;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // log-softmax, objective and residuals, 48 rows of the wave at a time: their
  // energies are parked in the (now free) LDS, every lane takes one row through
  // its states in registers and puts the residuals in the energies' place, then
  // lane 21 g + s takes state s of the rows 16 g .. 16 g + 15 to the field
  // gradient and to HBM, sixteen rows of a digit in one store.
  double facc = 0.0, ghacc = 0.0;
  const double rscale = a.rfrag == 4 ? ldexp(1.0, kR4ScaleLog2 - a.wexp[0]) : (double)(1 << kRiScaleLog2);
  __syncthreads();  // every wave is done with the last chunk
  AT* park = reinterpret_cast<AT*>(lds) + wid * (kParkRows * kSlot);
#pragma unroll 1
  for (int g = 0; g < ng; ++g) {
    const int b0 = tile0 + (g * kFwdWaves + wid) * kParkRows;  // the first of the 48 rows
    // this lane's row: its symbol at the site and its weight
    const int b = b0 + min(lane, kParkRows - 1);
    const int sr = gmem(a.msa_cm)[((size_t)(r / kFwdChunk) * a.B_pad + b) * kFwdChunk + r % kFwdChunk];
    const double wb = b < a.B ? gmem(a.w)[b] : 0.0;
    if (slot < kSlots) {
      // (one straight-line copy of the stores per g: the energies stay in registers)
      with_count<0, NB / 16 - 1>(g, [&](auto gc) {
#pragma unroll
        for (int jj = 0; jj < 16; ++jj)
          park[(3 * jj + slot) * kSlot + s] = s < q ? E[decltype(gc)::value * 16 + jj] : (AT)-INFINITY;
      });
    }
    wave_sync();
    if (lane < kParkRows) {
      AT* row = park + lane * kSlot;
      // four states at a time (fences keep the others in LDS, not in registers)
      AT m = row[kSlot - 1];
#pragma unroll
      for (int k = 0; k < kSlot - 1; ++k) m = fmax(m, row[k]);
      const AT esr = row[sr];
      AT part[5];
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        AT x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          x[u] = (AT)exp(row[4 * k + u] - m);
          row[4 * k + u] = x[u];
        }
        part[k] = (x[0] + x[1]) + (x[2] + x[3]);
        __builtin_amdgcn_sched_barrier(0);
      }
      const AT xl = (AT)exp(row[kSlot - 1] - m);
      row[kSlot - 1] = xl;
      // pairwise sum: a binary tree over the first sixteen states and over the last five
      const AT sum = ((part[0] + part[1]) + (part[2] + part[3])) + (part[4] + xl);
      const AT lse = m + (AT)log(sum);
      facc += wb * (double)(lse - esr);
      // P = x / sum by the reciprocal with one correction step
      const AT inv = (AT)1 / sum, wa = (AT)wb;
#pragma unroll
      for (int k = 0; k < kSlot; ++k) {
        const AT x = row[k];
        AT P = x * inv;
        P = fma(fma(-P, sum, x), inv, P);
        row[k] = wa * (P - (k == sr ? (AT)1 : (AT)0));
        if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
    wave_sync();
    if (a.rfrag == 0) {
      // FP32 rows: the 48 rows are contiguous
      auto Rr = gmem_w(a.R) + ((size_t)r * a.B3 + b0) * kSlot;
      const int n = min(kParkRows, a.B3 - b0) * kSlot;
#pragma unroll
      for (int k = 0; k < (kParkRows * kSlot + 63) / 64; ++k)
        if (lane + 64 * k < n) Rr[lane + 64 * k] = (float)park[lane + 64 * k];
    }
    if (slot < kSlots) {
      const int bg = b0 + 16 * slot;  // sixteen rows from here
      const AT* col = park + 16 * slot * kSlot + s;
      // rows of every tile are written, zeros past B; states past q hold zeros
      if (a.rfrag == 0) {
#pragma unroll
        for (int t = 0; t < 16; ++t) ghacc += (double)col[t * kSlot];
      } else if (a.rfrag == 1) {
        // FP16 hi/lo pieces of R * 2^12 in the grouped gradient's fragment order
        auto Rf = gmem_w(reinterpret_cast<u32x4_t*>(a.R));
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          u32x4_t hi, lo;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            uint32_t hw = 0, lw = 0;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const AT v = col[(8 * hf + 2 * t + u) * kSlot];
              ghacc += (double)v;
              const float y = (float)v * kRfScale;
              const _Float16 yh = (_Float16)y;
              const _Float16 yl = (_Float16)(y - (float)yh);
              hw |= (uint32_t)__builtin_bit_cast(uint16_t, yh) << (16 * u);
              lw |= (uint32_t)__builtin_bit_cast(uint16_t, yl) << (16 * u);
            }
            hi[t] = hw;
            lo[t] = lw;
          }
          const size_t ix = rfrag_index(r, a.B_pad >> 8, bg + 8 * hf, s);
          Rf[ix / 8] = hi;
          Rf[(ix + kRfPieceWords) / 8] = lo;
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        // int8 digits in the int8 gradient's fragment order: three of round(R * 2^22); with
        // rfrag = 3 three more, in a second set, of the remainder's round((R * 2^22 - v) * 2^22);
        // with rfrag = 4 four of round(R * 2^(30 - e))
        auto Ri = gmem_w(reinterpret_cast<u32x4_t*>(a.R));
        const int nch = a.B_pad >> 8;
        // the digits of sixteen integers: ND planes kRiDigitBytes apart from byte ix on, highest first
        auto put = [&](size_t ix, auto nd, auto&& integer) {
          constexpr int ND = decltype(nd)::value;
          u32x4_t dw[ND];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            uint32_t w[ND];
#pragma unroll
            for (int d = 0; d < ND; ++d) w[d] = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              int y = integer(col[(4 * t + u) * kSlot]);
#pragma unroll
              for (int d = ND - 1; d >= 0; --d) {
                const int lo = (int)(int8_t)(y & 255);
                w[d] |= (uint32_t)(lo & 255) << (8 * u);
                y = (y - lo) >> 8;
              }
            }
#pragma unroll
            for (int d = 0; d < ND; ++d) dw[d][t] = w[d];
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int d = 0; d < ND; ++d) Ri[(ix + (size_t)d * kRiDigitBytes) / 16] = dw[d];
        };
        constexpr std::integral_constant<int, 3> three;
        if (a.rfrag == 4) {
          put(r4frag_index(r, nch, bg, s), std::integral_constant<int, 4>{}, [&](AT v) {
            ghacc += (double)v;
            return (int)rint((double)v * rscale);
          });
        } else {
          const size_t ix = rifrag_index(r, nch, bg, s);
          if (sizeof(AT) == 4) {
            put(ix, three, [&](AT v) {
              ghacc += (double)v;
              return (int)rintf((float)v * (float)(1 << kRiScaleLog2));
            });
          } else {
            put(ix, three, [&](AT v) {
              ghacc += (double)v;
              return (int)rint((double)v * rscale);
            });
            put(ix + (size_t)a.N * nch * kRiChunkBytes, three, [&](AT v) {
              const double y = (double)v * rscale;
              return (int)rint((y - rint(y)) * rscale);
            });
          }
        }
      }
    }
    wave_sync();
  }
  const double ftot = block_sum_f64(facc, red);
  if (tid == 0) gmem_w(a.f_part)[(size_t)tile * N + r] = ftot;
  red[wid * 64 + lane] = (slot < kSlots) ? ghacc : 0.0;
  __syncthreads();
  if (tid < kSlot) {
    double t = 0.0;
    for (int w = 0; w < kFwdWaves; ++w)
      for (int c = 0; c < kSlots; ++c) t += red[w * 64 + c * kSlot + tid];
    gmem_w(a.gh_part)[((size_t)tile * N + r) * kSlot + tid] = t;
  }
}

// Persistent forward kernel: drains the forward work items of the batch.
template <int NB, class AT, bool LO>
__global__ __launch_bounds__(kFwdThreads, sizeof(AT) == 4 ? 4 : 2) void fwd_kernel(BatchArgs b) {
  __shared__ __attribute__((aligned(16))) float lds[fwd_lds_floats<AT, LO>()];
  __shared__ uint2 sgl[kFwdWaves * kSlots * NB];
  __shared__ double red[kFwdWaves * 64];
  __shared__ int32_t item_s;
  int32_t qi = -1;
  const int32_t total = total_items(b, KIND_FWD);
  for (;;) {
    if (threadIdx.x == 0) item_s = next_item(b.ctr + KIND_FWD * kQueues, total, qi);
    __syncthreads();
    const int32_t t = __builtin_amdgcn_readfirstlane(item_s);
    if (t < 0) break;
    const Item it = decode_item(b, KIND_FWD, t);
    EvalArgs a = load_uniform(b.ev + it.m);
    // path 0: FP32 rows where the weights' range is too wide for its digits
    if (sizeof(AT) == 4 && a.rfrag == 4 && __builtin_amdgcn_readfirstlane(it.wide)) a.rfrag = 0;
    fwd_item<NB, AT, LO>(a, it.r, it.sub, lds, sgl, red);
    __syncthreads();
  }
}

// The precise path accumulates in FP64 with tiles of kFwdF64Rows rows per wave.
constexpr int kFwdF64Rows = 32;
int32_t forward_f64_tile_seqs() { return kFwdWaves * kSlots * kFwdF64Rows; }

hipError_t launch_forward(const BatchArgs& b, int32_t nb, int32_t nblocks, int32_t f64, hipStream_t st) {
  if (f64 == 2) {
    hipLaunchKernelGGL((fwd_kernel<kFwdF64Rows, double, true>), dim3(nblocks), dim3(kFwdThreads), 0, st, b);
    return hipGetLastError();
  }
  if (f64) {
    hipLaunchKernelGGL((fwd_kernel<kFwdF64Rows, double, false>), dim3(nblocks), dim3(kFwdThreads), 0, st, b);
    return hipGetLastError();
  }
  switch (nb) {
    case 16: hipLaunchKernelGGL((fwd_kernel<16, float, false>), dim3(nblocks), dim3(kFwdThreads), 0, st, b); break;
    case 32: hipLaunchKernelGGL((fwd_kernel<32, float, false>), dim3(nblocks), dim3(kFwdThreads), 0, st, b); break;
    case 64: hipLaunchKernelGGL((fwd_kernel<64, float, false>), dim3(nblocks), dim3(kFwdThreads), 0, st, b); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

int32_t forward_resident_blocks(int32_t nb, int32_t f64) {
  int per = 0;
  hipError_t e = hipErrorInvalidValue;
  if (f64) {
    e = f64 == 2
            ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fwd_kernel<kFwdF64Rows, double, true>, kFwdThreads, 0)
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fwd_kernel<kFwdF64Rows, double, false>, kFwdThreads,
                                                           0);
    return (e == hipSuccess && per > 0) ? per : 1;
  }
  switch (nb) {
    case 16: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fwd_kernel<16, float, false>, kFwdThreads, 0); break;
    case 32: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fwd_kernel<32, float, false>, kFwdThreads, 0); break;
    case 64: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fwd_kernel<64, float, false>, kFwdThreads, 0); break;
    default: break;
  }
  return (e == hipSuccess && per > 0) ? per : 1;
}

}  // namespace plm
