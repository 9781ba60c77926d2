// LayerNorm in cluster order + quantization + packing for calls with few rows per compute unit: the arithmetic and the
// results of ln_quant.hip, arranged for latency.
//
// A workgroup takes R rows at once and is done.  The pipelined kernel walks one row per barrier, which hides
// everything behind the row loop when there is one; with one to four rows per workgroup its chain of waits is the time:
// tables, constants, row, partial sums, statistics wave, gather, row sum.  Here all loads (rows, per-position constants,
// one lane-wise read of the cluster tables) are requested at once, every wave reduces its own sums with cross-lane
// swaps, all waves derive the statistics of the R rows side by side (a row per 16 lanes) so that no result is handed
// back through a second barrier, and the barriers wait for LDS only, not for loads or stores in flight.
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "ln_common.h"
#include "rptq_internal.h"

namespace rptq {

// Cluster tables as the lanes read them: lane i holds cluster i (one coalesced read per table).
struct LnRowsTab {
  int32_t pad_off[RPTQ_MAX_CLUSTERS];      // padded start of cluster i; beyond the last cluster: INT32_MAX
  float inv_s[RPTQ_MAX_CLUSTERS];
  float s[RPTQ_MAX_CLUSTERS];
  int32_t z[RPTQ_MAX_CLUSTERS];
  int32_t zb[RPTQ_MAX_CLUSTERS];           // z - qmin
};

// Sums of four values over the wave; the 16 lanes of DPP row k end with the sum of v_k.  Two swaps halve the number
// of values while they add lanes up (21 instructions for four sums instead of 72).
__device__ __forceinline__ double swap_add(double a, double b, bool half) {
  const uint64_t x = static_cast<uint64_t>(__double_as_longlong(a)), y = static_cast<uint64_t>(__double_as_longlong(b));
  const uint32_t xl = static_cast<uint32_t>(x), xh = static_cast<uint32_t>(x >> 32);
  const uint32_t yl = static_cast<uint32_t>(y), yh = static_cast<uint32_t>(y >> 32);
  // half: lanes 32..63 of a and 0..31 of b change places; else odd rows of a and even rows of b
  const auto lo = half ? __builtin_amdgcn_permlane32_swap(xl, yl, false, false) : __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
  const auto hi = half ? __builtin_amdgcn_permlane32_swap(xh, yh, false, false) : __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
  return __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi[0]) << 32) | lo[0])) +
         __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi[1]) << 32) | lo[1]));
}
__device__ __forceinline__ double wave_sum4(double v0, double v1, double v2, double v3) {
  return row16_sum(swap_add(swap_add(v0, v2, true), swap_add(v1, v3, true), false));
}

// Workgroup barrier that orders LDS accesses only: global loads and stores stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kRowsMaxWaves = 16;
static size_t rows_lds_bytes(int d, int rows) { return static_cast<size_t>(rows) * (d * 2 + 16) + 3 * ((rows + 3) / 4 * 4) * kRowsMaxWaves * sizeof(double); }

template <int BITS, int NUNIT, int NCH, int R, bool LN>
__global__ void __launch_bounds__(1024) ln_rows_kernel(LnQuantArgs a, LnRowsTab tab) {
  constexpr int UC = Unit<BITS>::kCodes;
  constexpr int ND = UC / 4;
  constexpr float kUMax = static_cast<float>((1 << BITS) - 1);
  constexpr int kQMin = -(1 << (BITS - 1));
  constexpr int RG = (R + 3) / 4;                              // rows are summed four at a time, one per 16 lanes
  constexpr int RP = RG * 4;

  extern __shared__ __align__(16) unsigned char smem[];        // R row buffers, then the sums
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6), nw = static_cast<int>(blockDim.x) >> 6;
  const int TU = static_cast<int>(blockDim.x);
  const int rowbuf_bytes = a.d * 2 + 16;                       // (a spare slot for surplus lanes)
  // {sum x, sum x^2, de-quantized row sum} of every row and wave
  auto sums = reinterpret_cast<double(*)[RP][kRowsMaxWaves]>(smem + R * rowbuf_bytes);
  const int64_t row0 = static_cast<int64_t>(blockIdx.x) * R;

  // ---- every load, rows first: indices are clamped, nothing sits under a lane-dependent branch ------------
  u4v x[R][NCH];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t row = row0 + r < a.M ? row0 + r : a.M - 1;
    const u4v* p = reinterpret_cast<const u4v*>(a.x + row * a.chunks);
#pragma unroll
    for (int c = 0; c < NCH; ++c) x[r][c] = p[min(tid + c * TU, a.chunks - 1)];
  }
  const int t_off = tab.pad_off[lane], t_z = tab.z[lane], t_zb = tab.zb[lane];
  const float t_inv = tab.inv_s[lane], t_s = tab.s[lane];
  u4v pc[NUNIT][ND], pg[LN ? NUNIT : 1][LN ? ND : 1], pb[LN ? NUNIT : 1][LN ? ND : 1];
#pragma unroll
  for (int n = 0; n < NUNIT; ++n) {
    const int u = tid + n * TU, uu = u < a.n_units ? u : 0;
#pragma unroll
    for (int v = 0; v < ND; ++v) {                             // a unit's positions are runs of four
      const int pos = (BITS == 3) ? (uu >> 1) * kGroup + pos3(uu & 1, v * 4) : uu * 8 + v * 4;
      pc[n][v] = *reinterpret_cast<const u4v*>(a.perm_pad + pos);
      if (LN) {
        pg[n][v] = *reinterpret_cast<const u4v*>(a.gamma_pad + pos);
        pb[n][v] = *reinterpret_cast<const u4v*>(a.beta_pad + pos);
      }
    }
  }

  // ---- rows to LDS, exact fp64 sums ---------------------------------------------------------------------
  double s1[RP], s2[RP];
#pragma unroll
  for (int r = 0; r < RP; ++r) s1[r] = s2[r] = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int idx = tid + c * TU;
      const bool ok = idx < a.chunks;
      *reinterpret_cast<u4v*>(smem + r * rowbuf_bytes + (ok ? idx * 16 : a.d * 2)) = x[r][c];
      if (LN) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t w = ok ? x[r][c][k] : 0u;
          const double lo = static_cast<double>(bf16_lo(w)), hi = static_cast<double>(bf16_hi(w));
          s1[r] += lo;
          s2[r] = fma(lo, lo, s2[r]);
          s1[r] += hi;
          s2[r] = fma(hi, hi, s2[r]);
        }
      }
    }
  if (LN) {
#pragma unroll
    for (int g = 0; g < RP; g += 4) {
      const double w1 = wave_sum4(s1[g], s1[g + 1], s1[g + 2], s1[g + 3]), w2 = wave_sum4(s2[g], s2[g + 1], s2[g + 2], s2[g + 3]);
      if ((lane & 15) == 0) {
        sums[0][g + (lane >> 4)][wid] = w1;
        sums[1][g + (lane >> 4)][wid] = w2;
      }
    }
  }

  // ---- constants of this thread's units (while the sums travel) -------------------------------------------
  uint32_t src[NUNIT][UC];           // LDS byte offsets of the source channels inside a row buffer
  uint32_t keep[NUNIT][ND], fill[NUNIT][ND];
  float inv_s[NUNIT], round_back[NUNIT], code_floor[NUNIT];
  double sdq[NUNIT];
  int32_t usum_fix[NUNIT];
  bool unit_ok[NUNIT];
  int out_off[NUNIT];
#pragma unroll
  for (int n = 0; n < NUNIT; ++n) {
    const int u = tid + n * TU;
    unit_ok[n] = u < a.n_units;
    const int uu = unit_ok[n] ? u : 0;
    const int gbase = (BITS == 3) ? (uu >> 1) * kGroup : uu * 8;
    out_off[n] = (BITS == 3) ? (uu >> 1) * 12 + (uu & 1) * 4 : uu * BITS;
    // cluster of the unit: that of the wave's first unit, and the few boundaries that lie inside the wave's positions
    const int u_first = __builtin_amdgcn_readfirstlane(u);
    const int p_first = (BITS == 3) ? (u_first >> 1) * kGroup : u_first * 8;
    const int p_last = (BITS == 3) ? ((u_first + 63) >> 1) * kGroup : (u_first + 63) * 8;
    const int c_first = __builtin_popcountll(__ballot(t_off <= p_first)), c_last = __builtin_popcountll(__ballot(t_off <= p_last));
    int ci = c_first - 1;
    for (int i = c_first; i < c_last; ++i) ci += (gbase >= __builtin_amdgcn_readlane(t_off, i)) ? 1 : 0;
    if (!unit_ok[n]) ci = 0;
    const int z = __builtin_amdgcn_ds_bpermute(ci * 4, t_z);
    inv_s[n] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(ci * 4, __builtin_bit_cast(int, t_inv)));
    const float zbf = static_cast<float>(__builtin_amdgcn_ds_bpermute(ci * 4, t_zb));
    round_back[n] = kRoundMagic - zbf;
    sdq[n] = static_cast<double>(__builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(ci * 4, __builtin_bit_cast(int, t_s))));
    // (ReLU: a lower clamp of the biased code at the biased zero point, see ln_quant.hip)
    code_floor[n] = a.relu ? fminf(zbf, kUMax) : -__builtin_huge_valf();
    int n_real = 0;
#pragma unroll
    for (int w = 0; w < ND; ++w) {
      keep[n][w] = 0xffffffffu;
      fill[n][w] = 0u;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int ch = static_cast<int>(pc[n][w][b]);
        const bool real = ch >= 0;
        n_real += real ? 1 : 0;
        src[n][w * 4 + b] = real ? static_cast<uint32_t>(ch) * 2u : 0u;
        if (!real) {                                 // pad position: force code 0 (biased byte = -qmin)
          keep[n][w] &= ~(0xffu << (8 * b));
          fill[n][w] |= static_cast<uint32_t>(-kQMin) << (8 * b);
        }
      }
    }
    usum_fix[n] = UC * kQMin - n_real * z;
  }

  lds_barrier();                                               // rows and sums are in LDS
  float mu[RG], rstd[RG];                                      // lanes 16 k .. 16 k + 15: of row k of the four
#pragma unroll
  for (int g = 0; g < RG; ++g) {
    mu[g] = 0.0f;
    rstd[g] = 1.0f;
    if (LN) {
      const int w = lane & 15, r = g * 4 + (lane >> 4);
      const double v1 = sums[0][r][w], v2 = sums[1][r][w];
      row_stats(row16_sum(w < nw ? v1 : 0.0), row16_sum(w < nw ? v2 : 0.0), a.d, a.eps, &mu[g], &rstd[g]);
    }
  }

  // ---- gather in cluster order, normalize, quantize, pack ----------------------------------------------
  double rt[RP];
#pragma unroll
  for (int r = 0; r < RP; ++r) rt[r] = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool row_ok = row0 + r < a.M;
    // (by the lanes' permutation, into vector registers: an operand from a scalar register halves the rate of the
    // additions and products below)
    const float mu_r = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(64 * (r % 4), __builtin_bit_cast(int, mu[r / 4])));
    const float rstd_r = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(64 * (r % 4), __builtin_bit_cast(int, rstd[r / 4])));
    const unsigned char* rowbuf = smem + r * rowbuf_bytes;
    uint8_t* out_row = a.codes + (row0 + r) * a.row_bytes;
#pragma unroll
    for (int n = 0; n < NUNIT; ++n) {
      uint32_t D[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int e = 0; e < UC; ++e) {
        const uint32_t h = *reinterpret_cast<const uint16_t*>(rowbuf + src[n][e]);
        float y = __uint_as_float(h << 16);
        if (LN) y = ln_chain(y, mu_r, rstd_r, __uint_as_float(pg[n][e / 4][e & 3]), __uint_as_float(pb[n][e / 4][e & 3]));
        float b = round_biased(__fmul_rn(y, inv_s[n]), round_back[n]);
        b = (BITS < 8) ? __builtin_amdgcn_fmed3f(b, code_floor[n], kUMax) : fmaxf(b, code_floor[n]);
        D[e / 4] = __builtin_amdgcn_cvt_pk_u8_f32(b, e & 3, D[e / 4]);
      }
      uint32_t usum = 0;
#pragma unroll
      for (int w = 0; w < ND; ++w) {
        D[w] = (D[w] & keep[n][w]) | fill[n][w];
        usum = __builtin_amdgcn_sad_u8(D[w], 0u, usum);
      }
      const double part = sdq[n] * static_cast<double>(static_cast<int32_t>(usum) + usum_fix[n]);
      rt[r] += unit_ok[n] ? part : 0.0;
      store_unit<BITS>(D, tid & 1, unit_ok[n] && row_ok, out_row + out_off[n]);
    }
  }
  if (a.rowterm == nullptr) return;
#pragma unroll
  for (int g = 0; g < RP; g += 4) {
    const double w3 = wave_sum4(rt[g], rt[g + 1], rt[g + 2], rt[g + 3]);
    if ((lane & 15) == 0) sums[2][g + (lane >> 4)][wid] = w3;
  }
  lds_barrier();
  if (wid < RG) {
    const int r = wid * 4 + (lane >> 4);
    const double v3 = sums[2][r][lane & 15];
    const double total = row16_sum((lane & 15) < nw ? v3 : 0.0);
    if ((lane & 15) == 0 && r < R && row0 + r < a.M) a.rowterm[row0 + r] = static_cast<float>(total);
  }
}

template <int BITS, int NUNIT, int NCH, int R, bool LN>
static int32_t launch_rows_kernel(const LnQuantArgs& a, const LnRowsTab& tab, int threads, hipStream_t st) {
  auto kern = ln_rows_kernel<BITS, NUNIT, NCH, R, LN>;
  const size_t shmem = rows_lds_bytes(a.d, R);
  static LdsGrant lds_granted;
  if (int32_t s = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), shmem, &lds_granted, st)) return s;
  hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>((a.M + R - 1) / R)), dim3(threads), shmem, st, a, tab);
  RPTQ_HIP(hipGetLastError());
  return RPTQ_OK;
}

template <int BITS, int NUNIT, int NCH, bool LN>
static int32_t launch_rows_count(const LnQuantArgs& a, const LnRowsTab& tab, int rows, int threads, hipStream_t st) {
  if (rows == 4) return launch_rows_kernel<BITS, NUNIT, NCH, 4, LN>(a, tab, threads, st);
  if (rows == 2) return launch_rows_kernel<BITS, NUNIT, NCH, 2, LN>(a, tab, threads, st);
  return launch_rows_kernel<BITS, NUNIT, NCH, 1, LN>(a, tab, threads, st);
}

template <int BITS, int NUNIT>
static int32_t launch_rows_cfg(const LnQuantArgs& a, const LnRowsTab& tab, int nch, int rows, int threads, hipStream_t st) {
  const bool ln = a.gamma_pad != nullptr;
  if (nch == 1)
    return ln ? launch_rows_count<BITS, NUNIT, 1, true>(a, tab, rows, threads, st) : launch_rows_count<BITS, NUNIT, 1, false>(a, tab, rows, threads, st);
  return ln ? launch_rows_count<BITS, NUNIT, 2, true>(a, tab, rows, threads, st) : launch_rows_count<BITS, NUNIT, 2, false>(a, tab, rows, threads, st);
}

// Which calls come here.  R: one workgroup per compute unit as long as there are rows, up to four each (more rows share
// the per-position constants, 12 bytes a code against the row's 2; eight measured no better).  Beyond that the pipelined
// kernel catches up, the sooner the wider the row.  us, pipelined | this kernel, LayerNorm rows:
//      1 x  2048  4.9 |  3.5      333 x 4072 (3 bits)  8.8 |  6.1     2048 x 2048   9.8 |  7.4     32768 x  768  29.0 | 23.5
//    128 x   768  4.4 |  3.2      512 x 5120          10.3 |  5.7     2048 x 5120  16.3 | 11.2     16384 x 2048  33.4 | 30.9
//     32 x  5120  7.1 |  4.8     1024 x 5120          12.2 |  7.3     4096 x 5120  23.9 | 20.4      8192 x 4096  36.4 | 35.0
//     16 x 12288 10.3 |  7.5     1024 x 12288 (3)     17.2 | 13.9     8192 x 5120  38.7 | 37.7 (3 bits 38.9 | 40.3)
//   and not:  16384 x 4096  58.3 | 66.3    4096 x 6000  26.5 | 30.6    2048 x 8192 (8 bits)  21.0 | 21.7    2048 x 12288  26.1 | 28.8
// Without LayerNorm alike (16 x 12288 6.8 | 5.2, 2048 x 5120 10.9 | 7.6, 4096 x 5120 15.6 | 14.1, 8192 x 5120 23.6 | 23.8).
int32_t launch_ln_rows(const LnQuantArgs& a, const ClusterGeom& geom, const QuantTab& qt, int bits, int nunit, int nch,
                       int threads, int cus, hipStream_t st, bool* served) {
  *served = false;
  if (nch > 2 || nunit > 2 || (bits == 3 && nunit > 1)) return RPTQ_OK;
  const int most = a.d <= 2048 ? 128 : (a.d <= 4096 ? 32 : (a.d <= 5120 ? 16 : 4));     // rows per compute unit
  if (a.M > static_cast<int64_t>(cus) * most) return RPTQ_OK;
  const int rows = a.M <= cus ? 1 : (a.M <= 2 * static_cast<int64_t>(cus) ? 2 : 4);
  LnRowsTab tab;
  for (int i = 0; i < RPTQ_MAX_CLUSTERS; ++i) {
    tab.pad_off[i] = i < geom.g ? geom.pad_off[i] : INT32_MAX;
    tab.inv_s[i] = qt.inv_s[i];
    tab.s[i] = qt.s[i];
    tab.z[i] = qt.z[i];
    tab.zb[i] = qt.zb[i];
  }
  int32_t s;
  if (bits == 3) s = launch_rows_cfg<3, 1>(a, tab, nch, rows, threads, st);
  else if (bits == 4) s = nunit == 1 ? launch_rows_cfg<4, 1>(a, tab, nch, rows, threads, st) : launch_rows_cfg<4, 2>(a, tab, nch, rows, threads, st);
  else s = nunit == 1 ? launch_rows_cfg<8, 1>(a, tab, nch, rows, threads, st) : launch_rows_cfg<8, 2>(a, tab, nch, rows, threads, st);
  // (four wide rows need a raised LDS limit; while a graph is recorded it cannot be raised, and the other kernel serves)
  if (s == RPTQ_ERR_CAPTURE) return RPTQ_OK;
  *served = s == RPTQ_OK;
  return s;
}

}  // namespace rptq
