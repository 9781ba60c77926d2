// LayerNorm in cluster order + quantization + packing for calls with few rows per compute unit: the arithmetic and the
// results of ln_quant.hip, arranged for latency.
//
// A workgroup takes R rows at once and is done.  The pipelined kernel walks one row per barrier, which hides
// everything behind the row loop when there is one; with one to four rows per workgroup its chain of waits is the time:
// tables, constants, row, partial sums, statistics wave, gather, row sum.  Here all loads (rows, per-position constants,
// one lane-wise read of the cluster tables) are requested at once, the R rows' sums are added up by a wave each while
// the other waves lay out their constants, and the barriers wait for LDS only, not for loads or stores in flight.
//
// Every sum is added in the order of the pipelined kernel (per lane over the waves, then over the lanes), so that a row
// leaves with the same codes and the same row sum, bit for bit, whichever kernel its call runs on.
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "launch_rules.h"
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

// Workgroup barrier that orders LDS accesses only: global loads and stores stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS: R rows, then per row what the waves hand to the wave that adds it up: their lanes' {sum x, sum x^2}; then, in
// their place, {mean, 1/std}, and behind that the lanes' de-quantized row sums.  (Not a byte more: two workgroups with
// four rows of 5120 fill a compute unit's 160 KiB.)
constexpr int kRowsMaxLds = 160 * 1024;
struct RowsLds {
  int chunk_waves;                   // waves that hold input chunks
  int part, part_row;                // byte offset and bytes per row of the parts
  int bytes;
};
template <bool LN>
__host__ __device__ inline RowsLds rows_lds_layout(int d, int threads, int rows) {
  RowsLds l;
  const int nw = threads / kWave, in_chunks = (d / 8 + kWave - 1) / kWave;
  l.chunk_waves = in_chunks < nw ? in_chunks : nw;
  const int stats = LN ? l.chunk_waves * kWave * 16 : 0, row_sums = (nw + (LN ? 1 : 0)) * kWave * 8;
  l.part = rows * d * 2;
  l.part_row = stats > row_sums ? stats : row_sums;
  l.bytes = l.part + rows * l.part_row;
  return l;
}

template <int BITS, int NUNIT, int NCH, int R, bool LN>
__global__ void __launch_bounds__(1024) ln_rows_kernel(LnQuantArgs a, LnRowsTab tab) {
  constexpr int UC = Unit<BITS>::kCodes;
  constexpr int ND = UC / 4;
  constexpr float kUMax = static_cast<float>((1 << BITS) - 1);
  constexpr int kQMin = -(1 << (BITS - 1));

  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6), nw = static_cast<int>(blockDim.x) >> 6;
  const int TU = static_cast<int>(blockDim.x);
  const RowsLds lds = rows_lds_layout<LN>(a.d, TU, R);
  const int nwc = lds.chunk_waves;
  // this lane's parts of row r, wave by wave
  auto stats_parts = [&](int r) { return reinterpret_cast<double2*>(smem + lds.part + r * lds.part_row) + lane; };
  auto sum_parts = [&](int r) { return reinterpret_cast<double*>(smem + lds.part + r * lds.part_row) + (LN ? kWave : 0) + lane; };
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

  // ---- rows to LDS, fp64 sums ---------------------------------------------------------------------------
#pragma unroll
  for (int r = 0; r < R; ++r) {
    double s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int idx = tid + c * TU;
      const bool ok = idx < a.chunks;
      if (ok) *reinterpret_cast<u4v*>(smem + r * a.d * 2 + idx * 16) = x[r][c];
      if (LN) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t w = ok ? x[r][c][k] : 0u;
          const double lo = static_cast<double>(bf16_lo(w)), hi = static_cast<double>(bf16_hi(w));
          s1 += lo;
          s2 = fma(lo, lo, s2);
          s1 += hi;
          s2 = fma(hi, hi, s2);
        }
      }
    }
    if (LN && wid < nwc) stats_parts(r)[wid * kWave] = make_double2(s1, s2);
  }
  if (LN) {
    lds_barrier();                                             // rows and parts are in LDS
    if (wid < R) {                                             // wave r adds row r up; there are at least R
      __builtin_amdgcn_s_setprio(3);                           // (the other waves wait for it at the next barrier)
      double2* part = stats_parts(wid);
      double t1 = 0.0, t2 = 0.0;
      for (int j = 0; j < nwc; j += 4) {                       // four reads in flight; surplus ones re-read wave 0
        double2 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = part[(j + k < nwc ? j + k : 0) * kWave];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          t1 += j + k < nwc ? v[k].x : 0.0;
          t2 += j + k < nwc ? v[k].y : 0.0;
        }
      }
      float mu, rstd;
      row_stats(wave_sum(t1), wave_sum(t2), a.d, a.eps, &mu, &rstd);
      if (lane == 0) *reinterpret_cast<float2*>(part) = make_float2(mu, rstd);
      __builtin_amdgcn_s_setprio(0);
    }
  }

  // ---- constants of this thread's units (while the rows are added up) -------------------------------------------
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

  lds_barrier();                                               // {mean, 1/std} (without LayerNorm: the rows) are in LDS

  // ---- gather in cluster order, normalize, quantize, pack ----------------------------------------------
  double rt[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    rt[r] = 0.0;
    const bool row_ok = row0 + r < a.M;
    float mu_r = 0.0f, rstd_r = 1.0f;
    if (LN) {
      const float2 ms = *reinterpret_cast<const float2*>(smem + lds.part + r * lds.part_row);
      mu_r = ms.x;
      rstd_r = ms.y;
    }
    const unsigned char* rowbuf = smem + r * a.d * 2;
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
  for (int r = 0; r < R; ++r) sum_parts(r)[wid * kWave] = rt[r];
  lds_barrier();
  if (wid < R) {
    const double* part = sum_parts(wid);
    double t3 = 0.0;
    for (int j = 0; j < nw; j += 4) {
      double v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = part[(j + k < nw ? j + k : 0) * kWave];
#pragma unroll
      for (int k = 0; k < 4; ++k) t3 += j + k < nw ? v[k] : 0.0;
    }
    const double total = wave_sum(t3);
    if (lane == 0 && row0 + wid < a.M) a.rowterm[row0 + wid] = static_cast<float>(total);
  }
}

template <int BITS, int NUNIT, int NCH, int R, bool LN>
static int32_t raise_rows_limit(int d, int threads, hipStream_t st) {
  static LdsGrant lds_granted;
  return ensure_dynamic_lds(reinterpret_cast<const void*>(ln_rows_kernel<BITS, NUNIT, NCH, R, LN>),
                            rows_lds_layout<LN>(d, threads, R).bytes, &lds_granted, st);
}

template <int BITS, int NUNIT, int NCH, int R, bool LN>
static int32_t launch_rows_kernel(const LnQuantArgs& a, const LnRowsTab& tab, int threads, hipStream_t st) {
  if (int32_t s = raise_rows_limit<BITS, NUNIT, NCH, R, LN>(a.d, threads, st)) return s;
  hipLaunchKernelGGL((ln_rows_kernel<BITS, NUNIT, NCH, R, LN>), dim3(static_cast<unsigned>((a.M + R - 1) / R)), dim3(threads),
                     rows_lds_layout<LN>(a.d, threads, R).bytes, st, a, tab);
  RPTQ_HIP(hipGetLastError());
  return RPTQ_OK;
}

template <int BITS, int NUNIT, int NCH, bool LN>
static int32_t launch_rows_count(const LnQuantArgs& a, const LnRowsTab& tab, int rows, int threads, hipStream_t st) {
  // (four of the widest rows do not fit)
  if (rows == 4 && rows_lds_layout<LN>(a.d, threads, 4).bytes > kRowsMaxLds) rows = 2;
  if (rows < 4 && rows_lds_layout<LN>(a.d, threads, 4).bytes <= kRowsMaxLds) {
    // (a call of few rows stands for a recorded call of more: their limits are raised with it)
    const int32_t s = raise_rows_limit<BITS, NUNIT, NCH, 4, LN>(a.d, threads, st);
    if (s && s != RPTQ_ERR_CAPTURE) return s;
  }
  if (rows < 2) {
    const int32_t s = raise_rows_limit<BITS, NUNIT, NCH, 2, LN>(a.d, threads, st);
    if (s && s != RPTQ_ERR_CAPTURE) return s;
  }
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

// Which calls come here.  With many rows per compute unit the pipelined kernel catches up, the sooner the wider the row and the
// fewer waves hold it (a row's parts take 16 bytes of LDS per thread, so fewer rows are resident; at 3 bits a row has half the
// waves).  us in a recorded graph, pipelined | this kernel, 4 bits (or as stated):
//                       LayerNorm       without                            LayerNorm       without
//     1 x  2048          4.4 |  2.9     3.0 |  2.2      2048 x  768        6.1 |  4.5     4.3 |  3.3
//   128 x   768 (8)      3.8 |  3.0     2.8 |  2.5      2048 x  768 (3)    6.7 |  5.5     4.1 |  3.8
//    32 x  5120          6.3 |  4.0     4.5 |  3.2      8192 x  768       11.2 |  9.2     7.2 |  6.2
//    16 x 12288          9.1 |  6.1     7.6 |  4.5     16384 x 2048       33.0 | 30.0    19.1 | 19.0
//   333 x  4072 (3)      8.0 |  5.9     5.4 |  4.5      8192 x 4072       32.8 | 32.2    22.1 | 19.2
//   512 x  5120          8.6 |  5.4     6.6 |  3.9      2048 x 5120       14.0 | 10.4     9.9 |  7.3
//  1024 x  5120 (3)     10.8 |  8.3     7.5 |  6.0      4096 x 5120       21.1 | 19.2    14.5 | 14.5
//  1024 x  8192 (8)     13.3 | 11.1    13.8 |  8.5      1024 x 12288 (3)  16.5 | 13.1    11.1 |  9.3
//   and not (back to back):    8192 x  768 (3) 11.4 | 11.8    32768 x 1024  33.9 | 36.2    16384 x 2048 (3) 33.9 | 35.4
//                              4096 x 4072 (3) 21.9 | 25.8     6144 x 4072 (8) 27.0 | 29.3     4096 x 5120 (3) 24.1 | 29.2
// Narrow rows from memory, 4 bits, 8 clusters:
//                   LayerNorm                                        without
//             8192       16384       32768               8192        16384       32768       65536
//     256  10.5 |  8.2  14.7 | 13.7  23.4 | 24.1       6.4 |  6.1   8.4 |  9.4  12.4 | 16.4  20.3 | 28.6
//     768  13.0 | 10.6  20.7 | 19.1  33.2 | 32.5       8.3 |  7.5  12.9 | 12.4  19.4 | 21.5  35.0 | 38.1
//    1536  16.9 | 15.2  25.2 | 25.4  42.0 | 45.3      11.4 | 10.6  16.9 | 17.2  27.7 | 30.2  51.2 | 54.4
//    2048  20.0 | 17.8  31.9 | 31.1  55.8 | 55.6      14.3 | 12.5  23.1 | 19.7  41.3 | 33.5  78.7 | 62.6
int32_t launch_ln_rows(const LnQuantArgs& a, const ClusterGeom& geom, const QuantTab& qt, int bits, int nunit, int nch,
                       int threads, int cus, hipStream_t st, bool* served) {
  *served = false;
  if (nch > 2 || nunit > 2 || (bits == 3 && nunit > 1)) return RPTQ_OK;
  const bool ln = a.gamma_pad != nullptr;
  int most;                                                  // rows per compute unit
  if (bits == 3) most = a.d <= 3072 ? 16 : (a.d <= 5120 ? 8 : 4);
  else if (a.d <= 2048) most = ln ? 64 : (a.d <= 640 ? 32 : (a.d <= 1792 ? 64 : 128));
  else most = a.d <= (bits == 4 ? 4096 : 3072) ? 32 : (a.d <= 5120 ? 16 : 4);
  if (a.M > static_cast<int64_t>(cus) * most) return RPTQ_OK;
  const int rows = ln_rows_per_workgroup(a.M, threads / kWave, nunit, cus, bits, ln);
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
  // (several wide rows need a raised LDS limit; while a graph is recorded it cannot be raised, and the other kernel serves)
  if (s == RPTQ_ERR_CAPTURE) return RPTQ_OK;
  *served = s == RPTQ_OK;
  return s;
}

}  // namespace rptq
