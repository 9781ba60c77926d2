// Per-channel minimum / maximum of a site's activation over calibration rows
// (Sec. 4.1, first displayed equation).  The activation is LayerNorm(x) computed with the
// same arithmetic as the online kernel (fp64 row sums, fp32 elementwise chain), or x
// itself at a non-LayerNorm site, optionally through max(.,0).
//
// One launch covers all batches.  A workgroup of up to 1024 threads holds several rows at a time, one
// per thread group; each thread owns up to CH chunks of 8 channels of its group's rows and keeps running
// extrema in registers.  The groups of a workgroup merge in LDS, the workgroups through atomic min/max
// on an order-preserving integer image of the floats, so the result does not depend on order.
//
// What bounds it is the global atomics, 2d per workgroup on the same 2d words, against the depth of one
// group's row loop: few rows want few workgroups, many rows the whole chip (the rule and its table are in the launcher).
#include <hip/hip_runtime.h>

#include <cmath>

#include "device_common.h"
#include "rptq_internal.h"

namespace rptq {

constexpr int kCalBatches = 64;           // batches one launch takes (by value)
constexpr int kCalRowsPerGroup = 2;       // rows a thread group walks at least

struct CalBatches {
  int32_t n;
  const uint4* x[kCalBatches];
  int64_t end[kCalBatches];               // first row (counted over all batches) after batch b
};

__global__ void minmax_init_kernel(uint32_t* keys, int d) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < d) {
    keys[i] = 0xffffffffu;        // running minimum (as key)
    keys[d + i] = 0u;             // running maximum (as key)
  }
}

__global__ void minmax_final_kernel(const uint32_t* keys, int d, float* ch_min, float* ch_max) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < d) {
    ch_min[i] = key_float(keys[i]) + 0.0f;        // -0.0 -> +0.0
    ch_max[i] = key_float(keys[d + i]) + 0.0f;
  }
}

// CH: 16-byte chunks of a row per thread.  `tpr` threads (a multiple of the wave size) share a row.
template <bool LN, int CH>
__global__ void __launch_bounds__(1024) minmax_kernel(CalBatches cb, int d, int tpr, const float* gamma, const float* beta,
                                                      float eps, int relu, uint32_t* keys) {
  __shared__ double red[2][2][kMaxWaves];
  extern __shared__ uint32_t sh_keys[];                        // [2][d], several groups only
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wpr = tpr >> 6;                                     // waves per row
  const int grp = wid / wpr, groups = static_cast<int>(blockDim.x) / tpr;
  const int t = tid - grp * tpr;                                // thread of its group
  const int chunks = d / 8;
  const int64_t total = cb.end[cb.n - 1];
  const int64_t stride = static_cast<int64_t>(gridDim.x) * groups;

  if (groups > 1) {
    for (int i = tid; i < d; i += blockDim.x) {
      sh_keys[i] = 0xffffffffu;
      sh_keys[d + i] = 0u;
    }
  }
  float vmin[CH][8], vmax[CH][8];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      vmin[c][k] = __builtin_huge_valf();
      vmax[c][k] = -__builtin_huge_valf();
    }
  }
  int ch_idx[CH];                                               // clamped: a surplus lane reads the last chunk again
  bool ch_ok[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    ch_ok[c] = t + c * tpr < chunks;
    ch_idx[c] = ch_ok[c] ? t + c * tpr : chunks - 1;
  }
  int b = 0;                                                    // batch of the row fetched last (rows only ascend)
  uint4 nxt[CH];
  auto fetch = [&](int64_t row) {
    if (row >= total) row = total - 1;
    while (row >= cb.end[b]) ++b;
    const uint4* p = cb.x[b] + (row - (b ? cb.end[b - 1] : 0)) * chunks;
#pragma unroll
    for (int c = 0; c < CH; ++c) nxt[c] = p[ch_idx[c]];
  };
  // all groups of a workgroup run the same number of passes (they share the barrier of a pass); a group
  // past the end repeats the last row, which changes no extremum
  const int64_t row0 = static_cast<int64_t>(blockIdx.x) * groups;
  constexpr bool kAhead = CH <= 2;                              // (four chunks: a second row does not fit the registers)
  if (kAhead) fetch(row0 + grp);
  int parity = 0;
  for (int64_t base = row0; base < total; base += stride, parity ^= 1) {
    if (!kAhead) fetch(base + grp);
    uint4 v[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) v[c] = nxt[c];
    if (kAhead) fetch(base + stride + grp);
    float mu = 0.0f, rstd = 1.0f;
    if (LN) {
      double s1 = 0.0, s2 = 0.0;
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const uint32_t w[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double lo = ch_ok[c] ? static_cast<double>(bf16_lo(w[k])) : 0.0;
          const double hi = ch_ok[c] ? static_cast<double>(bf16_hi(w[k])) : 0.0;
          s1 += lo;
          s2 = fma(lo, lo, s2);
          s1 += hi;
          s2 = fma(hi, hi, s2);
        }
      }
      const double r1 = wave_sum(s1), r2 = wave_sum(s2);
      if (lane == 0) {
        red[parity][0][wid] = r1;
        red[parity][1][wid] = r2;
      }
      __syncthreads();
      const double t1 = partials_sum(&red[parity][0][grp * wpr], wpr, lane);
      const double t2 = partials_sum(&red[parity][1][grp * wpr], wpr, lane);
      row_stats(t1, t2, d, eps, &mu, &rstd);
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const uint32_t w[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
      float gam[8], bet[8];
      if (LN) {
        // not kept in registers: the extrema need the space
        const float4* gp = reinterpret_cast<const float4*>(gamma + ch_idx[c] * 8);
        const float4* bp = reinterpret_cast<const float4*>(beta + ch_idx[c] * 8);
        const float4 g0 = gp[0], g1 = gp[1], b0 = bp[0], b1 = bp[1];
        gam[0] = g0.x; gam[1] = g0.y; gam[2] = g0.z; gam[3] = g0.w; gam[4] = g1.x; gam[5] = g1.y; gam[6] = g1.z; gam[7] = g1.w;
        bet[0] = b0.x; bet[1] = b0.y; bet[2] = b0.z; bet[3] = b0.w; bet[4] = b1.x; bet[5] = b1.y; bet[6] = b1.z; bet[7] = b1.w;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        float y = (k & 1) ? bf16_hi(w[k / 2]) : bf16_lo(w[k / 2]);
        if (LN) y = ln_chain(y, mu, rstd, gam[k], bet[k]);
        if (relu) y = fmaxf(y, 0.0f);
        vmin[c][k] = fminf(vmin[c][k], y);
        vmax[c][k] = fmaxf(vmax[c][k], y);
      }
    }
  }

  if (groups > 1) {
    __syncthreads();                                            // (a site without LayerNorm has had no barrier since the clearing)
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (ch_ok[c]) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          // (the k-th channels of all chunks side by side: neighbouring lanes update neighbouring words.  In channel order
          // eight lanes shared a bank: 16 batches of 128 x 2048 18.5 | 16.2 us in all)
          atomicMin(&sh_keys[k * chunks + ch_idx[c]], float_key(vmin[c][k]));
          atomicMax(&sh_keys[d + k * chunks + ch_idx[c]], float_key(vmax[c][k]));
        }
      }
    __syncthreads();
    for (int i = tid; i < d; i += blockDim.x) {
      const int at = (i & 7) * chunks + (i >> 3);
      atomicMin(&keys[i], sh_keys[at]);
      atomicMax(&keys[d + i], sh_keys[d + at]);
    }
  } else {
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (ch_ok[c]) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          atomicMin(&keys[ch_idx[c] * 8 + k], float_key(vmin[c][k]));
          atomicMax(&keys[d + ch_idx[c] * 8 + k], float_key(vmax[c][k]));
        }
      }
  }
}

int32_t launch_channel_minmax(const void* const* x_batches, const int64_t* rows, int32_t n_batches, int32_t d,
                              const float* gamma, const float* beta, float eps, int32_t relu,
                              float* ch_min_dev, float* ch_max_dev, uint32_t* keys, hipStream_t st) {
  const int chunks = d / 8;
  // one or two chunks per thread while 1024 threads hold a row so, else four (up to 32768 channels)
  const int ch = chunks <= kWave ? 1 : (chunks <= 2048 ? 2 : 4);
  const int tpr = ((chunks + ch - 1) / ch + kWave - 1) / kWave * kWave;
  if (tpr > 1024) return RPTQ_ERR_SHAPE;
  // (several groups merge in 8 bytes of LDS per channel: as many as stay inside the default 64 KiB)
  const int groups = d <= 8064 ? 1024 / tpr : 1;
  const size_t shmem = groups > 1 ? static_cast<size_t>(d) * 8 : 0;
  hipLaunchKernelGGL(minmax_init_kernel, dim3((d + 255) / 256), dim3(256), 0, st, keys, d);
  RPTQ_HIP(hipGetLastError());
  for (int b = 0; b < n_batches;) {
    CalBatches cb = {};
    int64_t total = 0;
    for (; b < n_batches && cb.n < kCalBatches; ++b) {
      if (rows[b] == 0) continue;
      total += rows[b];
      cb.x[cb.n] = static_cast<const uint4*>(x_batches[b]);
      cb.end[cb.n++] = total;
    }
    if (total == 0) continue;
    const int64_t per_wg = static_cast<int64_t>(groups) * kCalRowsPerGroup;
    // Time of W workgroups: c + a d W + p passes / W (a: a workgroup's 2 d atomic updates at the end, all on the same words;
    // a pass: one row of every group), so W = sqrt(p / a * passes / d), between 64 and one workgroup per compute unit; where a
    // pass costs little (no LayerNorm) and there are more than twenty for every one of two per unit, two.  p / a was taken
    // from this table, us by the largest number of workgroups; * is what the rule takes (or the nearest to it).  Several
    // groups per workgroup:
    //   LayerNorm   d = 2048      64    128    256    512     d = 8000      64    128    192    256    512
    //     2048 rows             21.6  17.3*  17.3   17.3                  59.1   41.4  35.3*   39.5   46.6
    //     8192                  55.3  34.5   26.8*  32.2                 202.2  112.0   83.3  76.0*   84.2
    //   131072                 833.1 427.3  229.4* 229.6                3358.5 1699.5 1143.4 871.0*  881.3
    //   none        d = 5120                                d = 8000
    //     2048                  23.3  19.9*  22.0   26.9                  32.0  27.6*   27.9   32.1   43.8
    //    32768                 238.1 132.1   83.4   75.4*                353.7  194.5  138.8  118.5  113.1*
    // One group (its updates are not in order of address):
    //   LayerNorm   d = 12288     64    128    192    256    512     none     64     128    192    256    512
    //      512 rows            77.2*  121.0  168.1  220.6  221.5            62.4*  107.3  153.9  203.9  203.9
    //     2048                132.1*  148.7  185.3  235.4  377.6            80.6*  117.4  160.2  205.5  368.9
    //     8192                 345.4  254.8 255.8*  289.2  423.4            165.9 156.4*  191.1  233.5  376.6
    //    32768                1356.6  752.3  582.7 514.8*  640.6            576.6  354.6  316.1 334.1*  443.7
    //   131072                5349.7 2718.3 1897.3 1504.6* 1598.9          2197.5 1148.5  843.9 730.6*  761.8
    constexpr int64_t kUnits = 256;                          // compute units
    const double passes = static_cast<double>(total) / groups;
    const double best = std::sqrt((groups > 1 ? 180e3 : 21.5e3) * (gamma ? 2.0 : 1.0) * passes / d);
    const int64_t most = !gamma && best > 2 * kUnits && passes > 20.0 * 2 * kUnits
                             ? 2 * kUnits : std::min<int64_t>(std::max<int64_t>(static_cast<int64_t>(best), 64), kUnits);
    const dim3 grid(static_cast<unsigned>(std::min<int64_t>((total + per_wg - 1) / per_wg, most))), block(tpr * groups);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, shmem, st, cb, d, tpr, gamma, beta, eps, relu, keys); };
    if (gamma) {
      if (ch == 1) go(minmax_kernel<true, 1>);
      else if (ch == 2) go(minmax_kernel<true, 2>);
      else go(minmax_kernel<true, 4>);
    } else {
      if (ch == 1) go(minmax_kernel<false, 1>);
      else if (ch == 2) go(minmax_kernel<false, 2>);
      else go(minmax_kernel<false, 4>);
    }
    RPTQ_HIP(hipGetLastError());
  }
  hipLaunchKernelGGL(minmax_final_kernel, dim3((d + 255) / 256), dim3(256), 0, st, keys, d, ch_min_dev, ch_max_dev);
  RPTQ_HIP(hipGetLastError());
  return RPTQ_OK;
}

}  // namespace rptq
