// Cluster-wise integer product (App. A.4, second method) for products with few output tiles: decoding
// (a few tokens, the weights are streamed once) and short prompts.
//
// The prefill kernel gives a workgroup a 64 x 256 tile and all of K; with 40 to 250 such tiles most of the
// chip is idle and the few waves at work cannot keep enough bytes in flight.  Here the waves of a workgroup
// share one small tile and split K among them: each runs its own pipeline over its range of K steps - its own
// LDS stage, so there is no barrier in the loop - and the fp32 tiles are added in a fixed order at the end.
// A cluster that two waves share is scaled in both (its integer sums are exact, so is their split).
// Operand formats, MFMA use and rescale are those of the prefill kernel.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.h"
#include "gemm_common.h"
#include "rptq_internal.h"

namespace rptq {

constexpr int kSmallPad = 32;              // bytes added to a slice's LDS stride: the staging stores of 8 consecutive lanes
                                           // (two rows x four slices) fall into distinct 16-byte bank groups

// Waves: WGN side by side over the columns x KS over K; a wave's tile is 32 WM tokens x 32 WN channels; a K step
// has S slices of 32 codes.
//
// The loop body is one step, with one register set of weights and one of activations, each refilled with the
// next step's bytes as it is used up, and one LDS stage: a wave that has little to do runs every instruction a
// few times only, so the code's own way through the instruction cache counts.  (The rescale of a finished cluster exists
// once per slice.  Four steps per pass with as many register sets of weights in flight and two LDS stages took 34.8 us
// where this takes 30.3, at 512 x 8192 x 2048, and 17.9 against 15.4 at 32 x 20480 x 5120.)
// Latency is covered by several waves per SIMD instead.  (The second launch bound keeps the accumulators out of the
// AGPRs, where a rescale costs a move per element.)
template <int BITS, int WM, int WN, int WGN, int KS, int S, int OUT>
__global__ void __launch_bounds__(WGN * KS * 64, WM * WN == 1 ? 4 : 2) small_gemm_kernel(GemmArgs a, GemmTab tab) {
  constexpr bool YF32 = OUT == kOutF32;
  constexpr int NT = WGN * KS * 64;
  constexpr int BM = WM * 32;
  constexpr int BN = WGN * WN * 32;
  constexpr int A_SLICE = 2 * BM * 16 + kSmallPad;       // [half][row][16 B]
  constexpr int A_STAGE = S * A_SLICE;
  constexpr int A_PER = BM * S / 64;                     // (row, slice) units per lane and K step
  constexpr int GB = ActFmt<BITS>::kGroupBytes;
  constexpr int A_REGS = GB / 4;
  static_assert(S % 2 == 0 && S <= 8, "slice pairs; steps stay inside the padded width");
  typedef unsigned u4v __attribute__((ext_vector_type(4)));
  typedef unsigned u3v __attribute__((ext_vector_type(3)));
  constexpr int kRsrcFlags = 0x00020000;

  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % WGN, kg = wave / WGN;
  unsigned char* sA = smem + wave * A_STAGE;              // this wave's stage

  // every XCD gets a contiguous range of tiles, the row tiles of one column tile back to back
  const int total = a.tiles_m * a.tiles_n;
  const int xcd = blockIdx.x & 7, q8 = total >> 3, r8 = total & 7;
  const int lin = xcd * q8 + (xcd < r8 ? xcd : r8) + static_cast<int>(blockIdx.x >> 3);
  const int tm = lin % a.tiles_m, tn = lin / a.tiles_m;
  const int64_t m0 = static_cast<int64_t>(tm) * BM;
  const int n0 = tn * BN;

  // ---- this wave's K steps ------------------------------------------------------------------
  const int all_steps = (a.used_slices + S - 1) / S;
  const int step0 = all_steps * kg / KS;
  const int steps = all_steps * (kg + 1) / KS - step0;
  const int last = (steps > 0 ? steps : 1) - 1;           // (an empty range loads a valid step and uses nothing)

  const int64_t rows_here = (a.M - m0) < BM ? (a.M - m0) : BM;
  const int wblocks = a.slices / (kWBlockCols / kGroup);   // packed weight blocks per 32-row band
  const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(a.codes) + m0 * a.row_bytes, 0, static_cast<int>(rows_here) * a.row_bytes, kRsrcFlags);
  const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(a.Wq) + static_cast<size_t>(n0 / 32) * wblocks * 2048, 0, (BN / 32) * wblocks * 2048, kRsrcFlags);
  int a_off[A_PER], a_lds[A_PER], w_off[WN];
#pragma unroll
  for (int i = 0; i < A_PER; ++i) {
    const int unit = lane + i * 64;
    const int row = unit / S, s = unit % S;
    const int lrow = row < rows_here ? row : static_cast<int>(rows_here) - 1;   // clamp: rows past M are never stored
    a_off[i] = lrow * a.row_bytes + s * GB;
    a_lds[i] = s * A_SLICE + row * 16;
  }
#pragma unroll
  for (int j = 0; j < WN; ++j) w_off[j] = (wn * WN + j) * wblocks * 2048 + lane * 16;

  uint32_t ra[A_PER][A_REGS];
  u4v wreg[WN][S / 2];
  auto clamp_step = [&](int t) { return step0 + (t < last ? t : last); };
  auto load_a = [&](int t) {
    const int soff = clamp_step(t) * (S * GB);
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
      if (A_REGS == 3) {
        const u3v r = __builtin_amdgcn_raw_buffer_load_b96(a_rsrc, a_off[i], soff, 0);
#pragma unroll
        for (int k = 0; k < 3; ++k) ra[i][k % A_REGS] = r[k];
      } else {
#pragma unroll
        for (int h = 0; h < A_REGS / 4; ++h) {
          const u4v r = __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, a_off[i] + h * 16, soff, 0);
#pragma unroll
          for (int k = 0; k < 4; ++k) ra[i][(h * 4 + k) % A_REGS] = r[k];
        }
      }
    }
  };
  auto load_w_pair = [&](int t, int j, int p) {             // two slices of column block j
    const int pair = clamp_step(t) * (S / 2) + p;            // (a packed block holds two pairs, 1 KiB each)
    wreg[j][p] = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, w_off[j], pair * 1024, 0);
  };
  auto store_a = [&](int i) {                               // unpack a unit to int8 into LDS
    unsigned char* d = sA + a_lds[i];
    uint4 lo, hi;
    if (BITS == 8) {
      lo = make_uint4(ra[i][0], ra[i][1], ra[i][2], ra[i][3 % A_REGS]);
      hi = make_uint4(ra[i][4 % A_REGS], ra[i][5 % A_REGS], ra[i][6 % A_REGS], ra[i][7 % A_REGS]);
    } else if (BITS == 4) {
      unpack4(make_uint4(ra[i][0], ra[i][1], ra[i][2], ra[i][3 % A_REGS]), &lo, &hi);
    } else {
      unpack3(ra[i][0], ra[i][1], ra[i][2], &lo, &hi);
    }
    *reinterpret_cast<uint4*>(d) = lo;
    *reinterpret_cast<uint4*>(d + BM * 16) = hi;
  };

  v16i acc[WM][WN];
  v16f facc[WM][WN];
  auto clear_tile = [&](int i, int j) {                     // (opaque zeros: see the prefill kernel)
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      unsigned long long zz;
      asm volatile("v_mov_b64 %0, 0" : "=v"(zz));
      acc[i][j][r] = static_cast<int>(zz);
      acc[i][j][r + 1] = static_cast<int>(zz >> 32);
    }
  };
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      clear_tile(i, j);
#pragma unroll
      for (int r = 0; r < 16; ++r) facc[i][j][r] = 0.0f;
    }

  // cluster tables in one register each (lane i: cluster i); this wave starts inside cluster ci
  const float tab_scale = tab.scale[lane];
  const int tab_end = tab.slice_end[lane];
  int ci = __builtin_popcountll(__ballot(lane < tab.g && tab_end <= step0 * S));
  int next_end = __builtin_amdgcn_readlane(tab_end, ci & 63);
  auto rescale = [&]() {
    const float sc = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, tab_scale), ci & 63));
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) {
#pragma unroll
        for (int r = 0; r < 16; ++r) facc[i][j][r] = fmaf(static_cast<float>(acc[i][j][r]), sc, facc[i][j][r]);
        clear_tile(i, j);
      }
  };

  // ---- main loop --------------------------------------------------------------------------------
  load_a(0);
#pragma unroll
  for (int p = 0; p < S / 2; ++p)
#pragma unroll
    for (int j = 0; j < WN; ++j) load_w_pair(0, j, p);
#pragma unroll
  for (int i = 0; i < A_PER; ++i) store_a(i);
  load_a(1);
  __builtin_amdgcn_wave_barrier();                          // (one wave: LDS executes its instructions in order)

  const int a_frag = (lane >> 5) * (BM * 16) + (lane & 31) * 16;
  v4i fa[2][WM], fb[2][WN];
  auto load_frags = [&](int s) {
#pragma unroll
    for (int i = 0; i < WM; ++i) fa[s & 1][i] = *reinterpret_cast<const v4i*>(sA + s * A_SLICE + a_frag + i * 512);
  };
  auto unpack_w = [&](int s) {
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      const u4v w = wreg[j][s >> 1];
      const uint32_t x = (s & 1) ? w.z : w.x, y = (s & 1) ? w.w : w.y;
      fb[s & 1][j][0] = static_cast<int>(x & 0xf0f0f0f0u);
      fb[s & 1][j][1] = static_cast<int>((x << 4) & 0xf0f0f0f0u);
      fb[s & 1][j][2] = static_cast<int>(y & 0xf0f0f0f0u);
      fb[s & 1][j][3] = static_cast<int>((y << 4) & 0xf0f0f0f0u);
    }
  };
  load_frags(0);
  unpack_w(0);
  for (int t = 0; t < steps; ++t) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if (s + 1 < S) {                                      // next slice's operands
        load_frags(s + 1);
        unpack_w(s + 1);
      } else {                                              // every read of this step is issued: the stage takes the next step
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < A_PER; ++i) store_a(i);
        load_a(t + 2);
        __builtin_amdgcn_wave_barrier();
        load_frags(0);
        unpack_w(0);                                        // (pair 0 already holds the next step)
      }
      if ((s & 1) == 0) {                                   // both slices of pair s/2 are expanded
#pragma unroll
        for (int j = 0; j < WN; ++j) load_w_pair(t + 1, j, s >> 1);
      }
#pragma unroll
      for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[s & 1][j], fa[s & 1][i], acc[i][j], 0, 0, 0);
      if ((step0 + t) * S + s + 1 == next_end) {            // cluster ci is complete (uniform branch)
        rescale();
        ++ci;
        next_end = __builtin_amdgcn_readlane(tab_end, ci & 63);
      }
    }
  }
  rescale();                                                // the part of a cluster that another wave goes on with (else zeros)

  // ---- sum over the K ranges, zero-point terms, output scale, store -------------------------------
  // Every wave leaves its fp32 tile in LDS, row-major; a thread then owns a group of columns, adds the K ranges' values in
  // order in fp64 and finishes the prefill kernel's arithmetic there, with one rounding to fp32 at the end (norm of the
  // error against float64 on seven shapes: 4.6e-8 to 6.4e-8; unsplit 5.8e-8 to 9.0e-8; with these sums in fp32 5.9e-8 to
  // 8.8e-8).
  constexpr int TP = BN + 4;
  float* tile = reinterpret_cast<float*>(smem);             // [KS][BM][TP]
  __syncthreads();                                          // every wave is done with its stage
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(tile + (kg * BM + i * 32 + (lane & 31)) * TP + (wn * WN + j) * 32 + q * 8 + (lane >> 5) * 4) =
            make_float4(facc[i][j][q * 4], facc[i][j][q * 4 + 1], facc[i][j][q * 4 + 2], facc[i][j][q * 4 + 3]);
  __syncthreads();
  constexpr int CW = YF32 ? 4 : 8;                          // outputs per 16-byte store
  constexpr int CPR = BN / CW;
  static_assert(NT % CPR == 0, "a thread keeps its columns");
  const int cc = tid % CPR;
  const int n = n0 + cc * CW;
  float sw[CW], ct[CW];
  int zw[CW];
#pragma unroll
  for (int e = 0; e < CW; ++e) {
    const int ne = n + e < a.N ? n + e : a.N - 1;           // (columns past N are never stored)
    sw[e] = a.sW[ne];
    ct[e] = a.colterm[ne];
    zw[e] = a.zW[ne];
  }
  const bool vec_ok = (a.N % 8) == 0 && n + CW <= a.N;
  for (int row = tid / CPR; row < BM; row += NT / CPR) {
    const int64_t t = m0 + row;
    if (t >= a.M || n >= a.N) continue;
    const double rt = a.rowterm[t];
    double sum[CW];
#pragma unroll
    for (int e = 0; e < CW; ++e) sum[e] = 0.0;
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int e4 = 0; e4 < CW / 4; ++e4) {
        const float4 f = *reinterpret_cast<const float4*>(tile + (k * BM + row) * TP + cc * CW + e4 * 4);
        sum[e4 * 4 + 0] += f.x;
        sum[e4 * 4 + 1] += f.y;
        sum[e4 * 4 + 2] += f.z;
        sum[e4 * 4 + 3] += f.w;
      }
    float v[CW];
#pragma unroll
    for (int e = 0; e < CW; ++e)
      v[e] = static_cast<float>(static_cast<double>(sw[e]) * ((sum[e] - ct[e]) - static_cast<double>(zw[e]) * rt));
    store_outputs<YF32>(a, v, t, n, vec_ok);
  }
}

template <int BITS, int WM, int WN, int WGN, int KS, int S, int OUT>
static int32_t launch_small_cfg(const GemmArgs& a, const GemmTab& tab, hipStream_t st) {
  constexpr int BM = WM * 32, BN = WGN * WN * 32;
  constexpr size_t stages = static_cast<size_t>(WGN) * KS * S * (2 * BM * 16 + kSmallPad);
  constexpr size_t tiles = static_cast<size_t>(KS) * BM * (BN + 4) * 4;
  constexpr size_t shmem = stages > tiles ? stages : tiles;
  static_assert(shmem <= 160 * 1024, "LDS of a compute unit");
  auto kern = small_gemm_kernel<BITS, WM, WN, WGN, KS, S, OUT>;
  static LdsGrant lds_granted;
  if (int32_t s = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), shmem, &lds_granted, st)) return s;
  GemmArgs b = a;
  b.tiles_n = (a.N + BN - 1) / BN;
  b.tiles_m = static_cast<int32_t>((a.M + BM - 1) / BM);
  const dim3 grid(static_cast<unsigned>(b.tiles_n) * static_cast<unsigned>(b.tiles_m));
  hipLaunchKernelGGL(kern, grid, dim3(WGN * KS * 64), shmem, st, b, tab);
  RPTQ_HIP(hipGetLastError());
  return RPTQ_OK;
}

// Which split serves a product, by its number of 32 x 32 output tiles (T).  Measured, us: the best tile of the prefill /
// decode kernel first, then 32 x 32 with K in 8, in 4, 32 x 64 with K in 4:
//     1 x  8192 x  2048 (T =  256):  8.6   5.8   6.1   8.4      128 x 3072 x  768 (T =  384):  9.7   5.8   5.1   6.6
//    32 x  5120 x 12288 (T =  160): 28.8  12.1  15.4  19.9       32 x 20480 x 5120 (T =  640): 17.0  18.7  15.4  18.4
//    64 x  2048 x  2048 (T =  128): 16.5   5.7   5.9   8.4       64 x 16000 x 5120 (T = 1000): 22.4        18.7
//   200 x  5120 x  5120 (T = 1120): 22.6  25.7  21.8  21.4      333 x 4099 x 4072 (T = 1419): 23.5  29.0  24.5  21.2
//   512 x  3000 x  2048 (T = 1504): 12.8              13.7      512 x 4096 x 5120 (T = 2048): 24.0              28.2
//    16 x 49152 x 12288 (T = 1536): 55.8  74.5  72.6  61.2  (decode kernel: it streams the weights at the rate of memory)
// A cluster that is split between waves is rounded once per part.  With at least as many clusters as K ranges the sums in
// fp64 more than make up for that (figures above); with fewer, the parts can be larger than their sum: not split.
constexpr int kSmallMinClusters = 8;
enum SmallSplit { kSplitNone, kSplit32x32k8, kSplit32x32k4, kSplit32x64k4 };
static SmallSplit small_split(int64_t M, int32_t N, int32_t g) {
  if (g < kSmallMinClusters) return kSplitNone;
  const int64_t tiles = (M + 31) / 32 * ((N + 31) / 32);
  if (tiles <= 256) return kSplit32x32k8;
  if (tiles <= 1024) return kSplit32x32k4;
  if (tiles <= 1440 && M > 32) return kSplit32x64k4;
  return kSplitNone;
}

bool small_gemm_serves(int64_t M, int32_t N, int32_t g, int out_mode) {
  return (out_mode == kOutBf16 || out_mode == kOutF32) && small_split(M, N, g) != kSplitNone;
}

template <int BITS, int OUT>
static int32_t launch_small_out(const GemmArgs& a, const GemmTab& tab, hipStream_t st) {
  switch (small_split(a.M, a.N, tab.g)) {
    case kSplit32x32k8: return launch_small_cfg<BITS, 1, 1, 1, 8, 4, OUT>(a, tab, st);
    case kSplit32x32k4: return launch_small_cfg<BITS, 1, 1, 1, 4, 4, OUT>(a, tab, st);
    case kSplit32x64k4: return launch_small_cfg<BITS, 1, 2, 1, 4, 4, OUT>(a, tab, st);
    case kSplitNone: break;
  }
  return RPTQ_ERR_SHAPE;
}

int32_t launch_small_gemm(const GemmArgs& a, const GemmTab& tab, int bits, int out_mode, hipStream_t st) {
  const bool f32 = out_mode == kOutF32;
  if (bits == 3) return f32 ? launch_small_out<3, kOutF32>(a, tab, st) : launch_small_out<3, kOutBf16>(a, tab, st);
  if (bits == 4) return f32 ? launch_small_out<4, kOutF32>(a, tab, st) : launch_small_out<4, kOutBf16>(a, tab, st);
  return f32 ? launch_small_out<8, kOutF32>(a, tab, st) : launch_small_out<8, kOutBf16>(a, tab, st);
}

}  // namespace rptq
