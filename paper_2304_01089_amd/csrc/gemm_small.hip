// Cluster-wise integer product (App. A.4, second method) for products with few output tiles: decoding
// (a few tokens, the weights are streamed once) and short prompts.
//
// The prefill kernel gives a workgroup a 64 x 256 tile and all of K; with 40 to 250 such tiles most of the
// chip is idle and the few waves at work cannot keep enough bytes in flight.  Here the waves of a workgroup
// share one 32 x 32 tile and split K among them, each with its own pipeline and LDS stage.
//
// The result is the prefill kernel's, bit for bit: a token's outputs do not depend on how many rows or columns share
// its call.  What the waves hand over is therefore integers: where a cluster, or a wave's share of K, ends, the wave
// leaves its int32 tile in LDS (a piece).  The fp32 chain over the clusters - add a cluster's pieces (exact), convert,
// times sX_i, add, in cluster order - is run by the workgroup's threads, each on its own outputs.  A piece is 4 KiB (2 KiB
// up to 16 tokens), so K is walked in periods of as many clusters as LDS holds pieces of: the period's K steps are shared
// out, a barrier, its pieces enter the chain, a barrier.
// Operand formats, MFMA use and output arithmetic are those of the prefill kernel.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "gemm_common.h"
#include "rptq_internal.h"

namespace rptq {

// 16 bytes of 4-bit codes (32 codes) -> 32 int8 values (code << 4), natural order.
__device__ __forceinline__ void unpack4(const uint4 p, uint4* lo, uint4* hi) {
  lo->x = p.x & 0xf0f0f0f0u;
  lo->y = (p.x << 4) & 0xf0f0f0f0u;
  lo->z = p.y & 0xf0f0f0f0u;
  lo->w = (p.y << 4) & 0xf0f0f0f0u;
  hi->x = p.z & 0xf0f0f0f0u;
  hi->y = (p.z << 4) & 0xf0f0f0f0u;
  hi->z = p.w & 0xf0f0f0f0u;
  hi->w = (p.w << 4) & 0xf0f0f0f0u;
}

// 12 bytes of 3-bit codes (32 codes) -> 32 int8 values (code << 5), natural order.
__device__ __forceinline__ void unpack3(uint32_t x0, uint32_t x1, uint32_t x2, uint4* lo, uint4* hi) {
  lo->x = x0 & 0xe0e0e0e0u;
  lo->y = (x0 << 3) & 0xe0e0e0e0u;
  lo->z = x1 & 0xe0e0e0e0u;
  lo->w = (x1 << 3) & 0xe0e0e0e0u;
  hi->x = x2 & 0xe0e0e0e0u;
  hi->y = (x2 << 3) & 0xe0e0e0e0u;
  hi->z = ((x0 << 6) & 0xc0c0c0c0u) | ((x2 << 5) & 0x20202020u);
  hi->w = ((x1 << 6) & 0xc0c0c0c0u) | ((x2 << 4) & 0x20202020u);
}

constexpr int kSmallTile = 32;             // output rows and columns of a workgroup
constexpr int kSmallSlices = 4;            // slices (of 32 codes) per K step
constexpr int kSmallPad = 32;              // bytes added to a slice's LDS stride: the staging stores of 8 consecutive lanes
                                           // (two rows x four slices) fall into distinct 16-byte bank groups
constexpr int kSmallSlicePitch = 2 * kSmallTile * 16 + kSmallPad;    // [half][row][16 B]
constexpr int kSmallStage = kSmallSlices * kSmallSlicePitch;         // one wave's activations of a K step
constexpr int kMaxPeriods = 16;
constexpr int kMaxPieces = 60;             // of one period (a lane each)

// How the workgroups walk K (by value).
struct SmallPlan {
  int32_t periods;
  int32_t end[kMaxPeriods];                // first K step after period p
};

// The loop body is one step, with one register set of weights and one of activations, each refilled with the next
// step's bytes as it is used up, and one LDS stage: a wave that has little to do runs every instruction a few times
// only, so the code's own way through the instruction cache counts.  Latency is covered by several waves per SIMD.
// (The second launch bound keeps the accumulators out of the AGPRs, where reading one costs a move.)
template <int BITS, int KS, int ROWS, int OUT>
__global__ void __launch_bounds__(KS * 64, 4) small_gemm_kernel(GemmArgs a, GemmTab tab, SmallPlan plan) {
  constexpr bool YF32 = OUT == kOutF32;
  constexpr int NT = KS * 64;
  constexpr int S = kSmallSlices, BM = kSmallTile, BN = kSmallTile;
  constexpr int A_SLICE = kSmallSlicePitch;
  constexpr int A_PER = BM * S / 64;                     // (row, slice) units per lane and K step
  constexpr int GB = ActFmt<BITS>::kGroupBytes;
  constexpr int A_REGS = GB / 4;
  constexpr int PIECE = ROWS * BN * 4;                   // bytes; ROWS: tokens that a piece holds (M or more, or 32)
  constexpr int E = BM * BN / NT;                        // outputs of a thread in the chain over the clusters
  static_assert(S % 2 == 0 && S <= 8, "slice pairs; steps stay inside the padded width");
  static_assert(E == 2 || E == 4, "a thread's outputs lie in one register quad");
  typedef unsigned u4v __attribute__((ext_vector_type(4)));
  typedef unsigned u3v __attribute__((ext_vector_type(3)));
  constexpr int kRsrcFlags = 0x00020000;

  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int kg = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned char* sA = smem + kg * kSmallStage;            // this wave's stage
  unsigned char* pieces = smem + KS * kSmallStage;        // [piece][register quad][half][token][16 B]

  // every XCD gets a contiguous range of tiles, the row tiles of one column tile back to back
  const int total = a.tiles_m * a.tiles_n;
  const int xcd = blockIdx.x & 7, q8 = total >> 3, r8 = total & 7;
  const int lin = xcd * q8 + (xcd < r8 ? xcd : r8) + static_cast<int>(blockIdx.x >> 3);
  const int tm = lin % a.tiles_m, tn = lin / a.tiles_m;
  const int64_t m0 = static_cast<int64_t>(tm) * BM;
  const int n0 = tn * BN;

  const int64_t rows_here = (a.M - m0) < BM ? (a.M - m0) : BM;
  const int wblocks = a.slices / (kWBlockCols / kGroup);   // packed weight blocks per 32-row band
  const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(a.codes) + m0 * a.row_bytes, 0, static_cast<int>(rows_here) * a.row_bytes, kRsrcFlags);
  const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(a.Wq) + static_cast<size_t>(tn) * wblocks * 2048, 0, wblocks * 2048, kRsrcFlags);
  int a_off[A_PER], a_lds[A_PER];
#pragma unroll
  for (int i = 0; i < A_PER; ++i) {
    const int unit = lane + i * 64;
    const int row = unit / S, s = unit % S;
    const int lrow = row < rows_here ? row : static_cast<int>(rows_here) - 1;   // clamp: rows past M are never stored
    a_off[i] = lrow * a.row_bytes + s * GB;
    a_lds[i] = s * A_SLICE + row * 16;
  }

  // ---- this thread's E outputs: tokens vary fastest, then register quads (four columns) ----------
  typedef float fE __attribute__((ext_vector_type(E)));
  constexpr int kOutThreads = PIECE / (4 * E);
  const int my_out = tid % kOutThreads;                     // (surplus threads go along and store nothing)
  const int o_tok = my_out * E / 4 % ROWS, o_n = n0 + my_out * E / 4 / ROWS * 4 + my_out * E % 4;
  float p_sw[E], p_ct[E], p_zw[E];
  const float p_rt = a.rowterm[m0 + (o_tok < rows_here ? o_tok : 0)];
#pragma unroll
  for (int e = 0; e < E; ++e) {                             // (requested here: used at the very end)
    const int ne = min(o_n + e, a.N - 1);
    p_sw[e] = a.sW[ne];
    p_ct[e] = a.colterm[ne];
    p_zw[e] = static_cast<float>(a.zW[ne]);
  }

  // ---- this wave's K steps: its share of every period ----------------------------------------
  const int all_steps = (a.used_slices + S - 1) / S;
  const int tab_period = plan.end[lane % kMaxPeriods];      // lane p: end of period p
  struct Cursor { int p, t, e; };                           // period, step, end of the wave's share of that period
  auto period_begin = [&](int p) { return p ? __builtin_amdgcn_readlane(tab_period, p - 1) : 0; };
  // where wave w's share of n steps from b begins (of fewer steps than waves, the first waves get one each)
  auto share_begin = [&](int b, int n, int w) { return b + (n < KS ? min(w, n) : static_cast<int>(static_cast<unsigned>(n * w) / KS)); };
  auto settle = [&](Cursor& c) {                            // on to the next period that has a step for this wave
    while (c.t >= c.e && c.p + 1 < plan.periods) {
      ++c.p;
      const int b = period_begin(c.p), n = __builtin_amdgcn_readlane(tab_period, c.p) - b;
      c.t = share_begin(b, n, kg);
      c.e = share_begin(b, n, kg + 1);
    }
  };

  uint32_t ra[A_PER][A_REGS];
  u4v wreg[S / 2];
  // (behind a wave's last step a valid step is loaded again and never used)
  auto load_a = [&](const Cursor& c) {
    const int soff = min(c.t, all_steps - 1) * (S * GB);
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
  auto load_w_pair = [&](const Cursor& c, int p) {          // two slices (a packed block holds two pairs, 1 KiB each)
    wreg[p] = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, lane * 16, (min(c.t, all_steps - 1) * (S / 2) + p) * 1024, 0);
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

  v16i acc;                                                 // 2^shift * this wave's part of P_i
  auto clear_acc = [&]() {                                  // (opaque zeros: see the prefill kernel)
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      unsigned long long zz;
      asm volatile("v_mov_b64 %0, 0" : "=v"(zz));
      acc[r] = static_cast<int>(zz);
      acc[r + 1] = static_cast<int>(zz >> 32);
    }
  };
  clear_acc();

  // cluster tables in one register each (lane i: cluster i)
  const float tab_scale = tab.scale[lane];
  const int tab_end = tab.slice_end[lane];
  auto finished_before = [&](int slice) { return __builtin_popcountll(__ballot(lane < tab.g && tab_end <= slice)); };
  // Leaves this wave's part of a cluster in a piece.  A wave leaves one where a cluster ends and one where its share ends
  // (empty if a cluster ends there too), so that pieces numbered cluster (from the period's first) plus wave
  // follow each other along K without a gap.
  const bool tok_ok = (lane & 31) < ROWS;
  unsigned char* my_quads = pieces + (lane >> 5) * (ROWS * 16) + (lane & 31) * 16;
  auto leave = [&](int piece) {
    if (tok_ok) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<int4*>(my_quads + piece * PIECE + q * (ROWS * 32)) =
            make_int4(acc[q * 4], acc[q * 4 + 1], acc[q * 4 + 2], acc[q * 4 + 3]);
    }
    clear_acc();
  };

  // ---- the chain over the clusters: E neighbouring outputs per thread ---------------------------
  typedef int iE __attribute__((ext_vector_type(E)));
  const iE* my_ints = reinterpret_cast<const iE*>(pieces) + my_out;
  float f[E];
  int v[E];                                                 // the integers of the cluster under way
#pragma unroll
  for (int e = 0; e < E; ++e) {
    f[e] = 0.0f;
    v[e] = 0;
  }
  // `end_scale`, lane j: sX of the cluster that piece j ends, else 0 (f + v * 0 is f: f is never -0); `go_on`, lane j:
  // all ones where the cluster goes on in piece j + 1
  auto chain = [&](int count, int end_scale, int go_on) {
    int j = 0;
    auto some = [&](auto together) {
      constexpr int U = decltype(together)::value;
      iE x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = my_ints[(j + u) * kOutThreads];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float sc = __builtin_bit_cast(float, __builtin_amdgcn_readlane(end_scale, j + u));
        const int keep = __builtin_amdgcn_readlane(go_on, j + u);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          v[e] += x[u][e];
          f[e] = fmaf(static_cast<float>(v[e]), sc, f[e]);
          v[e] &= keep;
        }
      }
      j += U;
    };
    while (j + 4 <= count) some(std::integral_constant<int, 4>());
    while (j < count) some(std::integral_constant<int, 1>());
  };

  // ---- main loop --------------------------------------------------------------------------------
  Cursor nxt = {-1, 0, 0};                                  // the step whose operands are requested next
  settle(nxt);
  load_a(nxt);
#pragma unroll
  for (int p = 0; p < S / 2; ++p) load_w_pair(nxt, p);
#pragma unroll
  for (int i = 0; i < A_PER; ++i) store_a(i);
  ++nxt.t;
  settle(nxt);
  load_a(nxt);
  wave_lds_fence();

  const int a_frag = (lane >> 5) * (BM * 16) + (lane & 31) * 16;
  v4i fa[2], fb[2];
  auto load_frags = [&](int s) { fa[s & 1] = *reinterpret_cast<const v4i*>(sA + s * A_SLICE + a_frag); };
  auto unpack_w = [&](int s) {
    const u4v w = wreg[s >> 1];
    const uint32_t x = (s & 1) ? w.z : w.x, y = (s & 1) ? w.w : w.y;
    fb[s & 1][0] = static_cast<int>(x & 0xf0f0f0f0u);
    fb[s & 1][1] = static_cast<int>((x << 4) & 0xf0f0f0f0u);
    fb[s & 1][2] = static_cast<int>(y & 0xf0f0f0f0u);
    fb[s & 1][3] = static_cast<int>((y << 4) & 0xf0f0f0f0u);
  };
  load_frags(0);
  unpack_w(0);
  for (int p = 0; p < plan.periods; ++p) {
    const int b = period_begin(p), end = __builtin_amdgcn_readlane(tab_period, p);
    const Cursor mine = {p, share_begin(b, end - b, kg), share_begin(b, end - b, kg + 1)};
    const int first = finished_before(b * S);
    int ci = finished_before(mine.t * S);                   // the cluster this share starts in
    int next_end = __builtin_amdgcn_readlane(tab_end, ci & 63);
    for (int t = mine.t; t < mine.e; ++t) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        if (s + 1 < S) {                                    // next slice's operands
          load_frags(s + 1);
          unpack_w(s + 1);
        } else {                                            // every read of this step is issued: the stage takes the next step
          wave_lds_fence();
#pragma unroll
          for (int i = 0; i < A_PER; ++i) store_a(i);
          ++nxt.t;
          settle(nxt);
          load_a(nxt);
          wave_lds_fence();
          load_frags(0);
          unpack_w(0);                                      // (pair 0 already holds the next step)
        }
        if ((s & 1) == 0) load_w_pair(nxt, s >> 1);          // both slices of pair s/2 are expanded
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[s & 1], fa[s & 1], acc, 0, 0, 0);
        if (t * S + s + 1 == next_end) {                    // cluster ci ends here (uniform branch)
          leave(ci - first + kg);
          ++ci;
          next_end = __builtin_amdgcn_readlane(tab_end, ci & 63);
        }
      }
    }
    if (mine.t < mine.e && ci < tab.g) leave(ci - first + kg);
    __syncthreads();
    const bool last = p + 1 == plan.periods;
    const int until = finished_before(end * S);             // clusters first .. until - 1 end in this period
    int piece = lane - first;                               // lane i: the piece in which cluster i ends
#pragma unroll
    for (int w = 1; w < KS; ++w) piece += share_begin(b, end - b, w) * S < tab_end ? 1 : 0;
    const int to = (lane >= first && lane < until ? piece : 63) * 4;
    const int end_scale = __builtin_amdgcn_ds_permute(to, __builtin_bit_cast(int, tab_scale));
    const int go_on = __builtin_amdgcn_ds_permute(to, 1) - 1;
    // (the last wave of the last period leaves no piece behind the last cluster)
    // With up to 16 tokens half of eight waves have no outputs: they leave the issue slots to the others (16 x 5120 x 5120
    // 9.36 -> 9.13 us, 16 x 4096 x 12288 12.7 -> 12.2; of four waves, two, it is no gain).
    if (KS < 8 || kg * 64 < kOutThreads) chain(until - first + min(end - b, KS) - (last ? 1 : 0), end_scale, go_on);
    if (!last) __syncthreads();                             // the pieces have been read
  }

  // ---- zero-point terms, output scale, store: the prefill kernel's arithmetic ------------------------
  const int64_t t = m0 + o_tok;
  if (tid >= kOutThreads || t >= a.M) return;
  float y[E];
#pragma unroll
  for (int e = 0; e < E; ++e) y[e] = p_sw[e] * ((f[e] - p_ct[e]) - p_zw[e] * p_rt);
  const bool vec_ok = (a.N % E) == 0 && o_n < a.N;
  if (YF32) {
    float* dst = static_cast<float*>(a.y) + t * a.N + o_n;
    if (vec_ok) {
      fE o;
#pragma unroll
      for (int e = 0; e < E; ++e) o[e] = y[e];
      *reinterpret_cast<fE*>(dst) = o;
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (o_n + e < a.N) dst[e] = y[e];
    }
  } else {
    typedef __bf16 bE __attribute__((ext_vector_type(E)));
    fE o;
#pragma unroll
    for (int e = 0; e < E; ++e) o[e] = y[e];
    const bE h = __builtin_convertvector(o, bE);            // round to nearest even
    __bf16* dst = static_cast<__bf16*>(a.y) + t * a.N + o_n;
    if (vec_ok) {
      *reinterpret_cast<bE*>(dst) = h;
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (o_n + e < a.N) dst[e] = h[e];
    }
  }
}

// Divides K into periods (one if LDS holds all pieces).  A period that n clusters reach into leaves up to n + ks pieces;
// it ends on a multiple of ks steps where it is long enough, so that the shares are equal.  False: too many periods.
static bool make_small_plan(const GemmArgs& a, const GemmTab& tab, int ks, int piece_bytes, int lds_bytes, SmallPlan* plan,
                            int* used) {
  const int all_steps = (a.used_slices + kSmallSlices - 1) / kSmallSlices;
  const int stages = ks * kSmallStage;
  const int most = std::min((lds_bytes - stages) / piece_bytes, kMaxPieces) - ks;
  if (most < kSmallSlices) return false;                    // (a step touches up to four clusters)
  plan->periods = 0;
  int b = 0, first = 0;                                      // first step of the period; the cluster it starts in
  while (b < all_steps) {
    if (plan->periods == kMaxPeriods) return false;
    int e = all_steps;
    if (tab.g - first > most) {
      e = tab.slice_end[first + most - 1] / kSmallSlices;    // (the step that goes past it touches one more)
      if (e - b > ks) e = b + (e - b) / ks * ks;
    }
    plan->end[plan->periods++] = b = e;
    while (first < tab.g && tab.slice_end[first] <= b * kSmallSlices) ++first;
  }
  for (int p = plan->periods; p < kMaxPeriods; ++p) plan->end[p] = all_steps;
  *used = stages + piece_bytes * (std::min(most, tab.g) + ks);
  return true;
}

template <int BITS, int KS, int ROWS, int OUT>
static int32_t launch_small_cfg(const GemmArgs& a, const GemmTab& tab, int lds_bytes, hipStream_t st, bool* served) {
  SmallPlan plan;
  int shmem = 0;
  if (!make_small_plan(a, tab, KS, ROWS * kSmallTile * 4, lds_bytes, &plan, &shmem)) return RPTQ_OK;
  auto kern = small_gemm_kernel<BITS, KS, ROWS, OUT>;
  static LdsGrant lds_granted;
  if (shmem > 64 * 1024) {
    // (the limit is raised to the largest size at once; while a graph is recorded it cannot be, and the other kernels
    // give the same result)
    const int32_t s = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds_bytes, &lds_granted, st);
    if (s == RPTQ_ERR_CAPTURE) return RPTQ_OK;
    if (s) return s;
  }
  GemmArgs b = a;
  b.tiles_n = (a.N + kSmallTile - 1) / kSmallTile;
  b.tiles_m = static_cast<int32_t>((a.M + kSmallTile - 1) / kSmallTile);
  const dim3 grid(static_cast<unsigned>(b.tiles_n) * static_cast<unsigned>(b.tiles_m));
  *served = true;
  hipLaunchKernelGGL(kern, grid, dim3(KS * 64), shmem, st, b, tab, plan);
  RPTQ_HIP(hipGetLastError());
  return RPTQ_OK;
}

// Which calls are split, by the number of 32 x 32 output tiles (T).  us, unsplit | K in 8 | K in 4; g clusters:
//                                g = 8                 g = 16                g = 32
//     1 x  8192 x  2048 (T 256)   7.4 |  5.9 |  6.1     8.6 |  6.6 |  6.9    10.4 |  7.9 |  9.3
//    32 x  5120 x  5120 (T 160)  12.8 |  7.5 |  8.2    14.2 |  8.3 |  9.4    16.0 | 10.5 | 12.8
//    32 x  5120 x 20480 (T 160)  40.2 | 15.5 | 20.6    41.4 | 16.0 | 22.0    43.2 | 18.6 | 25.2
//   256 x  1024 x  1024 (T 256)   7.2 |  5.8 |  5.5     9.1 |  6.4 |  6.7    12.1 |  8.8 | 10.1
//    32 x 12288 x  2048 (T 384)   7.7 | 10.8 |  7.1     9.0 | 12.1 |  9.0    10.7 | 16.4 | 13.4
//   128 x  3072 x   768 (T 384)   6.9 |  8.7 |  5.8     8.6 | 10.8 |  8.9    12.2 | 15.3 | 12.1
//    64 x  5120 x  5120 (T 320)  16.4 | 13.4 |  9.7    18.3 | 15.2 | 11.4    21.2 | 19.6 | 16.1
//    16 x 16384 x 12288 (T 512)  26.8 | 19.2 | 19.1    28.0 | 23.7 | 19.6    29.8 | 26.9 | 23.2
//    64 x 12288 x  8192 (T 768)  23.9 |      | 22.2    25.9 |      | 25.1    28.8 |      | 34.6
//    64 x 16000 x  5120 (T 1000) 17.3 |      | 19.2    19.3 |      | 22.7    22.3 |      | 30.9
// Eight ranges fill the chip with one workgroup per compute unit (T up to 256), four with two.  What a split costs is the
// chain, by the cluster; beyond 256 tiles, where less is gained, it pays from 2.5 slices per cluster on average, against
// the weight-streaming kernel (up to 32 rows) from four (2.5 at 32 x 12288 x 2048 and 64 x 8192 x 2048, 32 clusters:
// 10.7 | 13.4 and 14.8 | 13.6; 2 at 128 x 3072 x 768, 16 clusters; 4.5 at 32 x 12288 x 2048, 16 clusters).
template <int BITS, int OUT>
static int32_t launch_small_out(const GemmArgs& a, const GemmTab& tab, hipStream_t st, bool* served) {
  const int64_t tiles = (a.M + kSmallTile - 1) / kSmallTile * ((a.N + kSmallTile - 1) / kSmallTile);
  if (tiles <= 256)
    return a.M <= 16 ? launch_small_cfg<BITS, 8, 16, OUT>(a, tab, 160 * 1024, st, served)
                     : launch_small_cfg<BITS, 8, 32, OUT>(a, tab, 160 * 1024, st, served);
  if (tiles <= 512 && 2 * a.used_slices >= (a.M > 32 ? 5 : 8) * tab.g)
    return a.M <= 16 ? launch_small_cfg<BITS, 4, 16, OUT>(a, tab, 80 * 1024, st, served)
                     : launch_small_cfg<BITS, 4, 32, OUT>(a, tab, 80 * 1024, st, served);
  return RPTQ_OK;
}

int32_t launch_small_gemm(const GemmArgs& a, const GemmTab& tab, int bits, int out_mode, hipStream_t st, bool* served) {
  *served = false;
  const bool f32 = out_mode == kOutF32;
  if (bits == 3) return f32 ? launch_small_out<3, kOutF32>(a, tab, st, served) : launch_small_out<3, kOutBf16>(a, tab, st, served);
  if (bits == 4) return f32 ? launch_small_out<4, kOutF32>(a, tab, st, served) : launch_small_out<4, kOutBf16>(a, tab, st, served);
  return f32 ? launch_small_out<8, kOutF32>(a, tab, st, served) : launch_small_out<8, kOutBf16>(a, tab, st, served);
}

}  // namespace rptq
