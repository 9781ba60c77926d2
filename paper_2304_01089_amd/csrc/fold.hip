// Offline folding of the reorder index (Sec. 4.2): LayerNorm parameters gathered into the
// padded cluster-order layout, weight columns permuted by the input reorder index (rows by
// the output reorder index when given), 4-bit Min-Max quantization per output channel
// (Eq. 1, Eq. 2 over the whole row), packing into the MFMA-fragment-major weight layout,
// and the per-cluster code sums the integer form of App. A.4 needs.
#include <hip/hip_runtime.h>

#include <condition_variable>
#include <mutex>

#include "device_common.h"
#include "pack_formats.h"
#include "rptq_internal.h"

namespace rptq {

// What the offline kernels report back: bit 0 = a weight is not finite, bit 1 = a row's Eq. 2
// scale is not a normal fp32 number.  A call owns one of the words from its clearing to its read-back, so
// that calls from several threads, on several streams, report their own weights.
constexpr int kStatusWords = 64;
__device__ int32_t g_fold_status[kStatusWords];

__global__ void fold_status_clear_kernel(int word) { g_fold_status[word] = 0; }

class StatusWord {
 public:
  StatusWord() {                                   // (a 65th call at one time waits for another to end)
    std::unique_lock<std::mutex> lock(state().mutex);
    state().freed.wait(lock, [] { return state().taken != ~uint64_t{0}; });
    word_ = __builtin_ctzll(~state().taken);
    state().taken |= uint64_t{1} << word_;
  }
  ~StatusWord() {
    {
      std::lock_guard<std::mutex> lock(state().mutex);
      state().taken &= ~(uint64_t{1} << word_);
    }
    state().freed.notify_one();
  }
  StatusWord(const StatusWord&) = delete;
  StatusWord& operator=(const StatusWord&) = delete;
  int index() const { return word_; }
  int32_t clear(hipStream_t st) const {
    hipLaunchKernelGGL(fold_status_clear_kernel, dim3(1), dim3(1), 0, st, word_);
    RPTQ_HIP(hipGetLastError());
    return RPTQ_OK;
  }
  // Waits for the stream; RPTQ_ERR_RANGE if the kernels reported anything.
  int32_t read(hipStream_t st) const {
    int32_t status = 0;
    RPTQ_HIP(hipMemcpyFromSymbolAsync(&status, HIP_SYMBOL(g_fold_status), sizeof(status), sizeof(status) * word_,
                                      hipMemcpyDeviceToHost, st));
    RPTQ_HIP(hipStreamSynchronize(st));
    return status ? RPTQ_ERR_RANGE : RPTQ_OK;
  }

 private:
  struct State {
    std::mutex mutex;
    std::condition_variable freed;
    uint64_t taken = 0;
  };
  static State& state() {
    static State s;
    return s;
  }
  static_assert(kStatusWords == 64, "a bit each");
  int word_;
};

__global__ void fold_ln_kernel(const float* gamma, const float* beta, const int32_t* perm_pad, int32_t k_padded,
                               float* gamma_pad, float* beta_pad) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= k_padded) return;
  const int c = perm_pad[j];
  gamma_pad[j] = c >= 0 ? gamma[c] : 0.0f;
  beta_pad[j] = c >= 0 ? beta[c] : 0.0f;
}

struct FoldArgs {
  const void* W;
  int32_t w_bf16;
  int32_t N;
  int32_t n_padded;
  int32_t has_perm_out;          // the caller's output index was uploaded into zW[0..N)
  const int32_t* perm_pad;
  uint8_t* Wq;
  float* sW;
  int32_t* zW;
  int32_t* wsum;
  float* colterm;
  int32_t status_word;
};

struct ScaleTab {
  double sz[RPTQ_MAX_CLUSTERS];     // sX_i * zX_i
};

// R output rows per workgroup (R divides 32, so they share a packed block's row band), read once, in order, into
// LDS as fp32 and gathered from there in cluster order.
//
// What bounds it is memory: 4 (or 2) bytes a weight in, half a byte out.  One row per workgroup, gathered from
// memory 4 bytes at a time and written 4 bytes at a time, took 76 us for 8192 x 2048 fp32 weights; rows staged in
// LDS and 16-byte pieces of R neighbouring rows written together take 25 us.  A row's pitch in LDS is odd
// in words, so that the R lanes that read one channel of R rows use R banks.
constexpr int kFoldThreads = 512;

struct FoldLds {
  int rows, wsum, cluster, total;                  // byte offsets, size
};
__host__ __device__ inline FoldLds fold_lds_layout(int r, int k, int g, int k_padded) {
  FoldLds l;
  l.rows = 0;
  l.wsum = r * (k | 1) * 4;
  l.cluster = l.wsum + r * g * 4;
  l.total = l.cluster + (k_padded / kGroup + 15) / 16 * 16;
  return l;
}

template <int R>
__global__ void __launch_bounds__(kFoldThreads) fold_weight_kernel(FoldArgs a, ClusterGeom geom, ScaleTab tab) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ float sh_inv[R];
  __shared__ int32_t sh_z[R], sh_src[R];
  const FoldLds lds = fold_lds_layout(R, geom.k, geom.g, geom.k_padded);
  float* rows = reinterpret_cast<float*>(smem + lds.rows);
  int32_t* sh_wsum = reinterpret_cast<int32_t*>(smem + lds.wsum);      // [R][g]
  uint8_t* sh_cluster = smem + lds.cluster;                            // cluster of every 32-code slice
  const int pitch = geom.k | 1;
  const int o0 = blockIdx.x * R;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int kWaves = kFoldThreads / 64;
  constexpr int kWavesPerRow = kWaves / R;         // waves that read one row (R <= 8)

  for (int sl = tid; sl < geom.k_padded / kGroup; sl += kFoldThreads) {
    int ci = 0;
    for (int i = 1; i < geom.g; ++i) ci += (sl * kGroup >= geom.pad_off[i]) ? 1 : 0;
    sh_cluster[sl] = static_cast<uint8_t>(ci);
  }
  for (int i = tid; i < R * geom.g; i += kFoldThreads) sh_wsum[i] = 0;

  // ---- read the rows, Eq. 2 over each whole row ---------------------------------------------
  __shared__ float red_min[kWaves], red_max[kWaves];
  const int my_row = wid / kWavesPerRow;           // each wave reads (a part of) one row
  const int t = (wid % kWavesPerRow) * 64 + lane;
  constexpr int kStep = kWavesPerRow * 64;
  const int my_o = o0 + my_row;
  // (zW[o] carries the validated source row of output o until it is overwritten with the row's zero
  // point behind the barrier below; rows added by rounding N up and pad rows of the output layout have none)
  const int src_row = my_o < a.N ? (a.has_perm_out ? a.zW[my_o] : my_o) : -1;
  float lo = __builtin_huge_valf(), hi = -__builtin_huge_valf();
  bool bad = false;
  if (src_row >= 0) {
    const uint16_t* wb = static_cast<const uint16_t*>(a.W) + static_cast<int64_t>(src_row) * geom.k;
    const float* wf = static_cast<const float*>(a.W) + static_cast<int64_t>(src_row) * geom.k;
    float* row = rows + my_row * pitch;
    auto take = [&](int c, float w) {
      bad |= !(fabsf(w) <= 3.4028234664e38f);      // NaN or infinity (min/max would skip a NaN)
      lo = fminf(lo, w);
      hi = fmaxf(hi, w);
      row[c] = w;
    };
    if (geom.k % 8 == 0) {                         // whole 16-byte chunks in every row
      if (a.w_bf16) {
#pragma unroll 4
        for (int c = t * 8; c < geom.k; c += kStep * 8) {
          const uint4 v = *reinterpret_cast<const uint4*>(wb + c);
          const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            take(c + 2 * k, bf16_lo(w[k]));
            take(c + 2 * k + 1, bf16_hi(w[k]));
          }
        }
      } else {
#pragma unroll 4
        for (int c = t * 4; c < geom.k; c += kStep * 4) {
          const float4 v = *reinterpret_cast<const float4*>(wf + c);
          take(c, v.x);
          take(c + 1, v.y);
          take(c + 2, v.z);
          take(c + 3, v.w);
        }
      }
    } else {
      for (int c = t; c < geom.k; c += kStep) take(c, a.w_bf16 ? __uint_as_float(static_cast<uint32_t>(wb[c]) << 16) : wf[c]);
    }
  }
  if (bad) atomicOr(&g_fold_status[a.status_word], 1);
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    lo = fminf(lo, __shfl_xor(lo, m, kWave));
    hi = fmaxf(hi, __shfl_xor(hi, m, kWave));
  }
  if (lane == 0) {
    red_min[wid] = lo;
    red_max[wid] = hi;
  }
  __syncthreads();
  if (t == 0) {                                    // one thread per row
    float s32 = 1.0f;
    int32_t z32 = 0;
    if (src_row >= 0) {
      for (int k = 0; k < kWavesPerRow; ++k) {
        lo = fminf(lo, red_min[wid + k]);
        hi = fmaxf(hi, red_max[wid + k]);
      }
      const double l = lo + 0.0f;
      const double h = hi + 0.0f;
      double s64, zz;
      if (h == l) {
        s64 = 1.0;
        zz = -rint(l);
      } else {
        s64 = (h - l) / 16.0;
        zz = -rint((h + l) / (2.0 * s64));
      }
      s32 = static_cast<float>(s64);
      if (!(s32 >= 1.17549435e-38f && s32 <= 3.4028234664e38f)) atomicOr(&g_fold_status[a.status_word], 2);
      z32 = static_cast<int32_t>(zz);
    }
    sh_inv[my_row] = static_cast<float>(1.0 / static_cast<double>(s32));
    sh_z[my_row] = z32;
    sh_src[my_row] = src_row;
    if (my_o < a.N) {                              // (a pad row: weights 0, s = 1, z = 0)
      a.sW[my_o] = s32;
      a.zW[my_o] = z32;
    }
  }
  __syncthreads();

  // ---- Eq. 1 per weight, pack: a thread owns a 16-byte piece of a packed block (two runs of 16 codes, in
  // neighbouring slices) of one row; neighbouring threads own the same piece of neighbouring rows
  const int r = tid % R;
  const int src = sh_src[r];
  const float inv = sh_inv[r];
  const float zf = static_cast<float>(sh_z[r]);
  const float* row = rows + r * pitch;
  const int pieces = geom.k_padded / kGroup;
  for (int p = tid / R; p < pieces; p += kFoldThreads / R) {
    const int sl = (p >> 1) * 2, h = p & 1;        // first slice of the pair; which half of its codes
    uint32_t word[4] = {0u, 0u, 0u, 0u};
    if (src >= 0) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        int sum = 0;
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          const int pos = (sl + q) * kGroup + h * 16 + v * 8;
          const int4 c0 = *reinterpret_cast<const int4*>(a.perm_pad + pos);
          const int4 c1 = *reinterpret_cast<const int4*>(a.perm_pad + pos + 4);
          const int c[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float b = __fadd_rn(rintf(__fmul_rn(row[c[e] < 0 ? 0 : c[e]], inv)), zf);
            b = fminf(fmaxf(b, -8.0f), 7.0f);
            const int code = c[e] < 0 ? 0 : static_cast<int>(b);
            sum += code;
            word[q * 2 + v] |= static_cast<uint32_t>(code & 15) << (8 * (e & 3) + (e < 4 ? 4 : 0));
          }
        }
        atomicAdd(&sh_wsum[r * geom.g + sh_cluster[sl + q]], sum);
      }
    }
    *reinterpret_cast<uint4*>(a.Wq + weight_dword_offset(o0 + r, sl * 4 + h * 2, geom.k_padded)) =
        make_uint4(word[0], word[1], word[2], word[3]);
  }
  __syncthreads();
  for (int i = tid; i < R * geom.g; i += kFoldThreads) {
    const int o = o0 + i / geom.g;
    if (o < a.N) a.wsum[static_cast<int64_t>(o0) * geom.g + i] = sh_wsum[i];
  }
  if (tid < R && o0 + tid < a.N) {
    double acc = 0.0;
    for (int i = 0; i < geom.g; ++i) acc += tab.sz[i] * static_cast<double>(sh_wsum[tid * geom.g + i]);
    a.colterm[o0 + tid] = static_cast<float>(acc);
  }
}


// ---- App. A.4 as printed: one Eq. 2 pair per (output channel, input cluster) ------------------
struct FoldCwArgs {
  const void* W;
  int32_t w_bf16;
  int32_t N;
  int32_t n_padded;
  int32_t has_perm_out;
  const int32_t* perm_pad;
  uint8_t* Wq;
  float* sW;            // [N, g]
  int32_t* zW;          // [N, g]; row o's first entry carries the source row until it is overwritten
  int32_t* wsum;        // [N, g]
  float* scale_tab;     // [g, n_padded]: sX_i * sW[o,i]
  float* cross_tab;     // [n_padded, g2], position of cluster i: (i & 1) * g2/2 + i/2; holds -sW[o,i] * zW[o,i]
  float* colterm;       // [N]: sum_i sX_i sW[o,i] zX_i wsum[o,i]
  int32_t g2;
  int32_t status_word;
};

struct ScaleTabCw {
  double sx[RPTQ_MAX_CLUSTERS];
  double zx[RPTQ_MAX_CLUSTERS];
};

__global__ void __launch_bounds__(256) fold_weight_cw_kernel(FoldCwArgs a, ClusterGeom geom, ScaleTabCw tab) {
  __shared__ uint32_t k_lo[RPTQ_MAX_CLUSTERS], k_hi[RPTQ_MAX_CLUSTERS];
  __shared__ float sh_inv[RPTQ_MAX_CLUSTERS], sh_s[RPTQ_MAX_CLUSTERS];
  __shared__ int32_t sh_z[RPTQ_MAX_CLUSTERS], sh_wsum[RPTQ_MAX_CLUSTERS];
  const int o = blockIdx.x;
  const int tid = threadIdx.x;
  const int n_units = geom.k_padded / 8;
  const int g = geom.g;

  for (int i = tid; i < a.g2; i += blockDim.x) a.cross_tab[static_cast<int64_t>(o) * a.g2 + i] = 0.0f;
  const int64_t src_row = (o < a.N) ? (a.has_perm_out ? a.zW[static_cast<int64_t>(o) * g] : o) : -1;
  if (src_row < 0) {                               // a pad row: weights 0, every scale 1, every zero point 0
    for (int u = tid; u < n_units; u += blockDim.x)
      *reinterpret_cast<uint32_t*>(a.Wq + weight_dword_offset(o, u, geom.k_padded)) = 0u;
    __syncthreads();
    if (tid < g) {
      a.scale_tab[static_cast<int64_t>(tid) * a.n_padded + o] = static_cast<float>(tab.sx[tid]);
      if (o < a.N) {
        a.wsum[static_cast<int64_t>(o) * g + tid] = 0;
        a.sW[static_cast<int64_t>(o) * g + tid] = 1.0f;
        a.zW[static_cast<int64_t>(o) * g + tid] = 0;
      }
    }
    if (tid == 0 && o < a.N) a.colterm[o] = 0.0f;
    return;
  }
  const uint16_t* wb = static_cast<const uint16_t*>(a.W) + src_row * geom.k;
  const float* wf = static_cast<const float*>(a.W) + src_row * geom.k;
  auto wval = [&](int c) -> float { return a.w_bf16 ? __uint_as_float(static_cast<uint32_t>(wb[c]) << 16) : wf[c]; };

  if (tid < g) {
    k_lo[tid] = 0xffffffffu;
    k_hi[tid] = 0u;
    sh_wsum[tid] = 0;
  }
  __syncthreads();
  // ---- minimum and maximum of every cluster block of the row (order-free: integer images of the floats)
  bool bad = false;
  for (int u = tid; u < n_units; u += blockDim.x) {
    int ci = 0;
    for (int i = 1; i < g; ++i) ci += (u * 8 >= geom.pad_off[i]) ? 1 : 0;
    float lo = __builtin_huge_valf(), hi = -__builtin_huge_valf();
    bool any = false;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = a.perm_pad[u * 8 + e];
      if (c >= 0) {
        const float w = wval(c);
        bad |= !(fabsf(w) <= 3.4028234664e38f);
        lo = fminf(lo, w);
        hi = fmaxf(hi, w);
        any = true;
      }
    }
    if (any) {
      atomicMin(&k_lo[ci], float_key(lo));
      atomicMax(&k_hi[ci], float_key(hi));
    }
  }
  if (bad) atomicOr(&g_fold_status[a.status_word], 1);
  __syncthreads();
  if (tid < g) {                                   // Eq. 2 for block (o, tid)
    const double l = key_float(k_lo[tid]) + 0.0f, h = key_float(k_hi[tid]) + 0.0f;
    double s64, zz;
    if (h == l) {
      s64 = 1.0;
      zz = -rint(l);
    } else {
      s64 = (h - l) / 16.0;
      zz = -rint((h + l) / (2.0 * s64));
    }
    const float s32 = static_cast<float>(s64);
    // (a block that lies far from zero relative to its width has a large zero point: at most
    // 8 * 2 * 2^24 for fp32 extrema that differ, so it always fits an int32)
    if (!(s32 >= 1.17549435e-38f && s32 <= 3.4028234664e38f) || !(fabs(zz) <= 1073741824.0)) atomicOr(&g_fold_status[a.status_word], 2);
    sh_s[tid] = s32;
    sh_inv[tid] = static_cast<float>(1.0 / static_cast<double>(s32));
    sh_z[tid] = static_cast<int32_t>(zz);
  }
  __syncthreads();
  // ---- Eq. 1 per weight with its block's pair, pack eight codes per dword
  for (int u = tid; u < n_units; u += blockDim.x) {
    int ci = 0;
    for (int i = 1; i < g; ++i) ci += (u * 8 >= geom.pad_off[i]) ? 1 : 0;
    const float inv = sh_inv[ci];
    const double zd = static_cast<double>(sh_z[ci]);
    int q[8];
    int sum = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = a.perm_pad[u * 8 + e];
      int code = 0;
      if (c >= 0) {
        const float r = __fmul_rn(wval(c), inv);           // one fp32 rounding, as everywhere
        double b = rint(static_cast<double>(r)) + zd;      // the zero point of a block may exceed fp32's exact integers
        b = fmin(fmax(b, -8.0), 7.0);
        code = static_cast<int>(b);
      }
      q[e] = code;
      sum += code;
    }
    uint32_t word = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) word |= static_cast<uint32_t>(((q[b] & 15) << 4) | (q[4 + b] & 15)) << (8 * b);
    *reinterpret_cast<uint32_t*>(a.Wq + weight_dword_offset(o, u, geom.k_padded)) = word;
    atomicAdd(&sh_wsum[ci], sum);
  }
  __syncthreads();
  if (tid < g) {
    const int64_t k = static_cast<int64_t>(o) * g + tid;
    a.wsum[k] = sh_wsum[tid];
    a.sW[k] = sh_s[tid];
    a.zW[k] = sh_z[tid];
    a.scale_tab[static_cast<int64_t>(tid) * a.n_padded + o] = static_cast<float>(tab.sx[tid] * static_cast<double>(sh_s[tid]));
    a.cross_tab[static_cast<int64_t>(o) * a.g2 + (tid & 1) * (a.g2 / 2) + (tid >> 1)] =
        static_cast<float>(-static_cast<double>(sh_s[tid]) * static_cast<double>(sh_z[tid]));
  }
  if (tid == 0) {
    double acc = 0.0;
    for (int i = 0; i < g; ++i)
      acc += tab.sx[i] * static_cast<double>(sh_s[i]) * tab.zx[i] * static_cast<double>(sh_wsum[i]);
    a.colterm[o] = static_cast<float>(acc);
  }
}

__global__ void unpack_weights_kernel(const uint8_t* Wq, int N, ClusterGeom geom, int8_t* out) {
  const int o = blockIdx.x;
  if (o >= N) return;
  for (int j = threadIdx.x; j < geom.k; j += blockDim.x) {
    int ci = 0;
    for (int i = 1; i < geom.g; ++i) ci += (j >= geom.off[i]) ? 1 : 0;
    const int pos = geom.pad_off[ci] + (j - geom.off[ci]);
    const int u = pos >> 3, e = pos & 7;
    const uint8_t byte = Wq[weight_dword_offset(o, u, geom.k_padded) + (e & 3)];
    const int nib = (e < 4) ? (byte >> 4) : (byte & 15);
    out[static_cast<int64_t>(o) * geom.k + j] = static_cast<int8_t>((nib ^ 8) - 8);
  }
}

template <int R>
static int32_t launch_fold_rows(const FoldArgs& a, const ClusterGeom& geom, const ScaleTab& tab, hipStream_t st) {
  const size_t shmem = static_cast<size_t>(fold_lds_layout(R, geom.k, geom.g, geom.k_padded).total);
  auto kern = fold_weight_kernel<R>;
  static LdsGrant lds_granted;
  if (int32_t s = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), shmem + 1024, &lds_granted, st)) return s;
  hipLaunchKernelGGL(kern, dim3(a.n_padded / R), dim3(kFoldThreads), shmem, st, a, geom, tab);
  RPTQ_HIP(hipGetLastError());
  return RPTQ_OK;
}

int32_t launch_fold(const float* gamma, const float* beta, const int32_t* perm_pad_host, const ClusterGeom& geom,
                    const float* sX, const int32_t* zX, const void* W, int32_t w_dtype, int32_t N,
                    const int32_t* perm_out_host, int32_t* perm_pad, float* gamma_pad, float* beta_pad,
                    void* Wq_packed, float* sW, int32_t* zW, int32_t* wsum, float* colterm, hipStream_t st) {
  // (refused before anything is recorded: a graph would keep copies from host arrays that end with this call)
  if (int32_t s = require_not_capturing(st)) return s;
  // the index arrays were validated on the host; they are uploaded from there, so what the
  // kernels read is what was checked
  RPTQ_HIP(hipMemcpyAsync(perm_pad, perm_pad_host, sizeof(int32_t) * geom.k_padded, hipMemcpyHostToDevice, st));
  if (gamma) {
    hipLaunchKernelGGL(fold_ln_kernel, dim3((geom.k_padded + 255) / 256), dim3(256), 0, st, gamma, beta, perm_pad,
                       geom.k_padded, gamma_pad, beta_pad);
    RPTQ_HIP(hipGetLastError());
  }
  if (!W) {
    RPTQ_HIP(hipStreamSynchronize(st));            // perm_pad_host belongs to the caller's frame
    return RPTQ_OK;
  }
  if (perm_out_host) RPTQ_HIP(hipMemcpyAsync(zW, perm_out_host, sizeof(int32_t) * N, hipMemcpyHostToDevice, st));
  FoldArgs a;
  a.W = W;
  a.w_bf16 = (w_dtype == RPTQ_DTYPE_BF16);
  a.N = N;
  a.n_padded = (N + RPTQ_N_ALIGN - 1) / RPTQ_N_ALIGN * RPTQ_N_ALIGN;
  a.has_perm_out = perm_out_host != nullptr;
  a.perm_pad = perm_pad;
  a.Wq = static_cast<uint8_t*>(Wq_packed);
  a.sW = sW;
  a.zW = zW;
  a.wsum = wsum;
  a.colterm = colterm;
  ScaleTab tab;
  for (int i = 0; i < RPTQ_MAX_CLUSTERS; ++i)
    tab.sz[i] = i < geom.g ? static_cast<double>(sX[i]) * static_cast<double>(zX[i]) : 0.0;
  const StatusWord status;
  a.status_word = status.index();
  if (int32_t s = status.clear(st)) return s;
  // As many rows per workgroup as leave two workgroups per compute unit (eight at most: their pieces fill whole
  // cache lines), down to one row, for which the LDS holds every width.
  auto fits = [&](int r) { return fold_lds_layout(r, geom.k, geom.g, geom.k_padded).total <= 80 * 1024 - 256; };
  static_assert(RPTQ_MAX_CHANNELS * 4 + RPTQ_MAX_CLUSTERS * 4 + RPTQ_MAX_K_PADDED / kGroup + 1024 <= 160 * 1024, "one row fits");
  int32_t rc;
  if (fits(8)) rc = launch_fold_rows<8>(a, geom, tab, st);
  else if (fits(4)) rc = launch_fold_rows<4>(a, geom, tab, st);
  else if (fits(2)) rc = launch_fold_rows<2>(a, geom, tab, st);
  else rc = launch_fold_rows<1>(a, geom, tab, st);
  if (rc) return rc;
  return status.read(st);
}


int32_t launch_fold_cw(const int32_t* perm_pad_host, const ClusterGeom& geom, const float* sX, const int32_t* zX,
                       const void* W, int32_t w_dtype, int32_t N, const int32_t* perm_out_host, int32_t* perm_pad,
                       void* Wq_packed, float* sW, int32_t* zW, int32_t* wsum, float* scale_tab, float* cross_tab,
                       float* colterm, hipStream_t st) {
  if (int32_t s = require_not_capturing(st)) return s;
  RPTQ_HIP(hipMemcpyAsync(perm_pad, perm_pad_host, sizeof(int32_t) * geom.k_padded, hipMemcpyHostToDevice, st));
  // the validated source rows travel in the first zero-point entry of every output row
  if (perm_out_host)
    RPTQ_HIP(hipMemcpy2DAsync(zW, sizeof(int32_t) * geom.g, perm_out_host, sizeof(int32_t), sizeof(int32_t), N,
                              hipMemcpyHostToDevice, st));
  FoldCwArgs a;
  a.W = W;
  a.w_bf16 = (w_dtype == RPTQ_DTYPE_BF16);
  a.N = N;
  a.n_padded = (N + RPTQ_N_ALIGN - 1) / RPTQ_N_ALIGN * RPTQ_N_ALIGN;
  a.has_perm_out = perm_out_host != nullptr;
  a.perm_pad = perm_pad;
  a.Wq = static_cast<uint8_t*>(Wq_packed);
  a.sW = sW;
  a.zW = zW;
  a.wsum = wsum;
  a.scale_tab = scale_tab;
  a.cross_tab = cross_tab;
  a.colterm = colterm;
  a.g2 = geom.g <= 32 ? 32 : 64;
  ScaleTabCw tab;
  for (int i = 0; i < RPTQ_MAX_CLUSTERS; ++i) {
    tab.sx[i] = i < geom.g ? static_cast<double>(sX[i]) : 0.0;
    tab.zx[i] = i < geom.g ? static_cast<double>(zX[i]) : 0.0;
  }
  const StatusWord status;
  a.status_word = status.index();
  if (int32_t s = status.clear(st)) return s;
  hipLaunchKernelGGL(fold_weight_cw_kernel, dim3(a.n_padded), dim3(256), 0, st, a, geom, tab);
  RPTQ_HIP(hipGetLastError());
  return status.read(st);
}

int32_t launch_unpack_weights(const void* Wq, int32_t N, const ClusterGeom& geom, int8_t* out, hipStream_t st) {
  hipLaunchKernelGGL(unpack_weights_kernel, dim3(N), dim3(256), 0, st, static_cast<const uint8_t*>(Wq), N, geom, out);
  RPTQ_HIP(hipGetLastError());
  return RPTQ_OK;
}

}  // namespace rptq
