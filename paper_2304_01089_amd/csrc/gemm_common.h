// Types shared by the cluster GEMM kernels (App. A.4, second method).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rptq_internal.h"

namespace rptq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

struct GemmArgs {
  const uint8_t* codes;      // packed activation codes, row-major
  int64_t M;
  int32_t row_bytes;         // K_p * bits / 8
  const uint8_t* Wq;         // packed weights, fragment-major
  int32_t N;
  int32_t slices;            // K_p / 32
  int32_t used_slices;       // slices up to the end of the last cluster
  int32_t tiles_m, tiles_n;  // output tiles along M and N
  int32_t grp_m, grp_n;      // tile order: blocks of grp_m row tiles x grp_n column tiles
  const float* sW;
  const int32_t* zW;
  const float* colterm;
  const float* rowterm;
  void* y;
  // weights with one parameter pair per (output, cluster) (App. A.4 as printed)
  const float* scale_tab;    // [g, n_padded]: sX_i * sW[o,i]
  const float* cross_tab;    // [n_padded, g2]: -sW[o,i] * zW[o,i], MFMA operand order
  const float* rtc;          // [M, g2]: de-quantized row sum of every cluster, MFMA operand order
  int32_t n_padded;
  int32_t g2;
  float cw_prescale;         // 2^-shift: the operand bytes are code << shift
  // verification mode
  const int32_t* xsum;
  const int32_t* wsum;
  int32_t* yq;
};

struct GemmTab {
  int32_t g;
  int32_t slice_end[RPTQ_MAX_CLUSTERS];   // first slice after cluster i
  float scale[RPTQ_MAX_CLUSTERS];         // sX_i / 2^shift (the operand bytes are code << shift)
  int32_t zx[RPTQ_MAX_CLUSTERS];
  int32_t n[RPTQ_MAX_CLUSTERS];           // channels in cluster i
};

// Output stage that quantizes for the next site instead of storing Y (Sec. 4.2: the rows of
// this layer's weights were reordered offline, so column n of the product is padded position
// n of the next site's cluster-order layout).  Passed by value; unused by the other kernels.
struct GemmQuantOut {
  uint8_t* codes;                          // packed codes of the next site, [M, N * bits / 8]
  double* rt_part;                         // [tiles_n, M]: per column tile, the de-quantized row sum
  int32_t row_bytes;                       // N * bits / 8
  int32_t relu;
  int32_t g;
  int32_t pad_off[RPTQ_MAX_CLUSTERS + 1];  // padded start of the next site's clusters
  int32_t n[RPTQ_MAX_CLUSTERS];            // channels in each
  float inv_s[RPTQ_MAX_CLUSTERS];
  float s[RPTQ_MAX_CLUSTERS];
  int32_t z[RPTQ_MAX_CLUSTERS];
  int32_t zb[RPTQ_MAX_CLUSTERS];           // z - qmin
};

constexpr int kStepSlices = 8;            // slices per K step (256 codes): one barrier per step
constexpr int kSlicePad = 16;             // bytes added to a slice's LDS stride.  The staging stores of 8 consecutive
                                          // lanes go to the 8 slices of one row: with a stride of 2^n + 16 bytes they
                                          // fall into distinct 16-byte bank groups (a stride of 2^n + 64 put them into
                                          // two groups: 2-4 % slower on every shape)

template <int BITS>
struct ActFmt {
  static constexpr int kGroupBytes = BITS * 4;             // bytes of 32 packed codes
  static constexpr int kShift = (BITS == 8) ? 0 : (BITS == 4 ? 4 : 5);
};

#if defined(__HIPCC__)
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

// OUT: what the output stage writes - kOutBf16 / kOutF32: Y; 3, 4 or 8: the next site's packed
// codes of that many bits (ReLU optional) and the partial row sums its product needs.
constexpr int kOutBf16 = 0, kOutF32 = 1;

// Stores the outputs of one row and 16 bytes of columns (4 fp32 or 8 bf16, rounded to nearest even).
template <bool YF32>
__device__ __forceinline__ void store_outputs(const GemmArgs& a, const float* v, int64_t t, int n, bool vec_ok) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  unsigned char* ybase = static_cast<unsigned char*>(a.y);
  if (YF32) {
    if (vec_ok) {
      *reinterpret_cast<float4*>(ybase + (t * a.N + n) * 4) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < a.N) reinterpret_cast<float*>(ybase)[t * a.N + n + e] = v[e];
    }
  } else {
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const f2 pr = {v[(2 * e) % (YF32 ? 4 : 8)], v[(2 * e + 1) % (YF32 ? 4 : 8)]};
      const b2 cv = __builtin_convertvector(pr, b2);
      w[e] = *reinterpret_cast<const uint32_t*>(&cv);
    }
    if (vec_ok) {
      *reinterpret_cast<uint4*>(ybase + (t * a.N + n) * 2) = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (n + e < a.N) reinterpret_cast<uint16_t*>(ybase)[t * a.N + n + e] = static_cast<uint16_t>(w[e / 2] >> (16 * (e & 1)));
    }
  }
}
#endif

// gemm_small.hip: the product with K split over a workgroup's waves, for few output tiles (the choice is made there)
bool small_gemm_serves(int64_t M, int32_t N, int32_t g, int out_mode);
int32_t launch_small_gemm(const GemmArgs& a, const GemmTab& tab, int bits, int out_mode, hipStream_t st);

}  // namespace rptq
