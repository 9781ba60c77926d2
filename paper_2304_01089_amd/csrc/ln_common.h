// What the two LayerNorm + quantize kernels (ln_quant.hip, ln_rows.hip) share.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_common.h"
#include "rptq_internal.h"

namespace rptq {

// 16 bytes as a plain vector value (copies of the runtime's uint4 struct are memory copies, which can keep
// register arrays in scratch memory)
typedef unsigned u4v __attribute__((ext_vector_type(4)));

struct LnQuantArgs {
  const uint4* x;          // bf16 [M, d], 8 values per uint4
  int64_t M;
  int32_t d;
  int32_t chunks;          // d / 8
  const float* gamma_pad;
  const float* beta_pad;
  float eps;
  int32_t relu;
  const int32_t* perm_pad;
  uint8_t* codes;
  float* rowterm;
  int32_t n_units;         // K_p / codes-per-unit
  int32_t row_bytes;       // K_p * bits / 8
  int32_t ring;            // row buffers in LDS: 3, or 2 (one more barrier per row) when three do not fit
};

template <int BITS>
struct Unit {
  static constexpr int kCodes = (BITS == 3) ? 16 : 8;
};

// Position inside its 32-group of local code e of a 3-bit unit with the given role.
// role 0 carries codes 0..7, 24..27, 16..19; role 1 carries 8..15, 28..31, 20..23.
__device__ __forceinline__ int pos3(int role, int e) {
  if (e < 8) return role * 8 + e;
  if (e < 12) return 24 + role * 4 + (e - 8);
  return 16 + role * 4 + (e - 12);
}

// Round half to even, then add an integer zero point z: adding 1.5 * 2^23 rounds r to an integer, taking away
// 1.5 * 2^23 - z (exact for |z| <= 2^21 + 128, as the difference is) leaves rint(r) + z.  From |r| = 2^22 on the result is
// no longer that integer, but stays beyond every code range, where the clamps put both.  Two additions at the full
// rate; the rounding instruction issues at half of it.
constexpr float kRoundMagic = 12582912.0f;
__device__ __forceinline__ float round_biased(float r, float magic_minus_z) { return __fsub_rn(__fadd_rn(r, kRoundMagic), magic_minus_z); }

// Packs one unit's biased code bytes and stores them at `dst` (its place in the output row).  A 3-bit unit of role
// 0 or 1 exchanges its half of the third dword with its partner in lane ^ 1.
template <int BITS>
__device__ __forceinline__ void store_unit(const uint32_t* D, int role, bool ok, uint8_t* dst) {
  if constexpr (BITS == 8) {
    uint2 o;
    o.x = D[0] ^ 0x80808080u;
    o.y = D[1] ^ 0x80808080u;
    if (ok) *reinterpret_cast<uint2*>(dst) = o;
  } else if constexpr (BITS == 4) {
    const uint32_t o = ((D[0] << 4) | D[1]) ^ 0x88888888u;
    if (ok) *reinterpret_cast<uint32_t*>(dst) = o;
  } else {
    // role 0 -> x0 and its half of x2; role 1 -> x1 and its half of x2 (partner = lane ^ 1)
    const uint32_t w1 = ((D[0] << 5) | (D[1] << 2) | ((D[2] >> 1) & 0x03030303u)) ^ 0x80808080u ^ 0x10101010u ^ 0x02020202u;
    const uint32_t mine = role ? (((D[3] << 2) ^ 0x10101010u) | ((D[2] & 0x01010101u) << 1))
                               : (((D[3] << 5) ^ 0x80808080u) | (D[2] & 0x01010101u));
    const uint32_t other = __shfl_xor(mine, 1, kWave);
    if (ok) {
      uint32_t* p = reinterpret_cast<uint32_t*>(dst);
      p[0] = w1;
      if (role) p[1] = mine | other;
    }
  }
}

// ln_rows.hip: the kernel for calls with few rows per compute unit; nunit units and nch 16-byte chunks of a row per
// thread.  *served tells whether it took the call (the choice is made there).
int32_t launch_ln_rows(const LnQuantArgs& a, const ClusterGeom& geom, const QuantTab& qt, int bits, int nunit, int nch,
                       int threads, int cus, hipStream_t st, bool* served);

}  // namespace rptq
