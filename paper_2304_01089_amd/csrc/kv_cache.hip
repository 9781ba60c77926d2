// Key / value cache codes (Sec. 5.1: the W4A4KV, W4A3KV and W3A3KV settings quantize only the
// key and value caches; one reorder index per attention head, shared by queries and keys,
// Sec. 4.2) - writing: per head, channels in cluster order, Eq. 1 with the cluster's Eq. 2
// pair, packed at 3, 4 or 8 bits; reading: x_hat = s (x_q - z) as bf16 in cluster order.
//
// The cache layout is dense (no padding of clusters: the cache is what the method saves
// memory on), so the quantizer constants are per position, in a device table built once.
// A reorder index never moves a channel out of its head, so the gather is local: one wave
// owns a tile of 1024 consecutive channels (whole heads) of a row and stages its 2 KiB through
// a private piece of LDS.  The only workgroup barrier is the one behind the table, which all waves share.
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "pack_formats.h"
#include "rptq_internal.h"

namespace rptq {

constexpr int kKvTile = 1024;                  // channels per wave tile
constexpr int kKvLaneCodes = 16;               // codes per lane

// position of local code e of a lane inside the wave tile
template <int BITS>
__device__ __forceinline__ int kv_local_pos(int lane, int e) {
  if (BITS == 3) {
    // lanes 2g, 2g+1 share the 32-code group g: lane 2g carries codes 0..7, 24..27, 16..19,
    // lane 2g+1 codes 8..15, 28..31, 20..23 (so that each owns whole dwords of the group)
    const int role = lane & 1, gbase = (lane >> 1) * kGroup;
    if (e < 8) return gbase + role * 8 + e;
    if (e < 12) return gbase + 24 + role * 4 + (e - 8);
    return gbase + 16 + role * 4 + (e - 12);
  }
  return lane * kKvLaneCodes + e;
}

template <int BITS>
__global__ void __launch_bounds__(256) kv_quant_kernel(const uint4* x, int64_t T, int32_t d, const KvPos* pos,
                                                       uint8_t* codes, int32_t segs, int32_t row_groups) {
  constexpr int kQMin = -(1 << (BITS - 1));
  constexpr float kUMax = static_cast<float>((1 << BITS) - 1);
  // The tile's table records, read by the whole workgroup in order.  (A lane's 16 records are 256 bytes of their own:
  // requested by the lanes that need them, every request touches 64 cache lines, and that was most of the time of few rows:
  // 16 x 2048 5.6 -> 3.1 us; from memory, 4 bits, 1000 x 2048 10.2 -> 5.3, 1000 x 12288 17.8 -> 10.9, 8192 x 12288 57 -> 51.)  16 bytes follow
  // every lane's records, so that eight lanes read from different banks.
  constexpr int kLaneTab = kKvLaneCodes * 16 + 16;
  __shared__ __align__(16) unsigned char tab[kWave * kLaneTab];
  __shared__ __align__(16) unsigned char lds[4][kKvTile * 2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int seg = blockIdx.x % segs, rg = blockIdx.x / segs;
  const int base_ch = seg * kKvTile;
  const int n_here = (d - base_ch) < kKvTile ? (d - base_ch) : kKvTile;      // channels of this tile (multiple of 32)
  unsigned char* my = lds[wave];

  const bool lane_ok = (BITS == 3) ? ((lane >> 1) * kGroup < n_here) : (lane * kKvLaneCodes < n_here);
  // this lane's two 16-byte chunks of the tile's input (clamped inside the tile; surplus data is never gathered)
  const int chunks_here = n_here / 8;
  const int64_t row_chunks = d / 8;
  const int64_t stride = static_cast<int64_t>(row_groups) * 4;
  int64_t row = static_cast<int64_t>(rg) * 4 + wave;
  const int64_t out_row_bytes = static_cast<int64_t>(d) * BITS / 8;
  const int64_t out_tile = static_cast<int64_t>(base_ch) * BITS / 8;

  // (scalars, not arrays handed to a helper by pointer: those ended up in scratch memory, re-written
  // every row)
  const int ch0 = lane < chunks_here ? lane : (chunks_here - 1);
  const int ch1 = (64 + lane) < chunks_here ? (64 + lane) : (chunks_here - 1);
  auto row_ptr = [&](int64_t r) {
    if (r >= T) r = T - 1;
    return x + r * row_chunks + base_ch / 8;
  };
  // (requested before the table, so that the two latencies run side by side)
  const uint4* p0 = row_ptr(row);
  uint4 cur0 = p0[ch0], cur1 = p0[ch1];
  const uint4* p1 = row_ptr(row + stride);
  uint4 nxt0 = p1[ch0], nxt1 = p1[ch1];
  typedef unsigned u4v __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int k = 0; k < kKvTile / 256; ++k) {
    const int i = k * 256 + static_cast<int>(threadIdx.x);
    *reinterpret_cast<u4v*>(tab + i * 16 + i / kKvLaneCodes * 16) = reinterpret_cast<const u4v*>(pos)[base_ch + (i < n_here ? i : 0)];
  }
  __syncthreads();
  // per-lane constants: source offset inside the tile, 1/s and the biased zero point of each code
  uint32_t src[kKvLaneCodes];
  float inv_s[kKvLaneCodes], zbf[kKvLaneCodes];
#pragma unroll
  for (int e = 0; e < kKvLaneCodes; ++e) {
    const int lp = kv_local_pos<BITS>(lane, e);
    const KvPos kp = *reinterpret_cast<const KvPos*>(tab + lp * 16 + lp / kKvLaneCodes * 16);
    src[e] = static_cast<uint32_t>(kp.src - base_ch) * 2u;
    inv_s[e] = kp.inv_s;
    zbf[e] = static_cast<float>(kp.z - kQMin);
  }
  for (; row < T; row += stride) {
    *reinterpret_cast<uint4*>(my + lane * 16) = cur0;
    *reinterpret_cast<uint4*>(my + (64 + lane) * 16) = cur1;
    cur0 = nxt0;
    cur1 = nxt1;
    const uint4* p2 = row_ptr(row + 2 * stride);
    nxt0 = p2[ch0];
    nxt1 = p2[ch1];
    wave_lds_fence();
    uint32_t D[4] = {0u, 0u, 0u, 0u};                // biased codes, one byte each
#pragma unroll
    for (int e = 0; e < kKvLaneCodes; ++e) {
      const uint32_t h = *reinterpret_cast<const uint16_t*>(my + src[e]);
      const float y = __uint_as_float(h << 16);
      const float r = __fmul_rn(y, inv_s[e]);
      float b = __fadd_rn(rintf(r), zbf[e]);         // round, then add the zero point (biased by -qmin)
      if (BITS < 8) b = fminf(b, kUMax);             // upper clamp; the conversion saturates at 0 and 255
      D[e / 4] = __builtin_amdgcn_cvt_pk_u8_f32(b, e & 3, D[e / 4]);
    }
    wave_lds_fence();
    uint8_t* out = codes + row * out_row_bytes + out_tile;
    if (BITS == 8) {
      const uint4 o = make_uint4(D[0] ^ 0x80808080u, D[1] ^ 0x80808080u, D[2] ^ 0x80808080u, D[3] ^ 0x80808080u);
      if (lane_ok) *reinterpret_cast<uint4*>(out + lane * 16) = o;
    } else if (BITS == 4) {
      uint2 o;
      o.x = ((D[0] << 4) | D[1]) ^ 0x88888888u;
      o.y = ((D[2] << 4) | D[3]) ^ 0x88888888u;
      if (lane_ok) *reinterpret_cast<uint2*>(out + lane * 8) = o;
    } else {
      const int role = lane & 1;
      const uint32_t w1 = ((D[0] << 5) | (D[1] << 2) | ((D[2] >> 1) & 0x03030303u)) ^ 0x80808080u ^ 0x10101010u ^ 0x02020202u;
      const uint32_t mine = role ? (((D[3] << 2) ^ 0x10101010u) | ((D[2] & 0x01010101u) << 1))
                                 : (((D[3] << 5) ^ 0x80808080u) | (D[2] & 0x01010101u));
      const uint32_t other = __shfl_xor(mine, 1, kWave);
      if (lane_ok) {
        uint32_t* p = reinterpret_cast<uint32_t*>(out + (lane >> 1) * 12 + role * 4);
        p[0] = w1;
        if (role) p[1] = mine | other;
      }
    }
  }
}

// Read-back.  Memory bound (d*bits/8 bytes in, 2d out per row), so the stores decide: a lane expands 8
// consecutive codes of a row into one 16-byte store, a wave's store is 1 KiB contiguous.  One lane per 32-code group with
// four 16-byte stores 64 bytes apart took 91 us at 8192 x 12288, 3 bits, this split 68, with non-temporal stores 42 us
// (5.7 TB/s; 39 to 50 inside a pass).  But attention reads the values next, and non-temporal stores send them past the
// 256 MiB last-level cache: they are used only where the keys and values of a layer together would not stay in it.  us for key and value of one
// layer, the two read-backs alone and followed by a full read of both, ordinary | non-temporal:
//    17 MB each   13.8 | 11.8    48 |  50        101 MB   48 | 47   101 | 119
//    34 MB        23.0 | 19.8    57 |  61        151 MB  110 | 64   211 | 170
//    67 MB        37.0 | 34.6    79 |  89        201 MB  138 | 84   265 | 254
// The 8 positions' constants stay in registers; kKvRowsAhead rows are requested while the rows
// before them are expanded (2, 4 and 8 rows measured the same).
constexpr int64_t kKvStreamBytes = 128ll << 20;
constexpr int kKvRowsAhead = 2;

template <int BITS, bool STREAM>
__global__ void __launch_bounds__(256) kv_dequant_kernel(const uint8_t* codes, int64_t T, int32_t d, const KvPos* pos,
                                                         uint16_t* out, int32_t blocks_per_row) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  typedef unsigned u4v __attribute__((ext_vector_type(4)));
  constexpr int ND = (BITS == 3) ? 3 : BITS / 4;       // dwords a lane reads per row
  // (s, z) of the workgroup's 2048 positions: the table is read in order and changes threads in LDS, as in kv_quant.  (From
  // memory, us for rows x channels, each thread reading its own 128 bytes of table | this: 4096 x 2048 8.1 | 7.1, 1000 x 2048
  // at 8 bits 5.2 | 4.4, 1000 x 12288 at 3 bits 10.9 | 9.0, 2048 x 12288 at 8 bits 23.1 | 18.5, 65536 x 768 at 8 bits 31.4 | 33.0.)
  // 16 bytes follow every thread's 64.
  typedef unsigned u2v __attribute__((ext_vector_type(2)));
  __shared__ __align__(16) unsigned char tab[256 * 80];
  const int u0 = static_cast<int>(blockIdx.x % blocks_per_row) * 256;
  const int u_here = u0 + static_cast<int>(threadIdx.x);
  const int u = u_here < d / 8 ? u_here : d / 8 - 1;      // unit of 8 codes, the same for every row
  const int64_t row_bytes = static_cast<int64_t>(d) * BITS / 8;
  const int64_t stride = gridDim.x / blocks_per_row;
  const int k3 = u & 3;                                // 3-bit: which quarter of the 32-code group
  const uint8_t* lane_src = codes + ((BITS == 3) ? static_cast<int64_t>(u >> 2) * 12 : static_cast<int64_t>(u) * BITS);
  uint16_t* lane_dst = out + static_cast<int64_t>(u) * 8;
  // (rows past the end: the last row again, never stored)
  auto load_row = [&](int64_t row, uint32_t (&w)[ND]) {
    if (row >= T) row = T - 1;
    const uint32_t* p = reinterpret_cast<const uint32_t*>(lane_src + row * row_bytes);
#pragma unroll
    for (int k = 0; k < ND; ++k) w[k] = p[k];
  };
  uint32_t cur[kKvRowsAhead][ND], nxt[kKvRowsAhead][ND];
  int64_t row = blockIdx.x / blocks_per_row;
  // (requested before the table, so that the two latencies run side by side)
#pragma unroll
  for (int k = 0; k < kKvRowsAhead; ++k) load_row(row + k * stride, cur[k]);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int i = k * 256 + static_cast<int>(threadIdx.x);
    const u4v rec = reinterpret_cast<const u4v*>(pos)[min(u0 * 8 + i, d - 1)];
    *reinterpret_cast<u2v*>(tab + i * 8 + i / 8 * 16) = u2v{rec[2], rec[3]};
  }
  __syncthreads();
  if (u_here >= d / 8) return;
  float s[8], zf[8];
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    const u4v r2 = *reinterpret_cast<const u4v*>(tab + threadIdx.x * 80 + j * 8);
    s[j] = __uint_as_float(r2[0]);
    zf[j] = static_cast<float>(static_cast<int>(r2[1]));
    s[j + 1] = __uint_as_float(r2[2]);
    zf[j + 1] = static_cast<float>(static_cast<int>(r2[3]));
  }
  auto store_row = [&](int64_t row, const uint32_t (&w)[ND]) {
    int q[8];
    if constexpr (BITS == 8) {
#pragma unroll
      for (int j = 0; j < 8; ++j) q[j] = static_cast<int>(w[(j / 4) % ND] << (24 - 8 * (j & 3))) >> 24;
    } else if constexpr (BITS == 4) {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        q[b] = static_cast<int>(w[0] << (24 - 8 * b)) >> 28;
        q[4 + b] = static_cast<int>(w[0] << (28 - 8 * b)) >> 28;
      }
    } else {
      // quarters 0..2 hold their codes in bits 7..5 and 4..2 of their own dword's bytes; quarter 3's are
      // spread over the three dwords and are brought into the same places
      const uint32_t w3 = ((w[0] << 6) & 0xc0c0c0c0u) | ((w[2 % ND] << 5) & 0x20202020u) | ((w[1 % ND] << 3) & 0x18181818u) |
                          ((w[2 % ND] << 1) & 0x04040404u);
      const uint32_t v = k3 == 0 ? w[0] : (k3 == 1 ? w[1 % ND] : (k3 == 2 ? w[2 % ND] : w3));
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        q[b] = static_cast<int>(v << (24 - 8 * b)) >> 29;
        q[4 + b] = static_cast<int>(v << (27 - 8 * b)) >> 29;
      }
    }
    u4v o;
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
      // s (x_q - z): the integer difference is exact in fp32, one rounded product, then bf16 (ties to even)
      const f2 pr = {__fmul_rn(s[j], static_cast<float>(q[j]) - zf[j]), __fmul_rn(s[j + 1], static_cast<float>(q[j + 1]) - zf[j + 1])};
      const b2 cv = __builtin_convertvector(pr, b2);
      o[j / 2] = *reinterpret_cast<const uint32_t*>(&cv);
    }
    if (row < T) {
      u4v* dst = reinterpret_cast<u4v*>(lane_dst + row * d);
      if (STREAM) __builtin_nontemporal_store(o, dst);
      else *dst = o;
    }
  };
  for (; row < T; row += kKvRowsAhead * stride) {
#pragma unroll
    for (int k = 0; k < kKvRowsAhead; ++k) load_row(row + (kKvRowsAhead + k) * stride, nxt[k]);
#pragma unroll
    for (int k = 0; k < kKvRowsAhead; ++k) store_row(row + k * stride, cur[k]);
#pragma unroll
    for (int k = 0; k < kKvRowsAhead; ++k)
#pragma unroll
      for (int j = 0; j < ND; ++j) cur[k][j] = nxt[k][j];
  }
}

int32_t launch_kv_quant(const void* x, int64_t T, int32_t d, const KvPos* pos, int32_t bits, void* codes, hipStream_t st) {
  if (T == 0) return RPTQ_OK;
  int cus = 0;
  if (int32_t s = device_compute_units(st, &cus)) return s;
  const int segs = (d + kKvTile - 1) / kKvTile;
  // Three workgroups of four waves per compute unit, rounded down: one round (25 KiB of LDS leave six resident), and enough
  // rows in flight.  us by that number 3 | 4 | 6 | 8 (the last a round and a third): 16384 x 12288 at 3 bits 97 | 98 | 106 | 106,
  // 32768 x 12288 190 | 191 | 217 | 206, 32768 x 5120 at 4 bits 78 | 81 | 80 | 80, 65536 x 5120 153 | 159 | 195 | 173, 65536 x 2048
  // 64 | 66 | 65 | 65.  But at least 32 rows per wave while that leaves two workgroups per compute unit (a workgroup reads
  // 16 KiB of table, as much as eight rows of its tile).  Every workgroup keeps one tile column.
  int64_t row_groups = static_cast<int64_t>(cus) * 3 / segs;
  row_groups = std::min<int64_t>(row_groups, std::max<int64_t>((T + 127) / 128, (static_cast<int64_t>(cus) * 2 + segs - 1) / segs));
  row_groups = std::min<int64_t>(std::max<int64_t>(row_groups, 1), (T + 3) / 4);
  const dim3 grid(static_cast<unsigned>(segs * row_groups)), block(256);
  const uint4* xp = static_cast<const uint4*>(x);
  uint8_t* cp = static_cast<uint8_t*>(codes);
  if (bits == 3) hipLaunchKernelGGL(kv_quant_kernel<3>, grid, block, 0, st, xp, T, d, pos, cp, segs, static_cast<int>(row_groups));
  else if (bits == 4) hipLaunchKernelGGL(kv_quant_kernel<4>, grid, block, 0, st, xp, T, d, pos, cp, segs, static_cast<int>(row_groups));
  else hipLaunchKernelGGL(kv_quant_kernel<8>, grid, block, 0, st, xp, T, d, pos, cp, segs, static_cast<int>(row_groups));
  RPTQ_HIP(hipGetLastError());
  return RPTQ_OK;
}

int32_t launch_kv_dequant(const void* codes, int64_t T, int32_t d, const KvPos* pos, int32_t bits, void* out, hipStream_t st) {
  if (T == 0) return RPTQ_OK;
  int cus = 0;
  if (int32_t s = device_compute_units(st, &cus)) return s;
  const int blocks_per_row = (d / 8 + 255) / 256;
  // eight workgroups per compute unit (20 KiB of LDS each: one round), but at least eight rows per thread while that leaves
  // two per compute unit (a workgroup reads 32 KiB of table, as much as it stores in eight rows)
  int64_t rows_par = (static_cast<int64_t>(cus) * 8 + blocks_per_row - 1) / blocks_per_row;
  rows_par = std::min<int64_t>(rows_par, std::max<int64_t>((T + 7) / 8, (static_cast<int64_t>(cus) * 2 + blocks_per_row - 1) / blocks_per_row));
  rows_par = std::min<int64_t>(std::max<int64_t>(rows_par, 1), T);
  const dim3 grid(static_cast<unsigned>(blocks_per_row * rows_par)), block(256);
  const uint8_t* cp = static_cast<const uint8_t*>(codes);
  uint16_t* op = static_cast<uint16_t*>(out);
  const bool stream = T * d * 2 > kKvStreamBytes;
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, st, cp, T, d, pos, op, blocks_per_row); };
  if (bits == 3) stream ? go(kv_dequant_kernel<3, true>) : go(kv_dequant_kernel<3, false>);
  else if (bits == 4) stream ? go(kv_dequant_kernel<4, true>) : go(kv_dequant_kernel<4, false>);
  else stream ? go(kv_dequant_kernel<8, true>) : go(kv_dequant_kernel<8, false>);
  RPTQ_HIP(hipGetLastError());
  return RPTQ_OK;
}

}  // namespace rptq
