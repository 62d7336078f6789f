// Compression primitives on the device (Section 3.2): group-wise linear quantization with float16
// scales, packing into the boundary format, and the two mirror maps (packed -> signed codes,
// packed -> fp32). These are the offline side of the path; they are written for exactness first. The usual group sizes and
// row widths have kernels bound by their fp32 reads or stores, the others simpler ones.
#include <type_traits>

#include "moeq_internal.h"

namespace moeq {
namespace {

// fp32 -> binary16 bits, round to nearest even, for a finite input >= 0.
// Normal results: the exponent is re-biased and the 13 dropped mantissa bits are rounded by adding 0xfff plus
// the lowest kept bit, one integer addition whose carry runs into the exponent where it must (so values that
// round up to 65536 come out as the infinity pattern 0x7c00). Results below 2^-14 are multiples of 2^-24:
// adding 0.5f puts the float's last mantissa bit exactly there, the addition itself rounds to nearest even
// (the wavefront's default mode), and the low bits of the sum are the binary16 pattern.
__device__ __forceinline__ uint32_t f32_to_f16_bits_rne(float f) {
  const uint32_t x = __float_as_uint(f);
  if (x >= 0x47800000u) return 0x7c00u;                            // 65536 and above
  if (x < 0x38800000u) return __float_as_uint(f + 0.5f) - 0x3f000000u;
  return (x + 0xc8000fffu + ((x >> 13) & 1u)) >> 13;               // 0xc8000000 = -(112 << 23): exponent bias 127 -> 15
}

// binary16 bits (finite, non-negative) -> fp32, exact.
__device__ __forceinline__ float f16_bits_to_f32(uint32_t h) {
  const uint32_t e = (h >> 10) & 0x1fu, m = h & 0x3ffu;
  if (e == 0) return (float)m * 5.9604644775390625e-08f;  // m * 2^-24, exact
  return __uint_as_float(((e + 112u) << 23) | (m << 13));
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}

// One group of `group` weights is handled by LPG lanes (a power of two <= 64); each lane walks the
// group's float4 slots with stride LPG, twice: once for the max magnitude, once to emit codes. For the group sizes
// that k_quantize_pack_once does not take (per-channel scales among them).
template <int BITS>
__global__ __launch_bounds__(256) void k_quantize_pack(const float* __restrict__ w, int64_t n_groups, int group,
                                                       int lpg, uint8_t* __restrict__ q, uint16_t* __restrict__ s) {
  constexpr int QMAX = (1 << (BITS - 1)) - 1;
  constexpr int OFF = 1 << (BITS - 1);
  const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t G = gtid / lpg;
  const int l = (int)(gtid % lpg);
  const bool live = G < n_groups;
  if (!live) G = n_groups - 1;  // keep the lane in the shuffles; it writes nothing
  const float4* wg = (const float4*)(w + G * group);
  const int n4 = group / 4;
  float a = 0.f;
  for (int i = l; i < n4; i += lpg) {
    const float4 v = wg[i];
    a = fmaxf(a, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
  }
  for (int off = lpg >> 1; off >= 1; off >>= 1) a = fmaxf(a, __shfl_xor(a, off, 64));
  uint32_t sh = 0;
  float sf = 0.f;
  if (a > 0.f) {
    const float s32 = __fdiv_rn(a, (float)QMAX);
    sh = f32_to_f16_bits_rne(s32);
    if (sh >= 0x7c00u) sh = 0x7bffu;
    else if (f16_bits_to_f32(sh) * (float)QMAX < a) sh += 1;  // next half up: the max element must not clamp
    if (sh >= 0x7c00u) sh = 0x7bffu;
    sf = f16_bits_to_f32(sh);
  }
  if (live && l == 0) s[G] = (uint16_t)sh;
  // 4 weights -> 4*BITS bits: one byte (INT2), two bytes (INT4), four bytes (INT8)
  uint8_t* qg = q + G * group * BITS / 8;
  for (int i = l; i < n4; i += lpg) {
    const float4 v = wg[i];
    const float e[4] = {v.x, v.y, v.z, v.w};
    uint32_t packed = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float r = 0.f;
      if (a > 0.f) {
        r = rintf(__fdiv_rn(e[j], sf));
        r = fminf(fmaxf(r, (float)-QMAX), (float)QMAX);
      }
      packed |= (uint32_t)((int)r + OFF) << (j * BITS);
    }
    if (!live) continue;
    if (BITS == 8) ((uint32_t*)qg)[i] = packed;
    else if (BITS == 4) ((uint16_t*)qg)[i] = (uint16_t)packed;
    else qg[i] = (uint8_t)packed;
  }
}

// The same for groups of 4 * n4 weights with n4 a power of two up to 64 (groups of 4 .. 256 weights, the usual ones):
// every float4 is read once, by the lane that also quantizes it. Weights, groups and codes are all linear in the
// float4's number i (group i / n4, codes 4 * BITS bits at i), so a wavefront reads 1 KB and writes 64 * BITS / 2
// bytes of consecutive addresses per step, and kQuantUnroll steps are loaded before the first is used.
// Bound by the fp32 reads and by the divisions: code = rint(w / scale) with the IEEE quotient. w times the
// approximate reciprocal is within 2.5 ulp (2^-21.5 relative, 4e-5 for magnitudes up to 128) of that quotient, so the
// two round to different integers only within 4e-5 of a half-integer; only float4s with such elements take the real division.
// A scale (division, rounding to binary16, the bump) is 40 instructions: lane j of a quad makes that of step j, not every lane all
// four. 14336 x 4096 weights at 4 bits: 43 us (6.2 TB/s); 52 with every lane's own scales and a branch per weight, 83-98 with two
// passes and a division per weight.
constexpr int kQuantUnroll = 4;
template <int BITS>
__global__ __launch_bounds__(256) void k_quantize_pack_once(const float* __restrict__ w, int64_t n_f4, int n4sh,
                                                            uint8_t* __restrict__ q, uint16_t* __restrict__ s) {
  using Code = typename std::conditional<BITS == 2, uint8_t, typename std::conditional<BITS == 4, uint16_t, uint32_t>::type>::type;
  typedef float float4_t __attribute__((ext_vector_type(4)));
  constexpr int QMAX = (1 << (BITS - 1)) - 1;
  constexpr int OFF = 1 << (BITS - 1);
  const int64_t base = (int64_t)blockIdx.x * (256 * kQuantUnroll) + threadIdx.x;
  const int n4 = 1 << n4sh;
  float4_t v[kQuantUnroll];
#pragma unroll
  for (int k = 0; k < kQuantUnroll; ++k) {      // (lanes past the end repeat the last weights; they write nothing)
    const int64_t i = base + k * 256 < n_f4 ? base + k * 256 : n_f4 - 1;
    v[k] = __builtin_nontemporal_load((const float4_t*)w + i);
  }
  // magnitude of every step's group, in all of its n4 lanes
  float am[kQuantUnroll];
#pragma unroll
  for (int k = 0; k < kQuantUnroll; ++k) {
    float a = fmaxf(fmaxf(fabsf(v[k].x), fabsf(v[k].y)), fmaxf(fabsf(v[k].z), fabsf(v[k].w)));
    a = fmaxf(a, 0.f);                           // four NaNs: the magnitude 0 that the running maximum starts from
    // maximum over the group's n4 lanes: the lane that differs in the lowest, second, ... bit of its number
    if (n4 > 1) a = fmaxf(a, dpp_f32<0xB1>(a));  // quad_perm [1,0,3,2]
    if (n4 > 2) a = fmaxf(a, dpp_f32<0x4E>(a));  // quad_perm [2,3,0,1]
    if (n4 > 4) a = fmaxf(a, dpp_f32<0x141>(a)); // mirror inside 8 lanes (whose quads agree by now)
    if (n4 > 8) a = fmaxf(a, dpp_f32<0x140>(a)); // mirror inside 16 lanes
    if (n4 > 16) a = fmaxf(a, __shfl_xor(a, 16, 64));
    if (n4 > 32) a = fmaxf(a, __shfl_xor(a, 32, 64));
    am[k] = a;
  }
  uint32_t shs[kQuantUnroll];
  float sfs[kQuantUnroll], invs[kQuantUnroll];
  auto scale_of = [&](float a, uint32_t& sh, float& sf, float& inv) __attribute__((always_inline)) {
    sh = 0;
    sf = 0.f;
    if (a > 0.f) {
      const float s32 = __fdiv_rn(a, (float)QMAX);
      sh = f32_to_f16_bits_rne(s32);
      if (sh >= 0x7c00u) sh = 0x7bffu;
      else if (f16_bits_to_f32(sh) * (float)QMAX < a) sh += 1;  // next half up: the max element must not clamp
      if (sh >= 0x7c00u) sh = 0x7bffu;
      sf = f16_bits_to_f32(sh);
    }
    inv = __builtin_amdgcn_rcpf(sf);             // (an all-zero group does not use it)
  };
  if (n4 >= 4) {                                 // quads lie inside groups: lane j of a quad makes the scale of step j for all four
    static_assert(kQuantUnroll == 4, "a step per lane of a quad");
    const int q4 = (int)threadIdx.x & 3;
    uint32_t sh;
    float sf, inv;
    scale_of(q4 == 0 ? am[0] : q4 == 1 ? am[1] : q4 == 2 ? am[2] : am[3], sh, sf, inv);
    const float shf = __uint_as_float(sh);
    sfs[0] = dpp_f32<0x00>(sf); sfs[1] = dpp_f32<0x55>(sf); sfs[2] = dpp_f32<0xAA>(sf); sfs[3] = dpp_f32<0xFF>(sf);
    invs[0] = dpp_f32<0x00>(inv); invs[1] = dpp_f32<0x55>(inv); invs[2] = dpp_f32<0xAA>(inv); invs[3] = dpp_f32<0xFF>(inv);
    shs[0] = __float_as_uint(dpp_f32<0x00>(shf)); shs[1] = __float_as_uint(dpp_f32<0x55>(shf));
    shs[2] = __float_as_uint(dpp_f32<0xAA>(shf)); shs[3] = __float_as_uint(dpp_f32<0xFF>(shf));
  } else {
#pragma unroll
    for (int k = 0; k < kQuantUnroll; ++k) scale_of(am[k], shs[k], sfs[k], invs[k]);
  }
#pragma unroll
  for (int k = 0; k < kQuantUnroll; ++k) {
    const int64_t i = base + k * 256;
    const bool live = i < n_f4;                  // whole groups: n_f4 is a multiple of n4 and n4 divides 64
    const float a = am[k], sf = sfs[k], inv = invs[k];
    float r[4];
    bool near = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float d = v[k][j] * inv;
      r[j] = rintf(d);
      near = near || fabsf(d - r[j]) > 0.49993f;
    }
    if (near) {                                  // one of the four: the IEEE quotients
#pragma unroll
      for (int j = 0; j < 4; ++j) r[j] = rintf(__fdiv_rn(v[k][j], sf));
    }
    uint32_t packed = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float c = a > 0.f ? fminf(fmaxf(r[j], (float)-QMAX), (float)QMAX) : 0.f;
      packed |= (uint32_t)((int)c + OFF) << (j * BITS);
    }
    if (live) {
      ((Code*)q)[i] = (Code)packed;
      if (((int)threadIdx.x & (n4 - 1)) == 0) s[i >> n4sh] = (uint16_t)shs[k];
    }
  }
}

__global__ __launch_bounds__(256) void k_unpack_codes(const uint8_t* __restrict__ q, int64_t n, int bits,
                                                      int8_t* __restrict__ codes) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // weight index (rows are whole bytes)
  if (i >= n) return;
  const int64_t bit = i * bits;
  const uint32_t u = (q[bit >> 3] >> (bit & 7)) & ((1u << bits) - 1u);
  codes[i] = (int8_t)((int)u - (1 << (bits - 1)));
}

// One weight per thread: any byte-aligned row length and any pointer alignment.
__global__ __launch_bounds__(256) void k_dequantize_any(const uint8_t* __restrict__ q, const uint16_t* __restrict__ s,
                                                        int64_t n, int64_t cols, int bits, int group,
                                                        float* __restrict__ w) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t bit = i * bits;
  const uint32_t u = (q[bit >> 3] >> (bit & 7)) & ((1u << bits) - 1u);
  const int64_t row = i / cols, col = i % cols;
  const float sc = f16_bits_to_f32(s[row * (cols / group) + col / group]);
  w[i] = sc * (float)((int)u - (1 << (bits - 1)));
}

// W^[row][col] = scale[row][col / group] * (code - 2^(bits-1)) as fp32 (Section 3.2: the decompression of
// an activated expert). Bound by the fp32 stores (16 bytes written per byte of 2-bit codes read). A thread takes
// four consecutive weights at a time, so that a wavefront's store is 1 KB of consecutive addresses; kDeqUnroll of
// them, a workgroup's width apart, are loaded before the first is stored. Groups divide the rows, so weight i has
// scale i / group whatever its row is (gsh = log2(group), or -1). The form with one 32-bit word of codes per
// thread, whose stores lay 64 / 32 / 16 bytes apart, took 75 us for a 14336 x 4096 matrix of 2-bit codes (3.3 TB/s
// of codes, scales and weights); this one takes 37.5 us (6.7 TB/s).
constexpr int kDeqUnroll = 4;
template <int BITS>
__global__ __launch_bounds__(256) void k_dequantize(const uint8_t* __restrict__ q, const uint16_t* __restrict__ s,
                                                    int64_t n4, uint32_t group, int gsh, float* __restrict__ w) {
  using Code = typename std::conditional<BITS == 2, uint8_t, typename std::conditional<BITS == 4, uint16_t, uint32_t>::type>::type;
  typedef float float4_t __attribute__((ext_vector_type(4)));
  constexpr uint32_t MASK = (1u << BITS) - 1u;
  constexpr int OFF = 1 << (BITS - 1);
  const int64_t base = (int64_t)blockIdx.x * (256 * kDeqUnroll) + threadIdx.x;    // in units of four weights
  uint32_t u[kDeqUnroll];
  uint32_t sh[kDeqUnroll][4];
  const bool one = group % 4 == 0;                  // the four weights share a scale
  auto scale_of = [&](int64_t i) { return (uint32_t)s[gsh >= 0 ? i >> gsh : i / group]; };
#pragma unroll
  for (int k = 0; k < kDeqUnroll; ++k) {
    const int64_t i = base + k * 256 < n4 ? base + k * 256 : n4 - 1;
    u[k] = ((const Code*)q)[i];
    sh[k][0] = scale_of(4 * i);
    if (!one)
      for (int e = 1; e < 4; ++e) sh[k][e] = scale_of(4 * i + e);
  }
#pragma unroll
  for (int k = 0; k < kDeqUnroll; ++k) {
    float4_t v;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = f16_bits_to_f32(one ? sh[k][0] : sh[k][e]) * (float)((int)((u[k] >> (e * BITS)) & MASK) - OFF);
    if (base + k * 256 < n4) __builtin_nontemporal_store(v, (float4_t*)w + (base + k * 256));
  }
}

}  // namespace

hipError_t launch_quantize_pack(const float* w, int64_t rows, int64_t cols, int bits, int group, uint8_t* q,
                                uint16_t* s, hipStream_t st) {
  const int64_t n_groups = rows * (cols / group);
  if (group <= 256 && (group & (group - 1)) == 0) {      // (a multiple of four: checked by the entry point)
    const int n4sh = __builtin_ctz((unsigned)(group / 4));
    const int64_t n_f4 = n_groups * (group / 4), nb = (n_f4 + 256 * kQuantUnroll - 1) / (256 * kQuantUnroll);
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 g1((unsigned)nb), b1(256);
    switch (bits) {
      case 2: hipLaunchKernelGGL(k_quantize_pack_once<2>, g1, b1, 0, st, w, n_f4, n4sh, q, s); break;
      case 4: hipLaunchKernelGGL(k_quantize_pack_once<4>, g1, b1, 0, st, w, n_f4, n4sh, q, s); break;
      default: hipLaunchKernelGGL(k_quantize_pack_once<8>, g1, b1, 0, st, w, n_f4, n4sh, q, s); break;
    }
    return hipGetLastError();
  }
  int lpg = 1;
  while (lpg < 64 && lpg * 2 <= group / 4) lpg *= 2;
  const int64_t threads = n_groups * lpg;
  const int64_t blocks = (threads + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(256);
  switch (bits) {
    case 2: hipLaunchKernelGGL(k_quantize_pack<2>, grid, block, 0, st, w, n_groups, group, lpg, q, s); break;
    case 4: hipLaunchKernelGGL(k_quantize_pack<4>, grid, block, 0, st, w, n_groups, group, lpg, q, s); break;
    default: hipLaunchKernelGGL(k_quantize_pack<8>, grid, block, 0, st, w, n_groups, group, lpg, q, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_unpack_codes(const uint8_t* q, int64_t rows, int64_t cols, int bits, int8_t* codes,
                               hipStream_t st) {
  const int64_t n = rows * cols, blocks = (n + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_unpack_codes, dim3((unsigned)blocks), dim3(256), 0, st, q, n, bits, codes);
  return hipGetLastError();
}

hipError_t launch_dequantize(const uint8_t* q, const uint16_t* s, int64_t rows, int64_t cols, int bits, int group,
                             float* w, hipStream_t st) {
  if ((cols * bits) % 32 || ((uintptr_t)q & 3u) || ((uintptr_t)w & 15u)) {
    const int64_t n = rows * cols, nb = (n + 255) / 256;
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_dequantize_any, dim3((unsigned)nb), dim3(256), 0, st, q, s, n, cols, bits, group, w);
    return hipGetLastError();
  }
  // whole words of codes per row: the number of weights is a multiple of four, and every thread's codes are aligned
  const int64_t n4 = rows * cols / 4, blocks = (n4 + 256 * kDeqUnroll - 1) / (256 * kDeqUnroll);
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(256);
  const int gsh = (group & (group - 1)) == 0 ? __builtin_ctz((unsigned)group) : -1;
  switch (bits) {
    case 2: hipLaunchKernelGGL(k_dequantize<2>, grid, block, 0, st, q, s, n4, (uint32_t)group, gsh, w); break;
    case 4: hipLaunchKernelGGL(k_dequantize<4>, grid, block, 0, st, q, s, n4, (uint32_t)group, gsh, w); break;
    default: hipLaunchKernelGGL(k_dequantize<8>, grid, block, 0, st, q, s, n4, (uint32_t)group, gsh, w); break;
  }
  return hipGetLastError();
}

}  // namespace moeq
