// Decode calls on layers whose work is small beside the latency of a launch: a workgroup's share of an expert is a few KB, so
// its life is a chain of memory round trips and of instructions executed once, not a stream. The kernels here keep both short:
//   - what a workgroup needs of an expert are contiguous blocks in memory (the slice's rows of W_in, its word columns of W_out),
//     fetched with linear copies straight to LDS and requested together as soon as the expert is known: one round trip for both
//     phases, no registers held, no address arithmetic; a second choice's are requested behind phase 1 of the first;
//   - the arithmetic is fp32 on the codes as they are converted (v_cvt_f32_ubyte): the activations enter as fp32, so there is no
//     binary16 pair order to bring them into and no pass over LDS per bitwidth;
//   - a thread keeps one piece (16 or 32 columns) of the rows and walks the rows, that piece's activations in registers; sixteen
//     lanes fold a row's partial sums.
// The routing's source is a template parameter: with all of them in one kernel every instance spills scalar registers. Those that
// select from the router kernel's logits still spill 40 to 67 of them (they hold the selection of up to 64, 128 and 1024 experts),
// the others 0 to 11.
// k_small_in, k_small_out: the two phases on the canonical layout, where a workgroup's rows are one block.
// k_small_cols: the whole layer for one (slice of d_ff, token), W_out in word columns (partial output vectors, summed by
// k_reduce_partials). Time stamps of a workgroup on a 64-expert Switch-base layer (us from its start): routed 1.0, all requested
// 1.9, blocks there 2.1, phase 1 2.8, h 3.2, phase 2 3.9, end 4.0; k_moe_decode_vec, which it replaces there: 1.6, 3.8, 5.0,
// 7.5 (one wavefront has rows, three have none), 8.9, 10.4, 10.7. The step of six layers, replayed eight times, 932 -> 620 us;
// error against 64 bits 3e-4 -> 7e-7 (binary16 activations before). What bounds it now: three launches of 1.3-1.6 us with
// nothing in them, and instructions that two wavefronts per SIMD issue one after the other.
#include <algorithm>

#include <hip/hip_ext.h>

#include "decode_core.h"
#include "small_split.h"

namespace moeq {
namespace {

constexpr int kSmInlineMaxE = 64, kSmMaxSegs = 8;
constexpr int kSmRouteBytes = kSmInlineMaxE * kSmMaxSegs * 4;    // k_small_cols: of the routing, in the place of the partial sums
constexpr size_t kSmLds = 150 * 1024, kSmLdsTwo = 80 * 1024;     // of a compute unit's 160 KB: one workgroup, two

__host__ __device__ inline int pad_to(int v, int a) { return (v + a - 1) / a * a; }

// Copies `bytes` (a multiple of 16) of contiguous memory to LDS, a wavefront 1 KB at a time; the region is padded to whole KB
// (lanes past the end repeat the last 16 bytes).
template <int NT>
__device__ __forceinline__ void fetch_block(const uint8_t* g, int bytes, uint32_t lds, int wave, int lane) {
  for (int o = wave * 1024; o < bytes; o += NT * 16) {
    const uint32_t off = (uint32_t)min(o + lane * 16, bytes - 16);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(g), "s"(lds + (uint32_t)o) : "memory");
  }
}
__device__ __forceinline__ void fetch_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Activations in LDS: fp32, 16-byte items, item i at i ^ ((i >> 4) & 15). Lanes that read chunk after chunk (16, 32 or 64
// columns apart) then touch different banks.
__device__ __forceinline__ int x_slot(int i) { return i ^ ((i >> 4) & 15); }

// U items per thread and pass, requested together; returns the thread's largest magnitude. XS[b] = 2^-8 times the sum of the
// columns 16 b .. 16 b + 15 (2^-8: the sum of sixteen stays in range where the values do).
template <int NT, int U>
__device__ __forceinline__ float stage_raw(const void* x, bool bf16, int n4, int tid, float4* XL, float* XS) {
  float m = 0.f;
  for (int i0 = tid; i0 < n4; i0 += U * NT) {                // (n4 is a multiple of 4: whole quads of lanes stay together)
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * NT;
      v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (i < n4) {
        if (bf16) {
          const uint2 b = ((const uint2*)x)[i];
          v[u] = make_float4(bf16_bits_to_f32(b.x & 0xffffu), bf16_bits_to_f32(b.x >> 16), bf16_bits_to_f32(b.y & 0xffffu), bf16_bits_to_f32(b.y >> 16));
        } else {
          v[u] = ((const float4*)x)[i];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * NT;
      float s = ((v[u].x + v[u].y) * 0.00390625f) + ((v[u].z + v[u].w) * 0.00390625f);
      s += dpp<kDppXor1>(s);
      s += dpp<kDppXor2>(s);
      if (i < n4) {
        XL[x_slot(i)] = v[u];
        if ((i & 3) == 0) XS[i >> 2] = s;
      }
      m = fmaxf(fmaxf(m, fmaxf(fabsf(v[u].x), fabsf(v[u].y))), fmaxf(fabsf(v[u].z), fabsf(v[u].w)));    // a NaN is skipped
    }
  }
  return m;
}
// The exponent that an activation vector of largest magnitude m is scaled by ahead of the products: none where fp32 has room
// for them anyway, else norm_exponent.
__device__ __forceinline__ int safe_exponent(float m) { return m > 0x1p60f || m < 0x1p-60f ? norm_exponent(m) : 0; }
template <int NT>
__device__ __forceinline__ float red_max(const float* red) {
  float M = 0.f;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) M = fmaxf(M, red[w]);
  return M;
}

__device__ __forceinline__ float ubyte(uint32_t w, int i) { return (float)((w >> (8 * i)) & 0xffu); }

// acc += sum of the codes u of a word (32 / BITS of them) times x.
template <int BITS>
__device__ __forceinline__ float word_fma(uint32_t w, const float* x, float acc) {
  if constexpr (BITS == 8) {
#pragma unroll
    for (int b = 0; b < 4; ++b) acc = fmaf(ubyte(w, b), x[b], acc);
  } else if constexpr (BITS == 4) {
    const uint32_t lo = w & 0x0f0f0f0fu, hi = (w >> 4) & 0x0f0f0f0fu;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      acc = fmaf(ubyte(lo, b), x[2 * b], acc);
      acc = fmaf(ubyte(hi, b), x[2 * b + 1], acc);
    }
  } else {
    const uint32_t f[4] = {w & 0x03030303u, (w >> 2) & 0x03030303u, (w >> 4) & 0x03030303u, (w >> 6) & 0x03030303u};
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = fmaf(ubyte(f[j], b), x[4 * b + j], acc);
  }
  return acc;
}

// A thread's piece of a row: 32 columns (8-bit codes: 16), two words of 2-bit codes, four of the others. It has one scale.
template <int BITS>
struct Piece {
  static constexpr int COLS = BITS == 8 ? 16 : 32, WORDS = COLS * BITS / 32;
};
__host__ __device__ inline int row_pieces(int cols, int bits) { return bits == 8 ? cols / 16 : cols / 32; }

// red[m][r * Cr + c] = the sum of row r over a thread's pieces, r < rows, for NM matrices whose rows lie in LDS (codes at
// WL + m * wl_stride, scales at SL + m * sl_stride as in memory). Cr = min(pieces per row, threads).
template <int NT, int BITS, int NM>
__device__ __forceinline__ void rows_dot(const uint8_t* WL, int wl_stride, const uint16_t* SL, int sl_stride, const float4* XL, const float* XS,
                                         int cols, int group, int gsh, int ng, int rows, float dn, int tid, float* red, int red_stride) {
  constexpr int COLS = Piece<BITS>::COLS, WORDS = Piece<BITS>::WORDS, Q = COLS / 4;
  const int C = cols / COLS;
  int rs = 0, c0 = tid, step = 1, Cr = NT;
  if (C < NT) {
    rs = small_div(tid, C);
    c0 = tid - rs * C;
    step = small_div(NT, C);
    Cr = C;
  }
  if (rs >= step) return;
  for (int c = c0; c < C; c += NT) {
    float x[COLS];
    const int i0 = c * Q, base = i0 & ~15, low = (i0 & 15) ^ ((i0 >> 4) & 15);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float4 v = XL[base + (low ^ q)];
      x[4 * q] = v.x; x[4 * q + 1] = v.y; x[4 * q + 2] = v.z; x[4 * q + 3] = v.w;
    }
    if (dn != 1.0f) {
#pragma unroll
      for (int i = 0; i < COLS; ++i) x[i] *= dn;
    }
    const float k0 = -256.0f * Fmt<BITS>::OFF * dn * (BITS == 8 ? XS[c] : XS[2 * c] + XS[2 * c + 1]);      // the offset term
    const int g = (int)div_group((uint32_t)(c * COLS), group, gsh);
#pragma unroll 1
    for (int r = rs; r < rows; r += step) {
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        uint32_t w[WORDS];
        const uint8_t* src = WL + m * wl_stride + (r * C + c) * (WORDS * 4);
        if constexpr (WORDS == 4) {
          const uint4 t = *(const uint4*)src;
          w[0] = t.x; w[1] = t.y; w[WORDS - 2] = t.z; w[WORDS - 1] = t.w;
        } else {
          const uint2 t = *(const uint2*)src;
          w[0] = t.x; w[1] = t.y;
        }
        float a = k0, b = 0.f;       // two chains
#pragma unroll
        for (int i = 0; i < WORDS; i += 2) {
          a = word_fma<BITS>(w[i], x + i * (32 / BITS), a);
          b = word_fma<BITS>(w[i + 1], x + (i + 1) * (32 / BITS), b);
        }
        float v = f16_bits_to_f32(SL[m * sl_stride + r * ng + g]) * (a + b);
        float* o = red + m * red_stride + r * Cr + c0;
        if (c != c0) v += *o;
        *o = v;
      }
    }
  }
}

// fn(r, sums of row r) for every row, by one lane of the sixteen that fold it.
template <int NT, int NM, typename Fn>
__device__ __forceinline__ void rows_fold(const float* red, int red_stride, int Cr, int rows, int tid, Fn fn) {
  const int l = tid & 15;
  for (int r = tid >> 4; r < rows; r += NT / 16) {
    float t[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      t[m] = 0.f;
      for (int i = l; i < Cr; i += 16) t[m] += red[m * red_stride + r * Cr + i];
      t[m] += dpp<kDppXor1>(t[m]);
      t[m] += dpp<kDppXor2>(t[m]);
      t[m] += dpp<kDppRor4>(t[m]);
      t[m] += dpp<kDppRor8>(t[m]);
    }
    if (l == 0) fn(r, t);
  }
}

// n2 pairs of binary16 scales, requested into registers and stored to LDS behind the wait (a direct copy would be 256 bytes an
// instruction, and scales need be aligned to two bytes only).
constexpr int kSmScales = 2;                 // pairs per thread held in registers; the rest goes through a loop
struct ScaleRegs { uint32_t v[kSmScales]; };
template <int NT>
__device__ __forceinline__ void scales_issue(ScaleRegs& S, const uint8_t* s, int n2, int tid) {
#pragma unroll
  for (int u = 0; u < kSmScales; ++u) S.v[u] = tid + u * NT < n2 ? gload_u32(s + (uint32_t)(tid + u * NT) * 4u) : 0u;
}
template <int NT>
__device__ __forceinline__ void scales_store(const ScaleRegs& S, const uint8_t* s, int n2, int tid, uint32_t* SL) {
#pragma unroll
  for (int u = 0; u < kSmScales; ++u)
    if (tid + u * NT < n2) SL[tid + u * NT] = S.v[u];
  for (int i = tid + kSmScales * NT; i < n2; i += NT) SL[i] = gload_u32(s + (uint32_t)i * 4u);
}

__device__ __forceinline__ float silu(float a) { return a / (1.0f + __expf(-a)); }

// The record of expert e (the same in every lane), as uniform values.
template <bool SWIGLU>
__device__ __forceinline__ DevExpert uniform_record(const DevExpert* t) {
  DevExpert ex;
  ex.q_in = uniform_ptr(t->q_in); ex.s_in = uniform_ptr(t->s_in);
  if constexpr (SWIGLU) { ex.q_gate = uniform_ptr(t->q_gate); ex.s_gate = uniform_ptr(t->s_gate); }
  ex.q_out = uniform_ptr(t->q_out); ex.s_out = uniform_ptr(t->s_out);
  ex.bits = __builtin_amdgcn_readfirstlane(t->bits);
  return ex;
}

// ---------------------------------------------------------------------------------------------
// One (slice of SW columns of d_ff, token).
enum SmallMode { kFromLogits, kInline, kGiven };     // routing: from the router kernel's logits, router evaluated here, given
struct SmallCols {
  const DevExpert* table;
  const void* x;
  const float* logits;        // kFromLogits: [T][E]
  const float* Wr;            // kInline
  const float* bias;
  const int32_t* route_idx;   // kGiven: [T][k], or null: fixed_expert for every token
  const float* route_gate;    // ... and the gates, or null (= 1)
  int32_t* idx_out;           // (not kGiven) [T][k] or null
  float* gate_out;
  float* part;
  int32_t fixed_expert, d, E, k, renorm, bf16, SW, n_slices, group, gsh, ng, group_out;
  // LDS: activations, their sums, h, partial sums, scales of W_in [, W_gate], codes of W_in [, W_gate], of W_out (two of these
  // with several choices)
  int32_t xs_off, h_off, red_off, red_stride, si_off, si_stride, wi_off, w_stride, lds;
};
constexpr int kSmThreads = 512;          // (small_split.h counts on them)

// Output rows RPT tid .. over the slice: acc = sum of the codes u times h (dn).
template <int BITS, int RPT>
__device__ __forceinline__ void slice_out(const uint8_t* WO, const float* HF, int SW, int d, int r0, float dn, float (&acc)[RPT]) {
  constexpr int CPD = 32 / BITS, WPB = 16 / CPD;      // words per 16 columns
#pragma unroll
  for (int r = 0; r < RPT; ++r) acc[r] = 0.f;
#pragma unroll 1
  for (int c = 0; c < SW; c += 16) {
    float hv[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = *(const float4*)(HF + c + 4 * q);
      hv[4 * q] = v.x; hv[4 * q + 1] = v.y; hv[4 * q + 2] = v.z; hv[4 * q + 3] = v.w;
    }
    if (dn != 1.0f) {
#pragma unroll
      for (int i = 0; i < 16; ++i) hv[i] *= dn;
    }
#pragma unroll
    for (int w = 0; w < WPB; ++w) {
      uint32_t v[RPT];
      const uint8_t* src = WO + ((c / CPD + w) * d + r0) * 4;
      if constexpr (RPT == 4) {
        const uint4 t = *(const uint4*)src;
        v[0] = t.x; v[1] = t.y; v[RPT - 2] = t.z; v[RPT - 1] = t.w;
      } else {
        const uint2 t = *(const uint2*)src;
        v[0] = t.x; v[1] = t.y;
      }
#pragma unroll
      for (int r = 0; r < RPT; ++r) acc[r] = word_fma<BITS>(v[r], hv + w * CPD, acc[r]);
    }
  }
}

template <bool SWIGLU, int MODE, int RPT>
__global__ __launch_bounds__(kSmThreads, 4) void k_small_cols(SmallCols P) {
  extern __shared__ uint4 smem4[];
  __shared__ int sel_ew[kSmThreads / 64][8];
  __shared__ float sel_gw[kSmThreads / 64][8];
  constexpr int NM = SWIGLU ? 2 : 1, NT = kSmThreads;
  const int d = P.d, E = P.E, k = P.k, SW = P.SW, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int token = blockIdx.y;
  // each XCD gets a contiguous range of slices
  const int slice = (P.n_slices & 7) == 0 ? (int)((blockIdx.x & 7u) * (P.n_slices >> 3) + (blockIdx.x >> 3)) : (int)blockIdx.x;
  char* smem = (char*)smem4;
  float4* XL = (float4*)smem;
  float* XS = (float*)(smem + P.xs_off);
  float* HF = (float*)(smem + P.h_off);
  float* red = (float*)(smem + P.red_off);
  // Two workgroups share a compute unit where the launch asks for half of its LDS (small_cols_fits): what the routing needs lies
  // where the partial sums and h come later, behind the loop's first barrier or its second. (2 KB beside it: 8-bit experts of
  // 1024 x 8192, 3 tokens 27.0 us, now 21.4, k_moe_decode_vec 23.7.) The choices of more than 64 experts stay apart: in the place
  // of the partial sums they cost the scalar registers of every call with logits (3 % of one with several choices).
  float* rpart = red;                                      // kInline: router sums, unit u = e * n_seg + seg
  float* red_m = HF;                                       // a wavefront's largest activation
  static_assert(NT / 64 <= 16, "a slice has at least 16 columns of h");
  const uint32_t lds0 = (uint32_t)(uintptr_t)(MOEQ_LDS char*)smem;
  const char* xt = (const char*)P.x + (size_t)token * d * (P.bf16 ? 2 : 4);

  // requests that depend on nothing but the inputs: in lane e the record of expert e (up to 64 experts)
  const bool lane_recs = MODE != kGiven && E <= 64;
  uint4 rec[4];
  if constexpr (MODE != kGiven) {
    const uint4* src = (const uint4*)(P.table + (lane_recs ? min(lane, E - 1) : 0));
    rec[0] = src[0];
    if constexpr (SWIGLU) rec[1] = src[1];
    rec[2] = src[2];
    rec[3].x = src[3].x;
  }
  auto stage_x = [&]() __attribute__((always_inline)) {
    const float m = wave_max(stage_raw<NT, 1>(xt, P.bf16 != 0, d / 4, tid, XL, XS));
    if (lane == 0) red_m[wave] = m;
  };
  int n_seg = (d + 2047) / 2048;
  if constexpr (MODE == kInline) {           // unit = (expert, segment of columns), as in k_moe_decode_wide
    constexpr int NW = 4;                    // (its order of sums is that of four wavefronts)
    while (n_seg * 2 <= kSmMaxSegs && E * n_seg * 2 <= NW && d >= n_seg * 2 * 256) n_seg *= 2;
    const int seg_cols = (small_div(d + n_seg - 1, n_seg) + 255) / 256 * 256;
    for (int u = wave; u < E * n_seg; u += NT / 64) {
      const int e = small_div(u, n_seg), seg = u - e * n_seg;
      const float* wr = P.Wr + (size_t)e * d;
      const int c_end = min(d, (seg + 1) * seg_cols);
      float4 w[8], v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int i = seg * seg_cols + q * 256 + lane * 4;
        w[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        v[q] = w[q];
        if (i < c_end) {
          w[q] = *(const float4*)(wr + i);
          if (P.bf16) {
            const uint2 b = *(const uint2*)((const uint16_t*)xt + i);
            v[q] = make_float4(bf16_bits_to_f32(b.x & 0xffffu), bf16_bits_to_f32(b.x >> 16), bf16_bits_to_f32(b.y & 0xffffu), bf16_bits_to_f32(b.y >> 16));
          } else {
            v[q] = *(const float4*)((const float*)xt + i);
          }
        }
      }
      float acc = 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        acc = fmaf(w[q].x, v[q].x, acc); acc = fmaf(w[q].y, v[q].y, acc);
        acc = fmaf(w[q].z, v[q].z, acc); acc = fmaf(w[q].w, v[q].w, acc);
      }
      acc = wave_sum(acc);
      if (lane == 0) rpart[u] = acc;
    }
    stage_x();
    __syncthreads();             // rpart is complete
  }

  // the routing, by every wavefront for itself: lane j < k gets choice j
  int my_e = 0;
  float my_g = 1.0f;
  if constexpr (MODE == kGiven) {
    if (P.route_idx) my_e = P.route_idx[(size_t)token * k + min(lane, k - 1)];
    else my_e = P.fixed_expert;
    if (P.route_gate) my_g = P.route_gate[(size_t)token * k + min(lane, k - 1)];
  } else if (MODE == kInline || lane_recs) {
    float v = -INFINITY;
    if (lane < E) {
      if constexpr (MODE == kInline) {
        v = 0.f;
        for (int sg = 0; sg < n_seg; ++sg) v += rpart[lane * n_seg + sg];
        v += P.bias ? P.bias[lane] : 0.f;
      } else {
        v = P.logits[(size_t)token * E + lane];
      }
    }
    const Top64 t = topk64(v, E, k, P.renorm, lane);
    my_e = t.e;
    my_g = t.gate;
  } else {
    topk_from_logits(P.logits + (size_t)token * E, E, k, P.renorm, lane, sel_ew[wave], sel_gw[wave], nullptr);
    my_e = sel_ew[wave][min(lane, k - 1)];
    my_g = sel_gw[wave][min(lane, k - 1)];
  }
  // the indices become addresses of expert records: whatever produced them, they stay inside the table
  my_e = min(max(my_e, 0), E - 1);
  if (MODE != kGiven && blockIdx.x == 0 && tid < k) {
    if (P.idx_out) P.idx_out[(size_t)token * k + tid] = my_e;
    if (P.gate_out) P.gate_out[(size_t)token * k + tid] = my_g;
  }

  const int r0 = min(tid * RPT, d - RPT);            // the thread's output rows
  float Y[RPT];
#pragma unroll
  for (int r = 0; r < RPT; ++r) Y[r] = 0.f;
  // step j: phase 1 of choice j, the requests of choice j + 1, phase 2 of choice j (its block of W_out lies in one of two places)
  int bits = 0, next_bits = 0, n2 = SW * P.ng / 2;
  const uint8_t *s0 = nullptr, *s1 = nullptr;
  ScaleRegs S[NM];
  uint2 sco = make_uint2(0u, 0u), next_sco = sco;
  float up = 1.0f, dn = 1.0f;
  const uint8_t* WI = (const uint8_t*)smem + P.wi_off;
  uint16_t* SI = (uint16_t*)(smem + P.si_off);
#pragma unroll 1
  for (int j = -1; j < k; ++j) {
    if (j >= 0) {
      bits = next_bits;
      sco = next_sco;
      fetch_wait();
      scales_store<NT>(S[0], s0, n2, tid, (uint32_t*)SI);
      if constexpr (SWIGLU) scales_store<NT>(S[NM - 1], s1, n2, tid, (uint32_t*)(SI + P.si_stride));
      __syncthreads();           // blocks, scales and activations are complete
      if (j == 0) {
        const int e = safe_exponent(red_max<NT>(red_m));
        dn = pow2f(-e);
        up = pow2f(e);
      }
      switch (bits) {
        case 2: rows_dot<NT, 2, NM>(WI, P.w_stride, SI, P.si_stride, XL, XS, d, P.group, P.gsh, P.ng, SW, dn, tid, red, P.red_stride); break;
        case 4: rows_dot<NT, 4, NM>(WI, P.w_stride, SI, P.si_stride, XL, XS, d, P.group, P.gsh, P.ng, SW, dn, tid, red, P.red_stride); break;
        default: rows_dot<NT, 8, NM>(WI, P.w_stride, SI, P.si_stride, XL, XS, d, P.group, P.gsh, P.ng, SW, dn, tid, red, P.red_stride); break;
      }
      __syncthreads();           // partial sums are complete, the blocks of W_in are used up
    }
    if (j + 1 < k) {
      const int e = __builtin_amdgcn_readlane(my_e, j + 1);
      DevExpert ex;
      if (lane_recs) {
        auto rl = [&](uint32_t v) __attribute__((always_inline)) { return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)v, e); };
        ex.q_in = (const uint8_t*)(rl(rec[0].x) | rl(rec[0].y) << 32);
        ex.s_in = (const uint16_t*)(rl(rec[0].z) | rl(rec[0].w) << 32);
        if constexpr (SWIGLU) {
          ex.q_gate = (const uint8_t*)(rl(rec[1].x) | rl(rec[1].y) << 32);
          ex.s_gate = (const uint16_t*)(rl(rec[1].z) | rl(rec[1].w) << 32);
        }
        ex.q_out = (const uint8_t*)(rl(rec[2].x) | rl(rec[2].y) << 32);
        ex.s_out = (const uint16_t*)(rl(rec[2].z) | rl(rec[2].w) << 32);
        ex.bits = (int)rl(rec[3].x);
      } else {
        ex = uniform_record<SWIGLU>(P.table + e);
      }
      next_bits = ex.bits;
      const int block = SW * ((d >> 3) * ex.bits);             // a slice's bytes of either matrix
      s0 = (const uint8_t*)ex.s_in + (size_t)slice * n2 * 4;
      scales_issue<NT>(S[0], s0, n2, tid);
      if constexpr (SWIGLU) {
        s1 = (const uint8_t*)ex.s_gate + (size_t)slice * n2 * 4;
        scales_issue<NT>(S[NM - 1], s1, n2, tid);
      }
      const uint8_t* so = (const uint8_t*)ex.s_out + (size_t)small_div(slice * SW, P.group_out) * d * 2 + (uint32_t)r0 * 2u;
      if constexpr (RPT == 4) next_sco = gload_u32x2(so);
      else next_sco.x = gload_u32(so);
      fetch_block<NT>(ex.q_in + (size_t)slice * block, block, lds0 + P.wi_off, wave, lane);
      if constexpr (SWIGLU) fetch_block<NT>(ex.q_gate + (size_t)slice * block, block, lds0 + P.wi_off + P.w_stride, wave, lane);
      fetch_block<NT>(ex.q_out + (size_t)slice * block, block, lds0 + P.wi_off + (NM + ((j + 1) & 1)) * P.w_stride, wave, lane);
    }
    if (j < 0) {
      if constexpr (MODE != kInline) stage_x();
      continue;
    }
    rows_fold<NT, NM>(red, P.red_stride, min(row_pieces(d, bits), NT), SW, tid, [&](int r, const float (&t)[NM]) __attribute__((always_inline)) {
      const float a = t[0] * up;
      if constexpr (SWIGLU) HF[r] = silu(a) * (t[NM - 1] * up);
      else HF[r] = fmaxf(a, 0.f);
    });
    __syncthreads();             // h of the slice is complete
    float hm = 0.f, hs = 0.f;
    for (int c = lane; c < SW; c += 64) {
      const float v = HF[c];
      hm = fmaxf(hm, fabsf(v));
      hs = fmaf(v, 0.00390625f, hs);
    }
    const int eh = safe_exponent(wave_max(hm));
    hs = wave_sum(hs);
    const float dh = pow2f(-eh), gate = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, my_g), j)) * pow2f(eh);
    const uint8_t* WO = WI + (NM + (j & 1)) * P.w_stride;
    float acc[RPT];
    switch (bits) {
      case 2: slice_out<2, RPT>(WO, HF, SW, d, r0, dh, acc); break;
      case 4: slice_out<4, RPT>(WO, HF, SW, d, r0, dh, acc); break;
      default: slice_out<8, RPT>(WO, HF, SW, d, r0, dh, acc); break;
    }
    const float off = hs * dh * (float)(-(128 << bits));                // -2^(bits - 1) * 2^8
    Y[0] = fmaf(f16_bits_to_f32(sco.x & 0xffffu) * gate, acc[0] + off, Y[0]);
    Y[1] = fmaf(f16_bits_to_f32(sco.x >> 16) * gate, acc[1] + off, Y[1]);
    if constexpr (RPT == 4) {
      Y[RPT - 2] = fmaf(f16_bits_to_f32(sco.y & 0xffffu) * gate, acc[RPT - 2] + off, Y[RPT - 2]);
      Y[RPT - 1] = fmaf(f16_bits_to_f32(sco.y >> 16) * gate, acc[RPT - 1] + off, Y[RPT - 1]);
    }
  }
  float* out = P.part + ((size_t)token * P.n_slices + slice) * d;
  if (tid < d / RPT) {
    if constexpr (RPT == 4) *(float4*)(out + r0) = make_float4(Y[0], Y[1], Y[RPT - 2], Y[RPT - 1]);
    else *(float2*)(out + r0) = make_float2(Y[0], Y[1]);
  }
}

// ---------------------------------------------------------------------------------------------
// The canonical layout, one phase a kernel: R consecutive rows of W_in (and W_gate) against x, of W_out against the h of every
// choice. A workgroup's rows are taken in passes of up to `room` bytes of LDS a matrix; the next pass is requested as soon as
// the one before has been multiplied. (Passes of 8 KB in a ring of four, with waits that count a wavefront's copies, multiply
// while they arrive, but their barriers and the loop around them cost more: 8 tokens on the layer below 23.2 -> 30.3 us.)
// Time stamps of 8 tokens on a 128-expert Switch-large layer (us from the start of a kernel, medians): k_small_in routed 1, blocks
// there 3.6, multiplied 5.5, end 6; k_small_out requested 1.3, there 3.2, multiplied 5.6, end 6.3. Bytes take 2.5 of either.
struct SmallRows {
  const DevExpert* table;
  const float* logits;        // k_small_in, kFromLogits: [T][E]
  int32_t* idx;               // routing: written (kFromLogits) or read (kGiven), [T][k]; null: fixed_expert for every token
  float* gate;                // k_small_out: null = 1
  DevExpert* sel_tab;         // the chosen experts' records, [T][k]: k_small_in writes, k_small_out reads (unless fixed)
  const void* act;            // x [T][cols] in the layer's dtype / h [T][k][cols]
  float* out;                 // h [T][k][rows] / y [T][rows]
  int32_t fixed_expert, cols, rows, E, k, renorm, bf16, accumulate, R, group, gsh, ng;
  int32_t room, xs_off, y_off, red_off, red_stride, si_off, si_stride, w_off, lds;
};
constexpr int kRowsRoom = 32768, kRowsMaxCols = kRowsRoom / 4;      // (four rows of 8-bit codes fit; two matrices share the room)

__host__ __device__ inline int pass_rows(int R, int room, int row_bytes) {
  const int n = (int)((unsigned)room / (unsigned)row_bytes) & ~3;
  return R < n ? R : n;
}

// PHASE 0 has one choice, whose activations are staged already; PHASE 1 the token's. record(j), act(j): of choice j. epi(j, row,
// sums, factor of the sums).
template <int PHASE, bool SWIGLU, typename Record, typename Act, typename Epi>
__device__ __forceinline__ void rows_kernel(const SmallRows& P, int choices, char* smem, float* red_m, int tid, int row0, Record record, Act act, Epi epi) {
  constexpr int NM = PHASE == 0 && SWIGLU ? 2 : 1, NT = kSmThreads;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float4* XL = (float4*)smem;
  float* XS = (float*)(smem + P.xs_off);
  float* red = (float*)(smem + P.red_off);
  uint16_t* SI = (uint16_t*)(smem + P.si_off);
  const uint8_t* W = (const uint8_t*)smem + P.w_off;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(MOEQ_LDS char*)smem;
  const int row_end = min(P.rows, row0 + P.R), cols = P.cols;
  int j = -1, row = 0, n = 0, bits = 0;               // the pass at work: choice, first row, rows, bitwidth
  int nj = 0, nrow = row0, nn = 0, nbits = 0;         // the pass requested
  const uint8_t *s0 = nullptr, *s1 = nullptr;
  ScaleRegs S[NM];
  DevExpert ex = record(0);
  float dn = 1.0f, up = 1.0f;
  auto stage = [&](int jj) __attribute__((always_inline)) {
    const float m = wave_max(stage_raw<NT, 4>(act(jj), false, cols / 4, tid, XL, XS));
    if (lane == 0) red_m[wave] = m;
  };
  if constexpr (PHASE == 1) stage(0);                 // (ahead of the first copies: loads return in order)
#pragma unroll 1
  for (;;) {
    if (n) {
      fetch_wait();
      scales_store<NT>(S[0], s0, n * P.ng / 2, tid, (uint32_t*)SI);
      if constexpr (NM == 2) scales_store<NT>(S[NM - 1], s1, n * P.ng / 2, tid, (uint32_t*)(SI + P.si_stride));
      __syncthreads();
      if (row == row0) {
        const int e = safe_exponent(red_max<NT>(red_m));
        dn = pow2f(-e);
        up = pow2f(e);
      }
      switch (bits) {
        case 2: rows_dot<NT, 2, NM>(W, P.room, SI, P.si_stride, XL, XS, cols, P.group, P.gsh, P.ng, n, dn, tid, red, P.red_stride); break;
        case 4: rows_dot<NT, 4, NM>(W, P.room, SI, P.si_stride, XL, XS, cols, P.group, P.gsh, P.ng, n, dn, tid, red, P.red_stride); break;
        default: rows_dot<NT, 8, NM>(W, P.room, SI, P.si_stride, XL, XS, cols, P.group, P.gsh, P.ng, n, dn, tid, red, P.red_stride); break;
      }
      __syncthreads();
      nj = j;
      nrow = row + n;
      if (nrow >= row_end) {
        nrow = row0;
        if (++nj < choices) ex = record(nj);
      }
    }
    const bool more = nj < choices;
    if (more) {
      if (PHASE == 1 && nj != j && nj > 0) stage(nj);
      nbits = ex.bits;
      const int row_bytes = (cols >> 3) * nbits;
      nn = min(pass_rows(P.R, P.room, row_bytes), row_end - nrow);
      const uint8_t* q0 = PHASE == 0 ? ex.q_in : ex.q_out;
      s0 = (const uint8_t*)(PHASE == 0 ? ex.s_in : ex.s_out) + (size_t)nrow * P.ng * 2;
      scales_issue<NT>(S[0], s0, nn * P.ng / 2, tid);
      if constexpr (NM == 2) {
        s1 = (const uint8_t*)ex.s_gate + (size_t)nrow * P.ng * 2;
        scales_issue<NT>(S[NM - 1], s1, nn * P.ng / 2, tid);
      }
      fetch_block<NT>(q0 + (size_t)nrow * row_bytes, nn * row_bytes, lds0 + P.w_off, wave, lane);
      if constexpr (NM == 2) fetch_block<NT>(ex.q_gate + (size_t)nrow * row_bytes, nn * row_bytes, lds0 + P.w_off + P.room, wave, lane);
    }
    if (n) {
      rows_fold<NT, NM>(red, P.red_stride, min(row_pieces(cols, bits), NT), n, tid,
                        [&](int r, const float (&t)[NM]) __attribute__((always_inline)) { epi(j, row + r, t, up); });
    }
    if (!more) return;
    j = nj; row = nrow; n = nn; bits = nbits;
  }
}

// The experts of a token: lane r < k gets the r-th choice, by the rules of topk64 / topk_impl (order on the logits, ties to the
// lowest index; a NaN or +Inf logit, or none finite: experts 0 .. k-1), without the softmax. v[j]: logit of expert lane + 64 j.
template <int MPL>
__device__ __forceinline__ int choose(const float (&v)[MPL], int E, int k, int lane) {
  float m = v[0];
  bool nan = false;
#pragma unroll
  for (int j = 0; j < MPL; ++j) {
    m = fmaxf(m, v[j]);
    nan = nan || v[j] != v[j];
  }
  m = wave_max(m);
  if (__ballot(nan) != 0ull || !(fabsf(m) < INFINITY)) return lane;
  int mine = 0;
  uint32_t taken = 0;
  for (int r = 0; r < k; ++r) {
    if (r) {
      m = -INFINITY;
#pragma unroll
      for (int j = 0; j < MPL; ++j)
        if (!((taken >> j) & 1u)) m = fmaxf(m, v[j]);
      m = wave_max(m);
    }
    int be = -1;
#pragma unroll
    for (int j = 0; j < MPL; ++j) {
      const unsigned long long mask = __ballot(v[j] == m && lane + 64 * j < E && !((taken >> j) & 1u));
      if (be < 0 && mask != 0ull) be = 64 * j + (__ffsll((long long)mask) - 1);
    }
#pragma unroll
    for (int j = 0; j < MPL; ++j)
      if (lane + 64 * j == be) taken |= 1u << j;
    mine = lane == r ? be : mine;
  }
  return mine;
}

template <bool SWIGLU, int MODE>
__global__ __launch_bounds__(kSmThreads, 4) void k_small_in(SmallRows P) {
  extern __shared__ uint4 smem4[];
  __shared__ int sel_ew[kSmThreads / 64][8];
  __shared__ float sel_gw[kSmThreads / 64][8];
  __shared__ float red_m[kSmThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), E = P.E, k = P.k;
  const int row0 = blockIdx.x * P.R;
  if (row0 >= P.rows) return;                        // (the first dimension of the grid is a multiple of the XCDs)
  const int token = small_div(blockIdx.y, k), jc = blockIdx.y - token * k;
  const float* lg = P.logits + (size_t)token * E;
  float v[2] = {-INFINITY, -INFINITY};
  if constexpr (MODE == kFromLogits) {
    if (lane < E) v[0] = lg[lane];
    if (E > 64 && lane + 64 < E) v[1] = lg[lane + 64];
  }
  float4* XL = (float4*)smem4;
  const float mx = wave_max(stage_raw<kSmThreads, 1>((const char*)P.act + (size_t)token * P.cols * (P.bf16 ? 2 : 4), P.bf16 != 0, P.cols / 4, tid, XL,
                                                     (float*)((char*)XL + P.xs_off)));
  if (lane == 0) red_m[wave] = mx;
  int my_e = P.fixed_expert;
  if constexpr (MODE == kGiven) {
    if (P.idx) my_e = P.idx[blockIdx.y];
  } else if (E <= 64) {
    const float v1[1] = {v[0]};
    my_e = __builtin_amdgcn_readlane(choose<1>(v1, E, k, lane), jc);
  } else if (E <= 128) {
    my_e = __builtin_amdgcn_readlane(choose<2>(v, E, k, lane), jc);
  } else {
    topk_from_logits(lg, E, k, P.renorm, lane, sel_ew[wave], sel_gw[wave], nullptr);
    my_e = sel_ew[wave][jc];
  }
  my_e = __builtin_amdgcn_readfirstlane(min(max(my_e, 0), E - 1));     // an address: kept inside the table
  const DevExpert* rec = P.table + my_e;
  float* h = P.out + (size_t)blockIdx.y * P.rows;
  rows_kernel<0, SWIGLU>(P, 1, (char*)smem4, red_m, tid, row0, [&](int) __attribute__((always_inline)) { return uniform_record<SWIGLU>(rec); },
                         [&](int) __attribute__((always_inline)) { return (const void*)nullptr; },
                         [&](int, int r, const auto& t, float up) __attribute__((always_inline)) {
                           const float a = t[0] * up;
                           if constexpr (SWIGLU) h[r] = silu(a) * (t[1] * up);
                           else h[r] = fmaxf(a, 0.f);
                         });
  // what phase 2 and the caller want to know, behind the work (the gates of more than 128 experts are there: selecting again would
  // hold the kernel's end up by 4 us)
  if (blockIdx.x == 0 && wave == 0) {
    if constexpr (MODE != kGiven) {
      if (E <= 128) topk_from_logits(lg, E, k, P.renorm, lane, sel_ew[0], sel_gw[0], nullptr);
      if (lane == 0) {
        P.idx[blockIdx.y] = my_e;
        P.gate[blockIdx.y] = sel_gw[0][jc];
      }
    }
    if (P.sel_tab && lane < 4) ((uint4*)(P.sel_tab + blockIdx.y))[lane] = ((const uint4*)rec)[lane];
  }
}

__global__ __launch_bounds__(kSmThreads, 4) void k_small_out(SmallRows P) {
  extern __shared__ uint4 smem4[];
  __shared__ float red_m[kSmThreads / 64];
  const int tid = threadIdx.x, k = P.k, token = blockIdx.y;
  const int row0 = blockIdx.x * P.R;
  if (row0 >= P.rows) return;
  float* ysum = (float*)((char*)smem4 + P.y_off);
  const int lane = tid & 63;
  const float gates = P.gate ? P.gate[(size_t)token * k + min(lane, k - 1)] : 1.0f;      // (in lane j that of choice j)
  // choices in top-k order, a row's by one lane at a time with barriers between: a fixed order of sums
  rows_kernel<1, false>(P, k, (char*)smem4, red_m, tid, row0,
                        [&](int j) __attribute__((always_inline)) {
                          return uniform_record<false>(P.fixed_expert >= 0 ? P.table + P.fixed_expert : P.sel_tab + (size_t)token * k + j);
                        },
                        [&](int j) __attribute__((always_inline)) { return (const void*)((const float*)P.act + ((size_t)token * k + j) * P.cols); },
                        [&](int j, int r, const auto& t, float up) __attribute__((always_inline)) {
                          const float g = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, gates), j));
                          const float v = g * (t[0] * up) + (j ? ysum[r - row0] : 0.f);
                          if (j + 1 < k) {
                            ysum[r - row0] = v;
                          } else {
                            float* y = P.out + (size_t)token * P.rows + r;
                            *y = P.accumulate ? *y + v : v;
                          }
                        });
}

template <bool SWIGLU, int RPT>
auto pick_small_cols(SmallMode mode) {
  return mode == kFromLogits ? k_small_cols<SWIGLU, kFromLogits, RPT> : mode == kInline ? k_small_cols<SWIGLU, kInline, RPT> : k_small_cols<SWIGLU, kGiven, RPT>;
}

SmallCols small_cols_plan(const LayerDims& L, int k, int SW, int bits_mask) {
  SmallCols P{};
  const int bits = bits_mask & 8 ? 8 : bits_mask & 4 ? 4 : 2, nm = L.act == MOEQ_ACT_SWIGLU ? 2 : 1, d = L.d_model;
  P.d = d; P.E = L.n_experts; P.renorm = L.renorm; P.bf16 = L.x_bf16; P.SW = SW; P.n_slices = L.d_ff / SW;
  P.group = L.group; P.gsh = (L.group & (L.group - 1)) == 0 ? __builtin_ctz(L.group) : -1; P.ng = d / L.group; P.group_out = L.group_out;
  P.red_stride = SW * std::min(row_pieces(d, bits), kSmThreads);
  P.w_stride = pad_to(SW * (d * bits / 8), 1024);
  P.si_stride = SW * P.ng;
  P.xs_off = pad_to(d, 64) * 4;
  P.h_off = P.xs_off + pad_to(d / 16, 4) * 4;
  P.red_off = P.h_off + SW * 4;
  P.si_off = P.red_off + std::max(nm * P.red_stride * 4, kSmRouteBytes);
  P.wi_off = pad_to(P.si_off + nm * P.si_stride * 2, 16);
  P.lds = P.wi_off + (nm + (k > 1 ? 2 : 1)) * P.w_stride;
  return P;
}

// LDS of a kernel over `rows` rows of `cols` columns, R of them a workgroup, nm matrices, in passes of up to `room` bytes a matrix.
SmallRows small_rows_plan_at(int cols, int rows, int group, int R, int nm, int room, int bits_mask) {
  SmallRows P{};
  P.cols = cols; P.rows = rows; P.R = R; P.room = room;
  P.group = group; P.gsh = (group & (group - 1)) == 0 ? __builtin_ctz(group) : -1; P.ng = cols / group;
  int pass = 0;
  for (int b = 2; b <= 8; b *= 2)
    if (bits_mask & b) {
      const int n = pass_rows(R, room, cols * b / 8);
      pass = std::max(pass, n);
      P.red_stride = std::max(P.red_stride, n * std::min(row_pieces(cols, b), kSmThreads));
    }
  P.si_stride = pad_to(pass * P.ng, 8);
  P.xs_off = pad_to(cols, 64) * 4;
  P.y_off = P.xs_off + pad_to(cols / 16, 4) * 4;
  P.red_off = P.y_off + pad_to(R, 4) * 4;
  P.si_off = P.red_off + nm * P.red_stride * 4;
  P.w_off = pad_to(P.si_off + nm * P.si_stride * 2, 16);
  P.lds = P.w_off + nm * room;
  return P;
}
// ... that hold the workgroup's rows at the widest bitwidth in as few equal passes as leave two workgroups a compute unit, kRowsRoom
// bytes in all at least. A pass is a round trip: SwiGLU, 1536 x 2048, 4 and 8 bits, 6 tokens in up to four passes of 16 KB a matrix
// 29.2 us, now 25.0 (28.7 in the kernels of ffn_decode.hip). Passes as large as fit, the last one small, lose 4 to 8 %.
SmallRows small_rows_plan(int cols, int rows, int group, int R, int nm, int bits_mask) {
  const int least = kRowsRoom / nm, row_bytes = cols / 8 * (bits_mask & 8 ? 8 : bits_mask & 4 ? 4 : 2);
  for (int passes = 1;; ++passes) {
    const int room = pad_to(pad_to((R + passes - 1) / passes, 4) * row_bytes, 1024);
    if (room <= least) return small_rows_plan_at(cols, rows, group, R, nm, least, bits_mask);
    const SmallRows P = small_rows_plan_at(cols, rows, group, R, nm, room, bits_mask);
    if ((size_t)P.lds <= kSmLdsTwo - 1024) return P;                  // (up to 544 bytes are static)
  }
}

}  // namespace

// Single tokens wherever a slice's blocks fit in LDS; calls of more where two workgroups share a compute unit and slices are at
// most 32 columns: wider ones are streams, which the kernels of decode_fused.hip keep busier. us per layer call, theirs / this
// one's: d_ff 16384 (slices of 64), d_model 1024, 4 bits, one token 18.1 / 14.3, 3 tokens 24.5 / 30.9, 31 tokens 189 / 261;
// one workgroup per compute unit (8 bits, d_model 1024, d_ff 8192, two choices) one token 24.3 / 18.4, 3 tokens 33.9 / 42.8; d_model
// 1536, d_ff 4096, 4 bits, 1 / 8 / 31 tokens 18.1 / 12.1, 83 / 41, 276 / 140. 440 calls within the line: 1.34 times faster on
// average, none slower by more than 1 %; 120 within 2 KB of it 2.0 times, the least 1.06 (8 bits, 1024 x 6144, 3 tokens). With logits
// a workgroup has 512 bytes beside the launch's, so that shapes of the last half KB run one: still 1.5 times faster or more.
bool small_cols_fits(const LayerDims& L, const FusedPlan& plan, int32_t bits_mask, int32_t T) {
  if (!plan.SW || plan.mx || L.d_model > 4 * kSmThreads || (T > 1 && plan.SW > 32)) return false;
  return (size_t)small_cols_plan(L, L.top_k, plan.SW, bits_mask).lds <= (T > 1 ? kSmLdsTwo : kSmLds);
}

hipError_t init_attrs_decode_small() {
  for (SmallMode m : {kFromLogits, kInline, kGiven})
    for (const void* kf : {(const void*)pick_small_cols<false, 2>(m), (const void*)pick_small_cols<true, 2>(m),
                           (const void*)pick_small_cols<false, 4>(m), (const void*)pick_small_cols<true, 4>(m)})
      if (hipError_t e = hipFuncSetAttribute(kf, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSmLds); e != hipSuccess) return e;
  for (const void* kf : {(const void*)k_small_in<false, kFromLogits>, (const void*)k_small_in<false, kGiven>, (const void*)k_small_in<true, kFromLogits>,
                         (const void*)k_small_in<true, kGiven>, (const void*)k_small_out})
    if (hipError_t e = hipFuncSetAttribute(kf, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSmLds); e != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_small_cols(const LayerDims& L, const FusedPlan& plan, const DevExpert* table, const float* router_w,
                             const float* router_bias, const float* logits, int32_t fixed_expert, const float* gate_in,
                             const int32_t* route_idx, const float* route_gate, int32_t bits_mask, const void* x, int32_t T,
                             float* part, int32_t* idx_out, float* gate_out, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const bool fixed = fixed_expert >= 0;
  SmallCols P = small_cols_plan(L, fixed ? 1 : L.top_k, plan.SW, bits_mask);
  const bool sw = L.act == MOEQ_ACT_SWIGLU, wide = L.d_model > 2 * kSmThreads;
  P.table = table; P.x = x; P.logits = logits; P.Wr = router_w; P.bias = router_bias; P.part = part;
  P.fixed_expert = fixed_expert; P.k = fixed ? 1 : L.top_k;
  P.route_idx = fixed ? nullptr : route_idx;
  P.route_gate = fixed ? gate_in : route_gate;
  P.idx_out = idx_out; P.gate_out = gate_out;
  const SmallMode mode = fixed || route_idx ? kGiven : logits ? kFromLogits : kInline;
  auto kernel = wide ? (sw ? pick_small_cols<true, 4>(mode) : pick_small_cols<false, 4>(mode))
                     : (sw ? pick_small_cols<true, 2>(mode) : pick_small_cols<false, 2>(mode));
  if (ev_start && ev_stop)
    hipExtLaunchKernelGGL(kernel, dim3(plan.n_slices, T), dim3(kSmThreads), (size_t)P.lds, st, ev_start, ev_stop, 0, P);
  else
    hipLaunchKernelGGL(kernel, dim3(plan.n_slices, T), dim3(kSmThreads), (size_t)P.lds, st, P);
  return hipGetLastError();
}

// By the multiplications of the call (a SwiGLU layer's third matrix counted). Beyond the line a call is a stream, or its
// instructions bound it, and the kernels of ffn_decode.hip spend half as many. us, theirs / these: 1024 x 4096, 4 bits, 1 / 4 / 8 / 14
// tokens on 128 experts 18.1 / 12.9, 22.2 / 17.6, 23.6 / 21 and 28.5 / 29.4; 2048 x 8192, 1 / 2 / 3 tokens 22.0 / 17.2, 24.7 /
// 21.3, 30.2 / 30. 662 calls within the line, of 1 to 84 tokens and 1 to 200 experts: 1.34 times faster on average, none slower (least
// 1.015). Both lines are cautious:
// of 174 calls of 34 to 60 million on widths that are a multiple of 512 these kernels are 1.12 times faster on average, but 17 are more
// than 5 % slower (0.82); of 233 calls of 18 to 34 million on other widths none is slower (1.06 to 6.5 times, 1.7 in the middle). 18
// was drawn on 768 x 3072 with 8 bits before the rows of a workgroup were chosen by the XCD's places (8 tokens 21.7 / 21.3, 10 tokens
// 22 / 24.6); calls of 8 and of 24 tokens of that layer run the same kernels by it, which test_gpu_group.py compares by their bits.
bool small_rows_fits(const LayerDims& L, int64_t pairs) {
  if (L.d_model > 2048 || L.d_ff > kRowsMaxCols) return false;
  const double work = (double)pairs * L.d_model * L.d_ff * (L.act == MOEQ_ACT_SWIGLU ? 1.5 : 1.0);
  return work <= (L.d_model % 512 == 0 ? 34e6 : 18e6);
}

hipError_t launch_small_in(const LayerDims& L, const DevExpert* table, const float* logits, int32_t* idx, float* gate, DevExpert* sel_tab,
                           int32_t fixed_expert, int32_t bits_mask, const void* x, int32_t T, float* h, hipStream_t st) {
  const bool fixed = fixed_expert >= 0, sw = L.act == MOEQ_ACT_SWIGLU;
  const int k = fixed ? 1 : L.top_k, nm = sw ? 2 : 1;
  const int R = small_rows_of_wg(L.d_ff, L.d_model, (int64_t)T * k);
  SmallRows P = small_rows_plan(L.d_model, L.d_ff, L.group, R, nm, bits_mask);
  P.table = table; P.logits = logits; P.idx = fixed ? nullptr : idx; P.gate = gate; P.sel_tab = fixed ? nullptr : sel_tab; P.act = x; P.out = h;
  P.fixed_expert = fixed_expert; P.E = L.n_experts; P.k = k; P.renorm = L.renorm; P.bf16 = L.x_bf16;
  const dim3 grid(pad_to((L.d_ff + R - 1) / R, 8), T * k);
  auto kernel = fixed || !logits ? (sw ? k_small_in<true, kGiven> : k_small_in<false, kGiven>) : (sw ? k_small_in<true, kFromLogits> : k_small_in<false, kFromLogits>);
  hipLaunchKernelGGL(kernel, grid, dim3(kSmThreads), (size_t)P.lds, st, P);
  return hipGetLastError();
}

hipError_t launch_small_out(const LayerDims& L, const DevExpert* table, const DevExpert* sel_tab, const float* gate, int32_t fixed_expert,
                            int32_t bits_mask, int32_t accumulate, const float* h, int32_t T, float* y, hipStream_t st) {
  const bool fixed = fixed_expert >= 0;
  const int k = fixed ? 1 : L.top_k;
  const int R = small_rows_of_wg(L.d_model, L.d_ff, T);
  SmallRows P = small_rows_plan(L.d_ff, L.d_model, L.group_out, R, 1, bits_mask);
  P.table = table; P.gate = (float*)gate; P.sel_tab = (DevExpert*)sel_tab; P.act = h; P.out = y;
  P.fixed_expert = fixed_expert; P.E = L.n_experts; P.k = k; P.accumulate = accumulate;
  hipLaunchKernelGGL(k_small_out, dim3(pad_to((L.d_model + R - 1) / R, 8), T), dim3(kSmThreads), (size_t)P.lds, st, P);
  return hipGetLastError();
}

}  // namespace moeq
