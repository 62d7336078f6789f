// Calls of many tokens on layers whose scale groups do not fit the tiles of prefill.hip (the Switch-shaped layers: groups
// of 32 or 64, a few hundred columns), and of 6 to 31 tokens with W_out in columns where it pays (api.cpp, group_pays): the (token, choice) pairs are grouped by expert, and every expert's packed rows
// are streamed once for a tile of up to 32 of its pairs, on the matrix cores (Section 2.1: only the chosen experts work
// on a token; Section 3.2: the codes are decompressed by the mirror of the linear quantization on their way into the
// instruction). ReLU layers, W_out canonical or in columns.
//
// Arithmetic: that of prefill.hip. Masked code fields are binary16 subnormals, the activations are normalised by a power
// of two (per token for x, per pair and 128 columns for h), converted to binary16 and pre-divided by the fields' powers
// of two, the accumulation of v_mfma_f32_16x16x32_f16 starts at the negated offset term, and scales are applied in fp32.
// One instruction covers a block of 32 columns, which lies inside one scale group whatever the group size: the four
// quarter wavefronts (kb) of the B operand hold the four quarters of the block. A lane loads 16 consecutive bytes, which
// are a whole block at 4 bits, two at 2 bits and half of one at 8 bits, so the words move between the quarters with
// v_permlane32_swap / v_permlane16_swap (one instruction per block and 16 rows).
//
// What bounds it: instruction issue and memory latency of workgroups that live for two units (500 tokens on a 64-expert
// Switch-base layer: k_grp_in and k_grp_out 38 us each for 91 MB each, half of a wavefront's life in waits, the vector port
// issuing 45 % of the time), and four small kernels (router 12.6, top-k, grouping, combine 4.7 each). The token-by-token
// kernels it replaces for these calls (159 + 146 us) pay the unpack arithmetic once per token instead of once per tile.
#include "decode_core.h"

namespace moeq {
namespace {

// 16-pair tiles of a work item (template parameter NT): two, or one where the experts' average load is small (half the
// operands to stage and twice the rows per workgroup)
constexpr int kGMaxTiles = 2;
constexpr int kGThreads = 512, kGWaves = 8;
constexpr int kGUnit = 128;                // rows a workgroup multiplies at a time (16 per wavefront); columns h shares an exponent over
constexpr int kGChunk = 1024;              // columns of d_ff a k_grp_out workgroup takes
constexpr int kGRing = 4;                  // 16-byte loads per lane in flight
constexpr int kGMaxPairs = 8192;           // pairs grouped at a time
constexpr int kGMaxBlocks = 64;            // blocks of 32 columns of d_model

struct alignas(16) GrpItem {   // pairs gpair[g0 .. g0 + n) of an expert, and what the kernels need of the expert's record
  int32_t n, g0, bits, pad;
  const uint8_t* q_in;
  const uint16_t* s_in;
  const uint8_t* q_out;
  const uint16_t* s_out;
};
static_assert(sizeof(GrpItem) == 48, "three 16-byte pieces");

struct GrpArgs {
  LayerDims L;
  const DevExpert* table;
  const void* x;
  const int32_t* idx;       // [M]
  int32_t M, k;
  GrpItem* items;
  int32_t* n_items;
  int32_t* gpair;           // [M] pairs in expert order
  int32_t* ginv;            // [M] a pair's place in it
  uint8_t* HQ;              // [M][d_ff / 128 rounded up][block 4][kb 4][16]: h as A operands
  float* HS;                // [M][d_ff / 128 rounded up]: 2^e of 128 columns
  float* HK;                // [M][d_ff / 32 rounded up to 4]: negated offset term of every block
  float* part;              // [chunks][M][d_model]
  int32_t tok;              // pairs of an item: 16 or 32
  int32_t rows_per_wg;      // k_grp_in: multiple of kGUnit; k_grp_out: of its unit
};

// ---------------------------------------------------------------------------------------------
// Workgroup e: the histogram of all pairs (redundantly, in LDS), from it the place of expert e's pairs and items, then
// its pairs in increasing order.
__global__ __launch_bounds__(256) void k_grp_plan(GrpArgs G) {
  __shared__ int h[1024];
  __shared__ int red[4][2];
  __shared__ int wcnt[4];
  const int kGTok = G.tok;
  const int E = G.L.n_experts, e = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < E; i += 256) h[i] = 0;
  __syncthreads();
  for (int p = tid; p < G.M; p += 256) atomicAdd(&h[min(max(G.idx[p], 0), E - 1)], 1);
  __syncthreads();
  int pairs = 0, items = 0;
  for (int i = tid; i < e; i += 256) { pairs += h[i]; items += (h[i] + kGTok - 1) / kGTok; }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) { pairs += __shfl_xor(pairs, off); items += __shfl_xor(items, off); }
  if (lane == 0) { red[wave][0] = pairs; red[wave][1] = items; }
  __syncthreads();
  int base = red[0][0] + red[1][0] + red[2][0] + red[3][0];
  const int ibase = red[0][1] + red[1][1] + red[2][1] + red[3][1];
  const int n = h[e], mine = (n + kGTok - 1) / kGTok;
  for (int i = tid; i < mine; i += 256)
    G.items[ibase + i] = GrpItem{min(kGTok, n - i * kGTok), base + i * kGTok, G.table[e].bits, 0,
                                 G.table[e].q_in, G.table[e].s_in, G.table[e].q_out, G.table[e].s_out};
  if (e == E - 1 && tid == 0) *G.n_items = ibase + mine;
  if (n == 0) return;
  for (int p0 = 0; p0 < G.M; p0 += 256) {
    const int p = p0 + tid;
    const bool hit = p < G.M && min(max(G.idx[p], 0), E - 1) == e;
    const unsigned long long mask = __ballot(hit);
    if (lane == 0) wcnt[wave] = __popcll(mask);
    __syncthreads();
    int before = __popcll(mask & ((1ull << lane) - 1ull));
    for (int w = 0; w < wave; ++w) before += wcnt[w];
    if (hit) {
      G.gpair[base + before] = p;
      G.ginv[p] = base + before;
    }
    base += wcnt[0] + wcnt[1] + wcnt[2] + wcnt[3];
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// A operand of block b, quarter kb: the columns c0 .. c0 + 3 and c1 .. c1 + 3.
template <int BITS>
__device__ __forceinline__ void block_cols(int b, int kb, int& c0, int& c1) {
  if (BITS == 4) { c0 = 32 * b + 8 * kb; c1 = c0 + 4; }
  else if (BITS == 8) { c0 = 32 * b + 16 * (kb & 1) + 8 * (kb >> 1); c1 = c0 + 4; }
  else { c0 = 32 * b + 16 * (kb & 1) + 4 * (kb >> 1); c1 = c0 + 8; }
}
__device__ __forceinline__ float4 load_x4(const char* row, bool bf16, int c) {
  if (bf16) {
    const uint2 w = *(const uint2*)(row + (size_t)c * 2);
    return make_float4(bf16_bits_to_f32(w.x & 0xffffu), bf16_bits_to_f32(w.x >> 16), bf16_bits_to_f32(w.y & 0xffffu), bf16_bits_to_f32(w.y >> 16));
  }
  return *(const float4*)(row + (size_t)c * 4);
}
// The eight values (already normalised) as binary16 in the order of codes8 / the masks of b_operand, pre-divided, and
// their sum as the consumer sees them.
template <int BITS>
__device__ __forceinline__ uint4 block_operand(const float (&a)[4], const float (&b)[4], float& sum) {
  uint32_t ha[4], hb[4];
  sum = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    ha[i] = f32_to_f16_bits(a[i]);
    hb[i] = f32_to_f16_bits(b[i]);
    sum += f16_bits_to_f32(ha[i]) + f16_bits_to_f32(hb[i]);
  }
  if (BITS == 8) return make_uint4(ha[0] | ha[2] << 16, ha[1] | ha[3] << 16, hb[0] | hb[2] << 16, hb[1] | hb[3] << 16);
  uint32_t r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r[i] = ha[i] | hb[i] << 16;
    if (BITS == 4 && (i & 1)) r[i] = pair_scale(r[i], 0.0625f);
    if (BITS == 2 && i > 0) r[i] = pair_scale(r[i], i == 1 ? 0.25f : i == 2 ? 0.0625f : 0.015625f);
  }
  return make_uint4(r[0], r[1], r[2], r[3]);
}

// Code fields two bits higher than they lie in a byte. The matrix instruction aligns its products by the exponents of its
// operands, subnormal ones as they stand, and what it drops below the largest weighs most against fields that begin at bit
// 0. Error of 500 tokens on 2-bit Switch-base experts against 64 bits: two bits up 2.95e-4, as they lie 3.05e-4 (the kernels
// that work token by token: 2.98e-4). It grows where a column of large activations meets zero weights: 60 tokens, an
// element 2^13 times the others, largest error of 4- / 8-bit experts 8.1e-4 / 5.7e-4 (as they lie 2.2e-3 / 2.6e-3, token by token
// 2.1e-3 / 2.1e-3).
// 2 bits: eight of the word's sixteen, by quarter; 4 and 8 bits: as codes8. The masks leave the rotations' wrapped bits out.
__device__ __forceinline__ half8_t codes8_2(uint32_t w, int kb) {
  const uint32_t v = __builtin_amdgcn_alignbit(w, w, kb & 2 ? 6u : 30u);
  const u32x4v_t r = {v & 0x000c000cu, v & 0x00300030u, v & 0x00c000c0u, v & 0x03000300u};
  return __builtin_bit_cast(half8_t, r);
}
__device__ __forceinline__ half8_t codes8_4(uint32_t w) {
  const uint32_t v = __builtin_amdgcn_alignbit(w, w, 30u), u = __builtin_amdgcn_alignbit(w, w, 6u);
  const u32x4v_t r = {v & 0x003c003cu, v & 0x03c003c0u, u & 0x003c003cu, u & 0x03c003c0u};
  return __builtin_bit_cast(half8_t, r);
}
__device__ __forceinline__ half8_t codes8_8(uint32_t w0, uint32_t w1) {
  const u32x4v_t r = {__builtin_amdgcn_alignbit(w0, w0, 30u) & 0x03fc03fcu, __builtin_amdgcn_alignbit(w0, w0, 6u) & 0x03fc03fcu,
                      __builtin_amdgcn_alignbit(w1, w1, 30u) & 0x03fc03fcu, __builtin_amdgcn_alignbit(w1, w1, 6u) & 0x03fc03fcu};
  return __builtin_bit_cast(half8_t, r);
}

// blocks of 32 columns that 64 bytes of a row hold (one load of four quarters), and that share one application of the
// scale (AB: 1, 2 or 4 by the group size, not more than a load's blocks)
template <int BITS> constexpr int load_blocks() { return 16 / BITS; }                 // 8, 4, 2
template <int BITS, int G4> constexpr int apply_blocks() { return G4 < load_blocks<BITS>() ? G4 : load_blocks<BITS>(); }

// B operands of the blocks of one load.
template <int BITS>
__device__ __forceinline__ void b_operands(uint4 v, int kb, half8_t (&B)[load_blocks<BITS>()]) {
  uint32_t w[4] = {v.x, v.y, v.z, v.w};
  if constexpr (BITS == 8) {
    swap32(w[0], w[2]);
    swap32(w[1], w[3]);
    B[0] = codes8_8(w[0], w[1]);
    B[1] = codes8_8(w[2], w[3]);
  } else {
    // quarters x words transposed: word j then holds, in quarter kb, word kb of the load's piece j
    swap32(w[0], w[2]);
    swap32(w[1], w[3]);
    swap16(w[0], w[1]);
    swap16(w[2], w[3]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (BITS == 4) {
        B[j] = codes8_4(w[j]);
      } else {
        uint32_t a = w[j], b = w[j];
        swap32(a, b);                    // (words 0, 1, 0, 1) and (words 2, 3, 2, 3) of the piece
        B[2 * j] = codes8_2(a, kb);
        B[2 * j + 1] = codes8_2(b, kb);
      }
    }
  }
}

// What turns the results of the instructions into sums of code * activation, and the offset of a code in their unit.
constexpr float kCodeUnit = 4194304.0f;     // 2^22
template <int BITS> constexpr float code_half() { return (float)(1 << (BITS - 1)) / kCodeUnit; }

struct GrpLds {             // byte offsets of the pieces of a workgroup's LDS
  int a, ks, up, scales, h, total;
};
// Row stride (in scales) of the scales in LDS: whole 16-byte pieces, an odd number of them (few bank conflicts).
__host__ __device__ constexpr int scale_stride(int ng) { return ((ng + 7) / 8 | 1) * 8; }
// nb: blocks of K rounded up to whole loads of every bitwidth; rows: rows whose scales are kept; ng: scale groups kept per row
__host__ __device__ inline GrpLds grp_lds(int nt, int nb, int rows, int ng, bool h) {
  const int kGTok = 16 * nt;
  GrpLds l{};
  l.a = 0;
  l.ks = l.a + nb * nt * 1024;
  l.up = l.ks + nb * kGTok * 4;
  l.scales = l.up + (h ? 1 : nb / 4) * kGTok * 4;        // (all offsets are multiples of 16)
  l.h = l.scales + rows * scale_stride(ng) * 2;
  l.total = l.h + (h ? kGTok * (kGUnit + 4) * 4 : 0);
  return l;
}
__host__ __device__ inline int chunk_groups(int group) { return kGChunk % group == 0 ? kGChunk / group : kGChunk / group + 2; }
__host__ __device__ inline int padded_blocks(int cols) { return (cols + 255) / 256 * 8; }

// The scales of rows [row0, row0 + rows) and groups [g0, g0 + ng) (zero past n_groups and past n_rows) into LDS. Whole
// 16-byte pieces where the matrix's rows of scales consist of aligned ones, several per thread in flight; else value by
// value, eight in flight.
__device__ __forceinline__ void stage_scales(const uint16_t* s, int n_rows, int n_groups, int row0, int rows, int g0, int ng,
                                             uint16_t* S) {
  const uint8_t* sp = (const uint8_t*)uniform_ptr(s);
  const int stride = scale_stride(ng), live = min(rows, n_rows - row0);
  if (((uint32_t)(uintptr_t)sp & 15u) == 0u && ((n_groups | g0 | ng) & 7) == 0 && g0 + ng <= n_groups) {
    const uint32_t per = (uint32_t)ng / 8u, total = (uint32_t)live * per;
    for (uint32_t i0 = threadIdx.x; i0 < total; i0 += 4 * kGThreads) {
      uint4 v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t i = min(i0 + k * kGThreads, total - 1u), r = i / per;
        v[k] = gload_u32x4(sp + ((size_t)(row0 + (int)r) * (uint32_t)n_groups + (uint32_t)g0 + (i - r * per) * 8u) * 2u);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t i = min(i0 + k * kGThreads, total - 1u), r = i / per;
        *(uint4*)(S + r * (uint32_t)stride + (i - r * per) * 8u) = v[k];
      }
    }
    return;
  }
  const uint32_t total = (uint32_t)rows * (uint32_t)ng;
  for (uint32_t i0 = threadIdx.x; i0 < total; i0 += 8 * kGThreads) {
    uint32_t v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t i = min(i0 + k * kGThreads, total - 1u), r = i / (uint32_t)ng, g = i - r * (uint32_t)ng;
      const bool ok = (int)r < live && g0 + (int)g < n_groups;
      v[k] = gload_u16(sp + (ok ? ((size_t)(row0 + (int)r) * (uint32_t)n_groups + (uint32_t)(g0 + (int)g)) * 2u : 0u));
      v[k] = ok ? v[k] : 0u;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t i = min(i0 + k * kGThreads, total - 1u), r = i / (uint32_t)ng, g = i - r * (uint32_t)ng;
      S[r * (uint32_t)stride + g] = (uint16_t)v[k];
    }
  }
}

// CNT blocks of a load (from its block OFF; block number blk, columns from col0 + 32 blk of the matrix) against the
// tiles: D = A B - offset per application of the scale, inner += scale * D. Blocks past the row's end have zero operands;
// their scale is any of the row's.
template <int NT, int AB0, int OFF, int CNT, int NB>
__device__ __forceinline__ void multiply_blocks(const half8_t (&B)[NB], int blk, int col0, int nt, int lane, int kb, const uint4* A,
                                                const float* KS, const uint16_t* srow, int g_first, int g_last, int group, int gsh,
                                                float (&inner)[NT][4]) {
  constexpr int kGTok = 16 * NT;
  constexpr int AB = AB0 < CNT ? AB0 : CNT;
  float sc[CNT / AB];
#pragma unroll
  for (int a = 0; a < CNT; a += AB)
    sc[a / AB] = f16_bits_to_f32(srow[min((int)div_group((uint32_t)(col0 + (blk + a) * 32), group, gsh), g_last) - g_first]);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t < nt) {
      float4_t D[CNT / AB];
#pragma unroll
      for (int a = 0; a < CNT; a += AB) {
        const float4 k4 = *(const float4*)(KS + (blk + a) * kGTok + 16 * t + 4 * kb);
        D[a / AB] = (float4_t){k4.x, k4.y, k4.z, k4.w};
      }
#pragma unroll
      for (int i = 0; i < AB; ++i)
#pragma unroll
        for (int a = 0; a < CNT; a += AB)
          D[a / AB] = mfma16(as_half8(A[((blk + a + i) * NT + t) * 64 + lane]), B[OFF + a + i], D[a / AB]);
#pragma unroll
      for (int a = 0; a < CNT; a += AB)
#pragma unroll
        for (int i = 0; i < 4; ++i) inner[t][i] = fmaf(D[a / AB][i], sc[a / AB], inner[t][i]);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// W_in (canonical): item x rows [blockIdx.x * rows_per_wg, + rows_per_wg).
template <int BITS, int G4, int NT>
__device__ __forceinline__ void grp_in(const GrpArgs& G, const GrpItem& item, char* smem) {
  constexpr int AB = apply_blocks<BITS, G4>(), NB = load_blocks<BITS>(), kGTok = 16 * NT;
  const LayerDims& L = G.L;
  const int d = L.d_model, f = L.d_ff, ng = d / L.group, gsh = group_shift(L.group);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, kb = lane >> 4;
  const int nbp = padded_blocks(d), nblk = d / 32;
  const int row_begin = blockIdx.x * G.rows_per_wg, row_end = min(f, row_begin + G.rows_per_wg);
  if (row_begin >= row_end) return;
  const GrpLds lds = grp_lds(NT, nbp, G.rows_per_wg, ng, true);
  uint4* A = (uint4*)(smem + lds.a);
  float* KS = (float*)(smem + lds.ks);
  float* UP = (float*)(smem + lds.up);
  uint16_t* SC = (uint16_t*)(smem + lds.scales);
  float* H = (float*)(smem + lds.h);
  const uint8_t* q = uniform_ptr(item.q_in);
  const int nt = (item.n + 15) / 16;
  const int NU = (f + kGUnit - 1) / kGUnit;

  // ---- the stream of packed rows: loads of 64 bytes of 16 rows, kGRing ahead, through all units of the workgroup
  const uint32_t row_bytes = (uint32_t)d * BITS / 8u, pieces = row_bytes / 16u;
  const int SPU = (nblk + NB - 1) / NB;                  // loads per unit
  const int SLOTS = (SPU + kGRing - 1) / kGRing * kGRing;
  const int u0 = row_begin / kGUnit, u1 = (row_end + kGUnit - 1) / kGUnit;
  auto issue = [&](int u, int s) __attribute__((always_inline)) {      // slots past the end repeat cached bytes
    const uint32_t row = (uint32_t)min(u * kGUnit + wave * 16 + n, f - 1);
    const uint32_t pc = min((uint32_t)(4 * min(s, SPU - 1) + kb), pieces - 1u);
    return gload_u32x4(q + (row * row_bytes + pc * 16u));
  };
  uint4 R[kGRing];
#pragma unroll
  for (int i = 0; i < kGRing; ++i) R[i] = issue(u0, i);

  // ---- the item's activations, normalised per token: wavefront w stages the pairs w, w + 8, ...; a lane holds its
  // pieces (block, quarter; a block's quarters are four lanes) of a pair in registers
  constexpr int IT = kGMaxBlocks * 4 / 64;
  const bool bf16 = L.x_bf16 != 0;
  struct Held { float4 a[IT], b[IT]; };
  auto load_pair = [&](Held& v, int m) __attribute__((always_inline)) {
    const int pair = G.gpair[item.g0 + min(m, item.n - 1)];
    const char* row = (const char*)G.x + (size_t)(pair / G.k) * d * (bf16 ? 2 : 4);
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int pc = lane + 64 * it, b = pc >> 2;
      v.a[it] = v.b[it] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (b < nblk) {
        int c0, c1;
        block_cols<BITS>(b, pc & 3, c0, c1);
        v.a[it] = load_x4(row, bf16, c0);
        v.b[it] = load_x4(row, bf16, c1);
      }
    }
  };
  auto max4 = [](const float4& v) { return fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))); };
  auto put_pair = [&](const Held& v, int m) __attribute__((always_inline)) {
    float mx = 0.f;
#pragma unroll
    for (int it = 0; it < IT; ++it) mx = fmaxf(mx, fmaxf(max4(v.a[it]), max4(v.b[it])));
    const int e = norm_exponent(wave_max(mx));
    const float dn = pow2f(-e);
    if (lane == 0) UP[m] = pow2f(e);
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int pc = lane + 64 * it, b = pc >> 2;
      if (pc < nbp * 4) {
        float sum;
        const float va[4] = {v.a[it].x * dn, v.a[it].y * dn, v.a[it].z * dn, v.a[it].w * dn};
        const float vb[4] = {v.b[it].x * dn, v.b[it].y * dn, v.b[it].z * dn, v.b[it].w * dn};
        A[(b * NT + (m >> 4)) * 64 + (pc & 3) * 16 + (m & 15)] = block_operand<BITS>(va, vb, sum);
        sum += dpp<kDppXor1>(sum);
        sum += dpp<kDppXor2>(sum);
        if constexpr (AB >= 2) sum += __shfl_xor(sum, 4);
        if constexpr (AB >= 4) sum += __shfl_xor(sum, 8);
        if ((pc & 3) == 0 && b % AB == 0) KS[b * kGTok + m] = sum * -code_half<BITS>();
      }
    }
  };
  for (int m = wave; m < item.n; m += kGWaves) {  // (rows of absent pairs stay as they are: nobody looks at their results)
    Held v;
    load_pair(v, m);
    put_pair(v, m);
  }
  stage_scales(item.s_in, f, ng, row_begin, G.rows_per_wg, 0, ng, SC);
  __syncthreads();

  const int l0 = row_begin;
  for (int u = u0; u < u1; ++u) {
    float inner[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) inner[t][i] = 0.f;
    const uint16_t* srow = SC + (u * kGUnit + wave * 16 + n - l0) * scale_stride(ng);
    for (int s0 = 0; s0 < SLOTS; s0 += kGRing) {
#pragma unroll
      for (int i = 0; i < kGRing; ++i) {
        const int s = s0 + i;
        if (s < SPU) {
          half8_t B[NB];
          b_operands<BITS>(R[i], kb, B);
          multiply_blocks<NT, AB, 0, NB < 4 ? NB : 4>(B, s * NB, 0, nt, lane, kb, A, KS, srow, 0, ng - 1, L.group, gsh, inner);
          if constexpr (NB == 8) multiply_blocks<NT, AB, 4, 4>(B, s * NB + 4, 0, nt, lane, kb, A, KS, srow, 0, ng - 1, L.group, gsh, inner);
        }
        const bool next = s + kGRing >= SLOTS;
        R[i] = issue(next ? min(u + 1, u1 - 1) : u, next ? s + kGRing - SLOTS : s + kGRing);
      }
    }
    // ---- 128 columns of h of every pair: to LDS, then normalised, converted and stored as k_grp_out's operands
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = 16 * t + 4 * kb + i;
        const float v = u * kGUnit + wave * 16 + n < f ? fmaxf(inner[t][i] * kCodeUnit * UP[t < nt ? m : 0], 0.f) : 0.f;
        if (t < nt) H[m * (kGUnit + 4) + wave * 16 + n] = v;
      }
    __syncthreads();
    {
      const int m = tid >> 4, b = (tid >> 2) & 3, qk = tid & 3;        // 512 threads = 32 pairs x 16 pieces
      int c0, c1;
      block_cols<BITS>(b, qk, c0, c1);
      float va[4], vb[4], mx = 0.f;
      const float* hr = H + (m < 16 * nt ? m : 0) * (kGUnit + 4);      // (one tile: half of the threads repeat pair 0)
      const float4 ha = *(const float4*)(hr + c0), hb = *(const float4*)(hr + c1);
      va[0] = ha.x; va[1] = ha.y; va[2] = ha.z; va[3] = ha.w;
      vb[0] = hb.x; vb[1] = hb.y; vb[2] = hb.z; vb[3] = hb.w;
#pragma unroll
      for (int i = 0; i < 4; ++i) mx = fmaxf(mx, fmaxf(fabsf(va[i]), fabsf(vb[i])));
      mx = fmaxf(mx, dpp<kDppXor1>(mx));
      mx = fmaxf(mx, dpp<kDppXor2>(mx));
      mx = fmaxf(mx, dpp<kDppRor4>(mx));
      mx = fmaxf(mx, dpp<kDppRor8>(mx));
      const int e = norm_exponent(mx);
      const float dn = pow2f(-e);
#pragma unroll
      for (int i = 0; i < 4; ++i) { va[i] *= dn; vb[i] *= dn; }
      float sum;
      const uint4 o = block_operand<BITS>(va, vb, sum);
      sum += dpp<kDppXor1>(sum);
      sum += dpp<kDppXor2>(sum);
      if (m < item.n) {
        const size_t g = (size_t)(item.g0 + m);          // HQ, HS, HK are in grouped order
        *(uint4*)(G.HQ + (g * NU + u) * 256 + (tid & 15) * 16) = o;
        if ((tid & 15) == 0) G.HS[g * NU + u] = pow2f(e);
        if (qk == 0) G.HK[(g * NU + u) * 4 + b] = sum * -code_half<BITS>();
      }
    }
    __syncthreads();
  }
}

// The workgroup's item (its number is blockIdx.y), n = 0 where there is none: one memory round trip.
__device__ __forceinline__ GrpItem load_item(const GrpArgs& G) {
  const int count = *G.n_items;
  GrpItem it = G.items[blockIdx.y];
  it.n = (int)blockIdx.y < count ? it.n : 0;
  it.n = __builtin_amdgcn_readfirstlane(it.n);
  it.g0 = __builtin_amdgcn_readfirstlane(it.g0);
  it.bits = __builtin_amdgcn_readfirstlane(it.bits);
  return it;
}

template <int G4, int NT>
__global__ __launch_bounds__(kGThreads, 4) void k_grp_in(GrpArgs G) {
  extern __shared__ __attribute__((aligned(16))) char gsm[];
  const GrpItem item = load_item(G);
  if (item.n == 0) return;
  if (item.bits == 2) grp_in<2, G4, NT>(G, item, gsm);
  else if (item.bits == 4) grp_in<4, G4, NT>(G, item, gsm);
  else grp_in<8, G4, NT>(G, item, gsm);
}

// ---------------------------------------------------------------------------------------------
// W_out, columns [blockIdx.z * kGChunk, + kGChunk) of d_ff, rows [blockIdx.x * rows_per_wg, ...), one item. The chunk's
// operands go HBM -> LDS directly. h has one exponent per 128 columns, so the sums of 128 columns (inner) are scaled
// into acc.
template <int BITS, int G4, bool COLS, int NT>
__device__ __forceinline__ void grp_out(const GrpArgs& G, const GrpItem& item, char* smem) {
  constexpr int AB = apply_blocks<BITS, G4>(), NB = load_blocks<BITS>(), kGTok = 16 * NT;
  const LayerDims& L = G.L;
  const int d = L.d_model, f = L.d_ff, group = L.group_out, ngt = f / group, gsh = group_shift(group);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, kb = lane >> 4;
  const int NU = (f + kGUnit - 1) / kGUnit;
  const int c_begin = blockIdx.z * kGChunk, cu0 = c_begin / kGUnit, cu = min(kGChunk / kGUnit, NU - cu0);   // 128-column units
  const int cb = cu * 4;                                                  // blocks of the chunk
  const int g_first = (int)div_group((uint32_t)c_begin, group, gsh);
  constexpr int kMaxBlocks = kGChunk / 32;
  const int ngc = chunk_groups(group);                                    // groups a chunk can touch, at most
  const GrpLds lds = grp_lds(NT, kMaxBlocks, COLS ? 0 : G.rows_per_wg, COLS ? 0 : ngc, false);
  uint4* A = (uint4*)(smem + lds.a);
  float* KS = (float*)(smem + lds.ks);
  float* HS = (float*)(smem + lds.up);                                    // [unit][pair]
  uint16_t* SC = (uint16_t*)(smem + lds.scales);
  const int row_begin = blockIdx.x * G.rows_per_wg, row_end = min(d, row_begin + G.rows_per_wg);
  if (row_begin >= row_end) return;
  const uint8_t* q = uniform_ptr(item.q_out);
  const int nt = (item.n + 15) / 16;

  // operands: lane (m, kb) of operand (block, tile) takes 16 bytes of pair 16 t + m (absent pairs repeat the last one)
  {
    const uint32_t a0 = (uint32_t)(uintptr_t)(MOEQ_LDS char*)A;
    for (int o = wave; o < cb * NT; o += kGWaves) {
      const int b = o / NT, t = o % NT;
      if (t < nt) {
        const size_t g = (size_t)(item.g0 + min(16 * t + n, item.n - 1));
        dma16(G.HQ + (g * NU + cu0) * 256 + b * 64 + kb * 16, a0 + (uint32_t)((b * NT + t) * 1024));
      }
    }
  }
  for (int i = tid; i < cb * kGTok; i += kGThreads) {
    const int b = i / kGTok, m = i % kGTok;
    const size_t g = (size_t)(item.g0 + min(m, item.n - 1));
    if (b % AB == 0) {
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < AB; ++j) s += G.HK[(g * NU + cu0) * 4 + b + j];
      KS[b * kGTok + m] = s;
    }
    if ((b & 3) == 0) HS[(b >> 2) * kGTok + m] = G.HS[g * NU + cu0 + (b >> 2)];
  }
  float* part = G.part + (size_t)blockIdx.z * (size_t)G.M * d;
  if constexpr (!COLS) {
    stage_scales(item.s_out, d, ngt, row_begin, G.rows_per_wg, g_first, ngc, SC);
    const uint32_t row_bytes = (uint32_t)f * BITS / 8u, pieces = row_bytes / 16u, p0 = (uint32_t)c_begin * BITS / 128u;
    const int SPU = (cb + NB - 1) / NB;                   // loads per row block
    const int SLOTS = (SPU + kGRing - 1) / kGRing * kGRing;
    const int u0 = row_begin / kGUnit, u1 = (row_end + kGUnit - 1) / kGUnit;
    auto issue = [&](int u, int s) __attribute__((always_inline)) {
      const uint32_t row = (uint32_t)min(u * kGUnit + wave * 16 + n, d - 1);
      const uint32_t pc = min(p0 + (uint32_t)(4 * min(s, SPU - 1) + kb), pieces - 1u);
      return gload_u32x4(q + ((size_t)row * row_bytes + pc * 16u));
    };
    uint4 R[kGRing];
#pragma unroll
    for (int i = 0; i < kGRing; ++i) R[i] = issue(u0, i);
    stage_wait<kGRing>();
    __syncthreads();
    for (int u = u0; u < u1; ++u) {
      float inner[NT][4], acc[NT][4];
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) inner[t][i] = acc[t][i] = 0.f;
      const uint16_t* srow = SC + (u * kGUnit + wave * 16 + n - row_begin) * scale_stride(ngc);
      auto fold = [&](int unit) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (t < nt) {
            const float4 hs = *(const float4*)(HS + unit * kGTok + 16 * t + 4 * kb);
            const float hv[4] = {hs.x, hs.y, hs.z, hs.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              acc[t][i] = fmaf(inner[t][i], hv[i], acc[t][i]);
              inner[t][i] = 0.f;
            }
          }
        }
      };
      for (int s0 = 0; s0 < SLOTS; s0 += kGRing) {
#pragma unroll
        for (int i = 0; i < kGRing; ++i) {
          const int s = s0 + i;
          if (s < SPU) {
            half8_t B[NB];
            b_operands<BITS>(R[i], kb, B);
            if constexpr (BITS == 2) {                    // 256 columns per load: two units of h
              multiply_blocks<NT, AB, 0, 4>(B, s * NB, c_begin, nt, lane, kb, A, KS, srow, g_first, g_first + ngc - 1, group, gsh, inner);
              fold(2 * s);
              if (2 * s + 1 < cu) {
                multiply_blocks<NT, AB, 4, 4>(B, s * NB + 4, c_begin, nt, lane, kb, A, KS, srow, g_first, g_first + ngc - 1, group, gsh, inner);
                fold(2 * s + 1);
              }
            } else {
              constexpr int LPU = BITS == 4 ? 1 : 2;      // loads per 128 columns
              multiply_blocks<NT, AB, 0, NB>(B, s * NB, c_begin, nt, lane, kb, A, KS, srow, g_first, g_first + ngc - 1, group, gsh, inner);
              if ((s + 1) % LPU == 0) fold(s / LPU);
            }
          }
          const bool next = s + kGRing >= SLOTS;
          R[i] = issue(next ? min(u + 1, u1 - 1) : u, next ? s + kGRing - SLOTS : s + kGRing);
        }
      }
      const int row = u * kGUnit + wave * 16 + n;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = 16 * t + 4 * kb + i;
          if (m < item.n && row < d) part[(size_t)(item.g0 + m) * d + row] = acc[t][i] * kCodeUnit;
        }
    }
  } else {
    // word columns: lane (n, kb) loads a word of the rows 4 n .. 4 n + 3; operand i belongs to the rows 4 n + i. Rows are
    // taken 64 at a time per wavefront, blocks one after the other.
    constexpr int WPB = BITS;                             // words per block of 32 columns
    constexpr int LPB = BITS == 8 ? 2 : 1;                // 16-byte loads per block (2 bits: half of the quarters load the same word)
    const uint32_t col = (uint32_t)d * 4u;
    const uint8_t* sT = (const uint8_t*)uniform_ptr(item.s_out);
    const int words = f * BITS / 32;
    const int n_rb = (row_end - row_begin + 63) / 64;
    const int my_rb = wave < n_rb ? (n_rb - wave + kGWaves - 1) / kGWaves : 0;
    const int total = my_rb * cb;
    struct Slot { uint4 t[LPB]; uint2 s; };
    int ib = 0, ir = 0;                                   // block and row block the next request is for
    auto issue = [&](Slot& R) __attribute__((always_inline)) {
      const int r0 = min(row_begin + (wave + min(ir, max(my_rb - 1, 0)) * kGWaves) * 64 + 4 * n, d - 4);   // past the end: repeated
      const int w0 = (c_begin / 32 + ib) * WPB;
#pragma unroll
      for (int j = 0; j < LPB; ++j) {
        const int w = min(BITS == 4 ? w0 + kb : BITS == 2 ? w0 + (kb & 1) : w0 + 4 * (kb & 1) + 2 * (kb >> 1) + j, words - 1);
        R.t[j] = gload_u32x4(q + ((size_t)w * col + (uint32_t)r0 * 4u));
      }
      const int g = min((int)div_group((uint32_t)(c_begin + ib * 32), group, gsh), ngt - 1);
      R.s = gload_u32x2(sT + ((size_t)g * ((size_t)d * 2) + (uint32_t)r0 * 2u));
      if (++ib == cb) { ib = 0; ++ir; }
    };
    Slot R[kGRing];
#pragma unroll
    for (int i = 0; i < kGRing; ++i) issue(R[i]);
    stage_wait<kGRing>();
    __syncthreads();
    float inner[4][NT][4], acc[4][NT][4];
    int b0 = 0, cr = 0;                                   // block and row block being multiplied
    for (int s0 = 0; s0 < total; s0 += kGRing) {          // (cb is a multiple of four: a row block ends with a ring)
#pragma unroll
      for (int i = 0; i < kGRing; ++i) {
        const int b = b0 + i;
        if (i == 0 && b == 0) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
              for (int j = 0; j < 4; ++j) acc[r][t][j] = 0.f;
        }
        if (i == 0) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
              for (int j = 0; j < 4; ++j) inner[r][t][j] = 0.f;
        }
        const uint32_t s4[4] = {R[i].s.x & 0xffffu, R[i].s.x >> 16, R[i].s.y & 0xffffu, R[i].s.y >> 16};
        auto word = [&](int j, int r) { return r == 0 ? R[i].t[j].x : r == 1 ? R[i].t[j].y : r == 2 ? R[i].t[j].z : R[i].t[j].w; };
        half8_t B[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (BITS == 4) B[r] = codes8_4(word(0, r));
          else if constexpr (BITS == 2) B[r] = codes8_2(word(0, r), kb);
          else B[r] = codes8_8(word(0, r), word(LPB - 1, r));
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (t < nt) {
            const half8_t a = as_half8(A[(b * NT + t) * 64 + lane]);
            const float4 k4 = *(const float4*)(KS + b * kGTok + 16 * t + 4 * kb);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float4_t D = mfma16(a, B[r], (float4_t){k4.x, k4.y, k4.z, k4.w});
              const float sc = f16_bits_to_f32(s4[r]);
#pragma unroll
              for (int j = 0; j < 4; ++j) inner[r][t][j] = fmaf(D[j], sc, inner[r][t][j]);
            }
          }
        }
        if (i == kGRing - 1) {                            // four blocks: 128 columns of h
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const float4 hs = *(const float4*)(HS + (b >> 2) * kGTok + 16 * t + 4 * kb);
            const float hv[4] = {hs.x, hs.y, hs.z, hs.w};
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
              for (int j = 0; j < 4; ++j) acc[r][t][j] = fmaf(inner[r][t][j], hv[j], acc[r][t][j]);
          }
          if (b == cb - 1) {
            const int row = row_begin + (wave + cr * kGWaves) * 64 + 4 * n;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                const int m = 16 * t + 4 * kb + j;
                if (m < item.n && row < row_end)
                  *(float4*)(part + (size_t)(item.g0 + m) * d + row) =
                      make_float4(acc[0][t][j] * kCodeUnit, acc[1][t][j] * kCodeUnit, acc[2][t][j] * kCodeUnit, acc[3][t][j] * kCodeUnit);
              }
          }
        }
        issue(R[i]);
      }
      b0 += kGRing;
      if (b0 == cb) { b0 = 0; ++cr; }
    }
  }
}

template <int G4, bool COLS, int NT>
__global__ __launch_bounds__(kGThreads, COLS && NT == 2 ? 2 : 4) void k_grp_out(GrpArgs G) {
  extern __shared__ __attribute__((aligned(16))) char gsm[];
  const GrpItem item = load_item(G);
  if (item.n == 0) return;
  // in columns a block is one application of the scale, whatever the group
  if (item.bits == 2) grp_out<2, COLS ? 1 : G4, COLS, NT>(G, item, gsm);
  else if (item.bits == 4) grp_out<4, COLS ? 1 : G4, COLS, NT>(G, item, gsm);
  else grp_out<8, COLS ? 1 : G4, COLS, NT>(G, item, gsm);
}

// y[t][r] = sum_j gate[t][j] * sum_c part[c][ginv[t k + j]][r], chunks and choices in order
__global__ __launch_bounds__(256) void k_grp_combine(const float* __restrict__ part, const int32_t* __restrict__ ginv,
                                                     const float* __restrict__ gate, int chunks, int M, int k, int d,
                                                     float* __restrict__ y) {
  const int t = blockIdx.x;
  for (int r = threadIdx.x * 4; r < d; r += 1024) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int j = 0; j < k; ++j) {
      const float* p = part + (size_t)ginv[(size_t)t * k + j] * d + r;
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
      for (int c = 0; c < chunks; ++c) {
        const float4 w = *(const float4*)(p + (size_t)c * M * d);
        a.x += w.x; a.y += w.y; a.z += w.z; a.w += w.w;
      }
      const float g = gate[(size_t)t * k + j];
      v.x = fmaf(g, a.x, v.x); v.y = fmaf(g, a.y, v.y); v.z = fmaf(g, a.z, v.z); v.w = fmaf(g, a.w, v.w);
    }
    float* o = y + (size_t)t * d + r;
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
  }
}

constexpr int kGLdsMost = 160 * 1024;

int grp_in_lds(const LayerDims& L, int nt, int rows) { return grp_lds(nt, padded_blocks(L.d_model), rows, L.d_model / L.group, true).total; }
int grp_out_lds(const LayerDims& L, int nt, int rows, bool cols) {
  return grp_lds(nt, kGChunk / 32, cols ? 0 : rows, cols ? 0 : chunk_groups(L.group_out), false).total;
}

template <int NT>
void (*grp_in_kernel(int g4))(GrpArgs) { return g4 == 4 ? k_grp_in<4, NT> : g4 == 2 ? k_grp_in<2, NT> : k_grp_in<1, NT>; }
template <int NT>
void (*grp_out_kernel(int g4, bool cols))(GrpArgs) {
  return cols ? k_grp_out<1, true, NT> : g4 == 4 ? k_grp_out<4, false, NT> : g4 == 2 ? k_grp_out<2, false, NT> : k_grp_out<1, false, NT>;
}

// Items of one tile where an expert has less than 12 pairs on average. Not a fitted line; us, one tile / two: Switch-base layer
// (2, 4, 8 bits) of 64 experts 69 / 79 for 4 pairs an expert, 88 / 98 for 12, 157 / 165 for 30, 564 / 550 for 125, with 8 bits
// 217 / 194 for 30; of 8 experts 404 / 382 for 1000; Switch-large layer of 33 experts 57 / 73 for 4, 84 / 103 for 15, 716 / 831
// for 240. Two tiles pay on narrow layers with 8-bit experts or many pairs.
inline int tiles_of(const LayerDims& L, int64_t M) { return M < 12 * (int64_t)L.n_experts ? 1 : kGMaxTiles; }

inline int g4_of(int group) { return group % 128 == 0 ? 4 : (group % 64 == 0 ? 2 : 1); }

}  // namespace

bool group_supported(const LayerDims& L) {
  return L.act == MOEQ_ACT_RELU && L.d_model % 32 == 0 && padded_blocks(L.d_model) <= kGMaxBlocks && L.d_ff % 32 == 0 && L.n_experts <= 1024 &&
         grp_in_lds(L, kGMaxTiles, kGUnit) <= kGLdsMost && grp_out_lds(L, kGMaxTiles, kGUnit, false) <= kGLdsMost;
}

int group_max_pairs() { return kGMaxPairs; }

GroupWs group_ws(const LayerDims& L, int64_t M) {
  GroupWs w{};
  const size_t NU = ((size_t)L.d_ff + kGUnit - 1) / kGUnit, chunks = ((size_t)L.d_ff + kGChunk - 1) / kGChunk, P = (size_t)M;
  size_t off = 0;
  w.items = off;   off += up256((P / 16 + (size_t)L.n_experts + 1) * sizeof(GrpItem));
  w.n_items = off; off += 256;
  w.gpair = off;   off += up256(P * 4);
  w.ginv = off;    off += up256(P * 4);
  w.hq = off;      off += up256(P * NU * 256);
  w.hs = off;      off += up256(P * NU * 4);
  w.hk = off;      off += up256(P * NU * 16);
  w.part = off;    off += up256(chunks * P * (size_t)L.d_model * 4);
  w.total = off;
  return w;
}

hipError_t init_attrs_group_gemm() {
  for (int g4 = 1; g4 <= 4; g4 *= 2)
    for (int cols = 0; cols < 2; ++cols)
      for (const void* k : {(const void*)grp_in_kernel<1>(g4), (const void*)grp_in_kernel<2>(g4), (const void*)grp_out_kernel<1>(g4, cols),
                            (const void*)grp_out_kernel<2>(g4, cols)})
        if (hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kGLdsMost); e != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_group(const LayerDims& L, const DevExpert* table, const void* x, int32_t T, const int32_t* idx,
                        const float* gate, char* ws, bool out_columns, float* y, hipStream_t st, const Prof& prof) {
  const int M = T * L.top_k;
  if (!group_supported(L) || T < 1 || M > kGMaxPairs) return hipErrorInvalidValue;
  const GroupWs w = group_ws(L, M);
  const int nt = tiles_of(L, M);
  const int NU = (L.d_ff + kGUnit - 1) / kGUnit, chunks = (L.d_ff + kGChunk - 1) / kGChunk;
  GrpArgs G{L, table, x, idx, M, L.top_k, (GrpItem*)(ws + w.items), (int32_t*)(ws + w.n_items),
            (int32_t*)(ws + w.gpair), (int32_t*)(ws + w.ginv), (uint8_t*)(ws + w.hq), (float*)(ws + w.hs), (float*)(ws + w.hk),
            (float*)(ws + w.part), 16 * nt, 0};
  const int max_items = M < L.n_experts + M / (16 * nt) ? M : L.n_experts + M / (16 * nt);
  prof_start(prof, MOEQ_KERNEL_FUSED, st);
  hipLaunchKernelGGL(k_grp_plan, dim3(L.n_experts), dim3(256), 0, st, G);
  // rows per workgroup: enough workgroups for the chip (three per compute unit), no more: each stages the item's activations
  constexpr int lds_want = kGLdsMost / 2;      // two workgroups on a compute unit (their registers allow no third)
  const int want = (768 + max_items - 1) / max_items;
  int gx = want < NU ? want : NU;
  int rows = (NU + gx - 1) / gx * kGUnit;
  while (rows > kGUnit && grp_in_lds(L, nt, rows) > lds_want) rows -= kGUnit;
  gx = (L.d_ff + rows - 1) / rows;
  G.rows_per_wg = rows;
  prof_start(prof, MOEQ_KERNEL_FFN_IN, st);
  hipLaunchKernelGGL(nt == 1 ? grp_in_kernel<1>(g4_of(L.group)) : grp_in_kernel<2>(g4_of(L.group)), dim3(gx, max_items), dim3(kGThreads),
                     grp_in_lds(L, nt, rows), st, G);
  prof_stop(prof, MOEQ_KERNEL_FFN_IN, st);
  const int unit = out_columns ? 64 * kGWaves : kGUnit, nu2 = (L.d_model + unit - 1) / unit;
  const int want2 = (768 + max_items * chunks - 1) / (max_items * chunks);
  gx = want2 < nu2 ? want2 : nu2;
  rows = (nu2 + gx - 1) / gx * unit;
  while (rows > unit && grp_out_lds(L, nt, rows, out_columns) > lds_want) rows -= unit;
  gx = (L.d_model + rows - 1) / rows;
  G.rows_per_wg = rows;
  prof_start(prof, MOEQ_KERNEL_FFN_OUT, st);
  hipLaunchKernelGGL(nt == 1 ? grp_out_kernel<1>(g4_of(L.group_out), out_columns) : grp_out_kernel<2>(g4_of(L.group_out), out_columns),
                     dim3(gx, max_items, chunks), dim3(kGThreads), grp_out_lds(L, nt, rows, out_columns), st, G);
  prof_stop(prof, MOEQ_KERNEL_FUSED, st);
  hipLaunchKernelGGL(k_grp_combine, dim3(T), dim3(256), 0, st, G.part, G.ginv, gate, chunks, M, L.top_k, L.d_model, y);
  prof_stop(prof, MOEQ_KERNEL_FFN_OUT, st);
  return hipGetLastError();
}

}  // namespace moeq
