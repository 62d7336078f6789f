// Decode calls of a few tokens on a layer of 4096-column experts with scale groups of 128, in any layout (a batch of
// sequences decoded together): the (token, choice) pairs are grouped by expert, and every expert's packed weights are
// streamed ONCE for up to 16 of its pairs (8 on layers that are not in the stream layout), against all of them on the
// matrix cores (Section 2.1: only the chosen experts work on a token; Section 3.2: the codes are decompressed by the mirror
// of the linear quantization - here they stay integers all the way into the multiplier).
//
// Arithmetic: that of decode_stream.hip. The activations of a scale group (128 columns) are block-floating-point
// integers, given as signed bytes; codes enter as bytes (2- and 4-bit codes with their offset, which is taken off with the
// group's sum of x_int; 8-bit codes made signed by one XOR). v_mfma_i32_16x16x64_i8 gives the exact integer sums of 16
// rows of activations x 16 rows of weights; per group sum * scale * 2^e in fp32, 2^e last and in the addition's fused
// multiply: sum * 2^e alone leaves fp32 from hidden states of about 2^108 on.
//   Stream layers: 15 bits below the largest and a sign, x_int = lo + 256 hi; an activation row per pair. h has one exponent
//   per 64 columns (an operand), as in k_moe_stream: with one per 128 an output of which the larger half met zero weights
//   was off by 8.5e-2 instead of 2e-4 when the halves differed by 2^10.
//   Other layers: 30 bits and a sign, in two such parts that are two rows of the operand (x_int = low + 2^16 high), so 8
//   pairs fill it. Their single-token kernels hold x and h as binary16, 11 bits of every element whatever its neighbours
//   are, and 15 bits below the largest are not that: where a column with activations 2^10 times the others of its group
//   meets zero weights, an output of 4-bit experts was off by 2.9e-2 (5.7e-4 token by token; now 8e-7, and 2.1e-7 instead
//   of 7.7e-5 on normally distributed inputs). The price is a second pass over the weights of experts with 9 to 16 pairs:
//   Mixtral layer in rows, 31 tokens 177 -> 232 us (669 token by token), 23 tokens 174 -> 180, up to 16 tokens within 3 %.
//
// Kernels (launch_moe_batch):
//   k_batch_prep     per token: router + top-k, x as byte digits in the operand order of every bitwidth of the layer
//   k_batch_in       W_in / W_gate, activation, h as byte digits (a unit of 128 rows is one scale group of W_out)
//   k_batch_out      W_out over 1024 columns of d_ff, partial outputs per pair
//   k_batch_combine  y[t] = sum_j gate_j * (sum of the pair's partial outputs), in a fixed order
//
// What bounds it: the bytes of the distinct experts. With one workgroup per (slice, token), as for a single token, a
// call of T tokens pays T times the unpack arithmetic. Mixtral layer (8 experts, 2 / 4 bits, d_ff 14336): 8 tokens
// 230 -> 117-144 us (by the experts they touch), 23 tokens 640 -> 148 us (550 MB: 3.7 TB/s over the whole call; k_batch_in 95,
// k_batch_out 46-48, the two small kernels 6.5 and 5); canonical layout 204 -> 170 and 23 tokens 846 -> 180. Where grouping pays: batch_pays (api.cpp).
#include <hip/hip_ext.h>

#include "decode_core.h"

namespace moeq {
namespace {

constexpr int kBD = 4096;                 // d_model
constexpr int kBGroup = 128;              // scale group of all matrices
constexpr int kBGroups = kBD / kBGroup;   // scale groups of a row of W_in
constexpr int kBRows = 16;                // rows of an A operand (columns of the matrix instruction)
// Pairs of a work item. Stream layers: one row per pair. Other layers: two, the low and the high half of its integers.
__host__ __device__ constexpr int batch_parts(bool stream) { return stream ? 1 : 2; }
__host__ __device__ constexpr int batch_tok(bool stream) { return kBRows / batch_parts(stream); }
constexpr int kBWaves = 8;                // wavefronts of a k_batch_in workgroup
constexpr int kBOutGroups = 8;            // scale groups of d_ff a k_batch_out workgroup takes
constexpr int kBOutRows = 256;            // output rows a k_batch_out workgroup takes (64 per wavefront)
constexpr int kBInlineMaxE = 64;          // the router runs inside k_batch_prep for at most this many experts

typedef int i32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ i32x4_t mfma_i8(const i32x4_t& a, const i32x4_t& b, const i32x4_t& c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// The 128 columns of a scale group are two operands (op) of 64; lane (m or n = l % 16, kb = l / 16) holds 16 of an
// operand's columns, byte j of them being column operand_col(..., j) of the group: W_in / W_gate in the stream layout, in
// the canonical one; W_out in columns. Rows of W_out in the canonical layout are read like those of W_in. Two swapped
// halves of a wavefront (swap32) stand behind the (kb & 1, kb >> 1) forms.
enum BatchOrder { BO_STREAM = 0, BO_ROWS = 1, BO_COLUMNS = 2 };
template <int BITS, int ORDER>
__device__ __forceinline__ int operand_col(int op, int kb, int j) {
  const int in8 = 2 * (j & 3) + ((j >> 2) & 1);                      // byte j of two words of eight 4-bit codes
  if constexpr (ORDER == BO_STREAM) {
    if constexpr (BITS == 4) return 64 * (kb & 1) + 32 * (kb >> 1) + 16 * op + 8 * (j >> 3) + in8;
    else if constexpr (BITS == 2) return 64 * (kb & 1) + 16 * (kb >> 1) + 32 * op + 4 * (j & 3) + (j >> 2);
    else return 64 * (kb & 1) + 16 * (kb >> 1) + 32 * op + j;
  } else if constexpr (ORDER == BO_ROWS) {
    if constexpr (BITS == 4) return 32 * kb + 16 * op + 8 * (j >> 3) + in8;
    else if constexpr (BITS == 2) return 64 * (kb & 1) + 16 * (kb >> 1) + 32 * op + 4 * (j & 3) + (j >> 2);
    else return 64 * op + 16 * kb + j;
  } else {
    if constexpr (BITS == 4) return 64 * op + 32 * (j >> 3) + 8 * kb + in8;
    else if constexpr (BITS == 2) return 64 * op + 16 * kb + 4 * (j & 3) + (j >> 2);
    else return 64 * op + 16 * (j >> 2) + 4 * kb + (j & 3);
  }
}

// 16 codes as operand bytes: from two words (4 bits), one word (2 bits), four words (8 bits)
__device__ __forceinline__ i32x4_t codes16_4(uint32_t w0, uint32_t w1) {
  return (i32x4_t){(int)(w0 & 0x0f0f0f0fu), (int)((w0 >> 4) & 0x0f0f0f0fu), (int)(w1 & 0x0f0f0f0fu), (int)((w1 >> 4) & 0x0f0f0f0fu)};
}
__device__ __forceinline__ i32x4_t codes16_2(uint32_t w) {
  return (i32x4_t){(int)(w & 0x03030303u), (int)((w >> 2) & 0x03030303u), (int)((w >> 4) & 0x03030303u), (int)((w >> 6) & 0x03030303u)};
}
__device__ __forceinline__ i32x4_t codes16_8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  return (i32x4_t){(int)(a ^ 0x80808080u), (int)(b ^ 0x80808080u), (int)(c ^ 0x80808080u), (int)(d ^ 0x80808080u)};
}
// what a code's offset adds to a dot product, in units of the sum of x_int
template <int BITS> constexpr int code_offset() { return BITS == 8 ? 0 : 1 << (BITS - 1); }

__device__ __forceinline__ uint32_t lo_byte(int v) { return (uint32_t)v & 255u; }
__device__ __forceinline__ uint32_t hi_byte(int v) { return (uint32_t)((v + 128) >> 8) & 255u; }

// A work item: up to batch_tok() pairs of one expert.
struct alignas(16) BatchItem { int32_t e, n; uint8_t pair[kBRows]; int32_t bits, pad; };
static_assert(sizeof(BatchItem) == 32, "two 16-byte pieces");

struct BatchArgs {
  LayerDims L;
  const DevExpert* table;
  const float* Wr;
  const float* bias;
  const void* x;
  int32_t T, k, fixed_expert, bits_mask, route_inline, out_columns;
  int32_t* idx;          // [T][k] written by k_batch_prep (route_inline) or read (unused with a fixed expert)
  float* gate;           // [T][k] likewise
  uint8_t* XQ;           // [bitwidths][T][kBGroups][op][part][digit][kb][16]: x as operand bytes
  float* XS;             // [T][kBGroups] 2^e of every group (NaN: the group holds a non-finite value)
  int32_t* XSUM;         // [T][kBGroups][part] sum of the part of x_int
  uint8_t* HQ;           // [pairs][d_ff / 128][op][part][digit][kb][16]: h likewise, in the order of its expert's bitwidth
  float* HS;             // [pairs][d_ff / 128][2]: of both halves of the group's columns (other than stream layers: the same)
  int32_t* HSUM;         // [pairs][d_ff / 128][2]: of both halves; other than stream layers: of both parts
  BatchItem* items;      // written by workgroup 0 of k_batch_in
  int32_t* n_items;
  float* part;           // [d_ff / 1024 rounded up][pairs][d_model]
};

__device__ __forceinline__ int bits_slot(int mask, int bits) {
  return __popc((unsigned)mask & ((unsigned)bits - 1u) & 14u);      // bitwidths 2, 4, 8 are the bits of the mask
}

// Maximum / sum over the LANES (16: a DPP row, or 8) that share an exponent, in every one of them.
template <int LANES>
__device__ __forceinline__ float lanes_max(float m) {
  m = fmaxf(m, dpp<kDppXor1>(m));
  m = fmaxf(m, dpp<kDppXor2>(m));
  if constexpr (LANES == 8) return fmaxf(m, dpp<kDppHalfMirror>(m));
  m = fmaxf(m, dpp<kDppRor4>(m));
  return fmaxf(m, dpp<kDppRor8>(m));
}
template <int LANES>
__device__ __forceinline__ int lanes_sum(int v) {
  v += dppi<kDppXor1>(v);
  v += dppi<kDppXor2>(v);
  if constexpr (LANES == 8) return v + dppi<kDppHalfMirror>(v);
  v += dppi<kDppRor4>(v);
  return v + dppi<kDppRor8>(v);
}
// x_int of eight values of the columns that LANES lanes share, and what its parts hold of it; returns 2^e (NaN if a value of
// these columns is not finite, x_int = 0 then) and the sums of the parts over them.
template <int PARTS, int LANES>
__device__ __forceinline__ float group_ints(const float (&v)[8], int (&part)[PARTS][8], int (&sum)[PARTS]) {
  float m = 0.f;
  bool bad = false;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    m = fmaxf(m, fabsf(v[i]));
    bad = bad || !(fabsf(v[i]) < INFINITY);
  }
  m = lanes_max<LANES>(bad ? INFINITY : m);
  // one part: the largest magnitude m * 2^-e lies in [2^14, 32639], what a signed byte pair holds (one bit more than the
  // digits of k_moe_stream). Two: in [2^29, 2^30), and the low part in [-32896, 32639]
  int e = 0;
  if (m > 0.f && m < INFINITY) {
    e = __builtin_amdgcn_frexp_expf(m) - (PARTS == 1 ? 15 : 30);
    if (PARTS == 1) e += m * pow2f(min(max(-e, -120), 120)) > 32639.f ? 1 : 0;
  }
  e = min(max(e, -120), 120);
  const float dn = pow2f(-e);
#pragma unroll
  for (int p = 0; p < PARTS; ++p) sum[p] = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    int xi = m < INFINITY ? __float2int_rn(v[i] * dn) : 0;
    if constexpr (PARTS == 2) {
      part[1][i] = (xi + 32896) >> 16;
      sum[1] += part[1][i];
      xi -= part[1][i] * 65536;
    }
    part[0][i] = xi;
    sum[0] += xi;
  }
#pragma unroll
  for (int p = 0; p < PARTS; ++p) sum[p] = lanes_sum<LANES>(sum[p]);
  return m < INFINITY ? pow2f(e) : __builtin_nanf("");
}

// ---------------------------------------------------------------------------------------------
// Workgroup = one token, thread t holds columns 8 t .. 8 t + 7. The router's sums are those of k_moe_stream, term by
// term, so a token's routing does not depend on how many tokens share its call.
template <bool STREAM>
__global__ __launch_bounds__(512) void k_batch_prep(BatchArgs G) {
  constexpr int PARTS = batch_parts(STREAM);
  __shared__ __align__(16) int16_t XI[PARTS][kBD];
  __shared__ float rpart[kBWaves * kBInlineMaxE];
  __shared__ float lg[kBInlineMaxE];
  const LayerDims& L = G.L;
  const int token = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, E = L.n_experts;
  const XItem xit = load_x_item((const char*)G.x + (size_t)token * kBD * (L.x_bf16 ? 2 : 4), L.x_bf16 ? X_BF16 : X_F32, tid);
  auto stage = [&]() __attribute__((always_inline)) {
    int part[PARTS][8], sum[PARTS];
    const float s = group_ints<PARTS, 16>(xit.v, part, sum);
    if ((tid & 15) == 0) G.XS[(size_t)token * kBGroups + (tid >> 4)] = s;
#pragma unroll
    for (int p = 0; p < PARTS; ++p) {
      if ((tid & 15) == 0) G.XSUM[((size_t)token * kBGroups + (tid >> 4)) * PARTS + p] = sum[p];
      uint32_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = ((uint32_t)part[p][2 * i] & 0xffffu) | ((uint32_t)part[p][2 * i + 1] << 16);
      ((uint4*)XI[p])[tid] = make_uint4(w[0], w[1], w[2], w[3]);
    }
  };
  bool staged = false;
  if (G.route_inline) {
    for (int e0 = 0; e0 < E; e0 += 8) {
      float4 w[8][2];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float* wr = G.Wr + (size_t)min(e0 + i, E - 1) * kBD + 8 * tid;     // rows past E repeat the last one
        w[i][0] = *(const float4*)wr;
        w[i][1] = *(const float4*)(wr + 4);
      }
      if (!staged) { stage(); staged = true; }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float acc = w[i][0].x * xit.v[0];
        acc = fmaf(w[i][0].y, xit.v[1], acc); acc = fmaf(w[i][0].z, xit.v[2], acc); acc = fmaf(w[i][0].w, xit.v[3], acc);
        acc = fmaf(w[i][1].x, xit.v[4], acc); acc = fmaf(w[i][1].y, xit.v[5], acc);
        acc = fmaf(w[i][1].z, xit.v[6], acc); acc = fmaf(w[i][1].w, xit.v[7], acc);
        acc = wave_sum(acc);
        if (lane == 0 && e0 + i < E) rpart[wave * kBInlineMaxE + e0 + i] = acc;
      }
    }
  }
  if (!staged) stage();
  __syncthreads();
  if (G.route_inline && wave == 0) {
    int* se = G.idx + (size_t)token * L.top_k;
    float* sg = G.gate + (size_t)token * L.top_k;
    if (lane < E) {
      float t = rpart[lane];
#pragma unroll
      for (int wv = 1; wv < kBWaves; ++wv) t += rpart[wv * kBInlineMaxE + lane];
      lg[lane] = t + (G.bias ? G.bias[lane] : 0.f);
    }
    if (E <= 8 && L.top_k <= 2) topk_tiny<8>(lg, E, L.top_k, L.renorm, lane, se, sg);
    else if (E <= 16 && L.top_k <= 2) topk_tiny<16>(lg, E, L.top_k, L.renorm, lane, se, sg);
    else topk_from_logits(lg, E, L.top_k, L.renorm, lane, se, sg, nullptr);
  }
  // the operand bytes: 256 pieces of 16 columns per bitwidth and part, both digits of a piece by one thread
  auto pieces = [&](auto bits_tag) __attribute__((always_inline)) {
    constexpr int BITS = decltype(bits_tag)::value, ORDER = STREAM ? BO_STREAM : BO_ROWS;
    uint8_t* out = G.XQ + ((size_t)bits_slot(G.bits_mask, BITS) * G.T + token) * (PARTS * 2 * kBD);
    for (int i = tid; i < PARTS * (kBD / 16); i += 512) {
      const int p = i / (kBD / 16), pc = i % (kBD / 16);
      const int g = pc >> 3, op = (pc >> 2) & 1, kb = pc & 3;
      uint32_t lo[4] = {0u, 0u, 0u, 0u}, hi[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int v = XI[p][g * kBGroup + operand_col<BITS, ORDER>(op, kb, j)];
        lo[j >> 2] |= lo_byte(v) << (8 * (j & 3));
        hi[j >> 2] |= hi_byte(v) << (8 * (j & 3));
      }
      uint4* dst = (uint4*)(out + (size_t)((g * 2 + op) * PARTS + p) * 128 + kb * 16);
      dst[0] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
      dst[4] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    }
  };
  if (G.bits_mask & 2) pieces(std::integral_constant<int, 2>{});
  if (G.bits_mask & 4) pieces(std::integral_constant<int, 4>{});
  if (G.bits_mask & 8) pieces(std::integral_constant<int, 8>{});
}

// ---------------------------------------------------------------------------------------------
// Groups the pairs of the call by expert into items (first come, first served; TOK pairs each), in LDS. Every thread of
// a workgroup of 512 calls it. O(pairs) broadcast reads per pair: a call has at most kBatchMaxPairs of them.
struct BatchLists {
  int32_t pe[kBatchMaxPairs];
  int32_t rank[kBatchMaxPairs];
  int32_t it[kBatchMaxPairs];
  int32_t wcnt[kBatchMaxPairs / 64];
  BatchItem items[kBatchMaxPairs];
};
template <int TOK>
__device__ __forceinline__ int batch_items(const BatchArgs& G, BatchLists& S) {
  const int p = threadIdx.x, P = G.T * G.k, E = G.L.n_experts;
  const int lane = p & 63, wave = p >> 6;
  int e = -1;
  if (p < P) {
    e = G.fixed_expert >= 0 ? G.fixed_expert : min(max(G.idx[p], 0), E - 1);
    S.pe[p] = e;
  }
  __syncthreads();
  int r = 0, total = 0;
  if (p < P) {
#pragma unroll 4
    for (int q = 0; q < P; ++q) {
      const int same = S.pe[q] == e ? 1 : 0;
      total += same;
      r += q < p ? same : 0;
    }
    S.rank[p] = r;
  }
  const bool first = p < P && (r & (TOK - 1)) == 0;
  const unsigned long long mask = __ballot(first);
  if (lane == 0 && wave < kBatchMaxPairs / 64) S.wcnt[wave] = __popcll(mask);
  __syncthreads();
  int n_items = 0, before = 0;
  for (int w = 0; w < kBatchMaxPairs / 64; ++w) {
    before += w < wave ? S.wcnt[w] : 0;
    n_items += S.wcnt[w];
  }
  if (first) {
    const int i = before + __popcll(mask & ((1ull << lane) - 1ull));
    S.it[p] = i;
    S.items[i].e = e;
    S.items[i].n = min(TOK, total - r);
    S.items[i].bits = G.table[e].bits;
  }
  __syncthreads();
  if (p < P) {
    int mine = 0;
#pragma unroll 4
    for (int q = 0; q < P; ++q)
      if (S.pe[q] == e && S.rank[q] == (r & ~(TOK - 1))) mine = q;
    const int i = S.it[mine];
    S.items[i].pair[r & (TOK - 1)] = (uint8_t)p;
  }
  __syncthreads();
  return n_items;
}

// A register set of k_batch_in: eight 16-byte loads (NH steps of 256 columns of NM matrices) and their scales.
template <int BITS, int NM>
struct BatchSet {
  static constexpr int LPS = BITS / 2 * NM;        // loads per 256 columns
  static constexpr int NH = 8 / LPS;               // 256-column steps
  static constexpr int GS = 2 * NH;                // scale groups
  static constexpr int NS = (GS + 3) / 4;          // scale words per matrix: lane (n, kb) holds group 4 i + kb of row n
  static constexpr int SPU = kBD / 256 / NH;       // sets per row block
  uint4 t[8];
  uint32_t s[NM][NS];
};

struct BatchInLds {
  uint4 A[kBGroups * 4][64];           // operand (g, op, digit): lane's 16 bytes
  float XS[kBGroups][kBRows];          // 2^e of every row (a high part's is 2^16 times its low part's)
  int32_t SX[kBGroups][kBRows];        // minus the code offset times the sum of the row's integers
  float H[2][kBRows][kBGroup + 4];     // h of a unit's rows, two units in turn
  BatchLists lists;
};

// Units [u0, u1) (128 rows of W_in / W_gate each) of one item. Wavefront w owns rows 16 w .. 16 w + 15 of a unit. Lane
// (n, kb) loads the 16-byte pieces 4 h + kb of row n: 64 consecutive bytes of 16 rows per load, the other half of the
// 128-byte lines with the next step's (5.6 TB/s as a bare access pattern with 16 loads per lane in flight, against 6.1
// for whole 1 KB tiles, which would have to be transposed through LDS). Stream layout: a scale group is two pieces of all
// the row's tiles, and swapping half wavefronts between two loads puts a group's codes into all four kb. Canonical rows:
// the pieces of a row follow each other, 4 h' + kb with h' = (load of the row); only 2-bit codes (two groups a load) swap.
template <int BITS, int NM, bool SWIGLU, bool STREAM>
__device__ __forceinline__ void batch_in_units(const BatchArgs& G, BatchInLds& S, const BatchItem& item, int u0, int u1) {
  using Set = BatchSet<BITS, NM>;
  constexpr int RB = 16 / BITS, TPR = BITS / 2, TOK = batch_tok(STREAM), PARTS = batch_parts(STREAM);
  constexpr uint32_t BB = 8192u + 64u * RB;
  constexpr int LPM = BITS / 2;                    // loads of one matrix per 256 columns
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, kb = lane >> 4;
  const DevExpert* ex = G.table + item.e;
  const uint8_t* q[NM];
  q[0] = uniform_ptr(ex->q_in);
  if constexpr (NM == 2) q[1] = uniform_ptr(ex->q_gate);
  const uint8_t* sp[NM];                           // (the stream layout keeps the scales with the codes)
  sp[0] = STREAM ? q[0] : (const uint8_t*)uniform_ptr(ex->s_in);
  if constexpr (NM == 2) sp[1] = STREAM ? q[1] : (const uint8_t*)uniform_ptr(ex->s_gate);
  const int NG = G.L.d_ff / kBGroup;
  const uint8_t* xq = G.XQ + (size_t)bits_slot(G.bits_mask, BITS) * G.T * (PARTS * 2 * kBD);

  __syncthreads();          // every wavefront is done with the previous item's operands
  // the item's 16 activation rows into LDS, operand by operand (row m: pair m % TOK, part m / TOK; absent pairs repeat the
  // first one, their results are dropped)
  // (their factors are requested first and stored behind the first weights' requests, which wait for nothing)
  const int sg = threadIdx.x >> 4, sm = threadIdx.x & 15;         // 512 threads = 32 groups x 16 rows
  const size_t sat = (size_t)(item.pair[sm % TOK < item.n ? sm % TOK : 0] / G.k) * kBGroups + sg;
  const float sxs = G.XS[sat];
  const int32_t sxsum = G.XSUM[sat * PARTS + sm / TOK];
  {
    const int pm = item.pair[n % TOK < item.n ? n % TOK : 0];
    const uint8_t* src = xq + (size_t)(pm / G.k) * (PARTS * 2 * kBD) + (n / TOK) * 128 + kb * 16;
    const uint32_t a0 = (uint32_t)(uintptr_t)(MOEQ_LDS char*)&S.A[0][0];
#pragma unroll 4
    for (int i = 0; i < kBGroups * 4 / kBWaves; ++i) {
      const int o = wave + i * kBWaves;              // (operand op of a group, digit) = (o / 2, o % 2)
      dma16(src + (o >> 1) * (PARTS * 128) + (o & 1) * 64, a0 + (uint32_t)o * 1024u);
    }
  }
  const int total = (u1 - u0) * Set::SPU;
  auto issue = [&](Set& R, int s) __attribute__((always_inline)) {
    const bool live = s < total;                   // past the end: cached bytes, so that every path issues the same loads
    const uint32_t unit = (uint32_t)(u0 + s / Set::SPU), h0 = (uint32_t)(s % Set::SPU) * Set::NH;
    const uint32_t row = unit * 128u + (uint32_t)(wave * 16 + n);
    const uint32_t blk = row / RB, rr = row % RB;
    // stream: part `part` of step h at part * 1024 + h * 64 in the row's tiles; rows: load LPM h + part at 64 bytes each
    const uint32_t off = !live ? (uint32_t)lane * 16u
                       : STREAM ? blk * BB + rr * (TPR * 1024u) + (uint32_t)kb * 16u + h0 * 64u
                                : row * (kBD * BITS / 8) + (uint32_t)kb * 16u + h0 * (64u * LPM);
#pragma unroll
    for (int hh = 0; hh < Set::NH; ++hh)
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const uint8_t* b = live ? q[m] : xq;
#pragma unroll
        for (int part = 0; part < LPM; ++part)
          R.t[(hh * NM + m) * LPM + part] = gload_u32x4(b + (off + (uint32_t)(STREAM ? part * 1024 + hh * 64 : (hh * LPM + part) * 64)));
      }
    // scales: group g of the row. Stream layout: in the row's half of the block's scale area (8 bits: RB = 2, the word of a
    // group holds both rows), the word's half n & 1; rows: one binary16 value
    const uint32_t sg = blk * BB + 8192u + (BITS == 8 ? 0u : (rr / (RB > 1 ? RB / 2 : 1)) * RB + ((rr % (RB / 2 > 0 ? RB / 2 : 1)) >> 1) * 4u);
    const uint32_t sstep = STREAM ? 2u * RB : 2u;
    const uint32_t soff = !live ? (uint32_t)lane * 4u : (STREAM ? sg : row * (kBGroups * 2u)) + h0 * 2u * sstep;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const uint8_t* b = live ? sp[m] : xq;
#pragma unroll
      for (int i = 0; i < Set::NS; ++i) {
        const uint32_t g = Set::GS >= 4 ? 4 * i + kb : (kb & (Set::GS - 1));
        const uint8_t* a = b + (soff + (live ? g * sstep : 0u));
        R.s[m][i] = STREAM ? gload_u32(a) : gload_u16(a);
      }
    }
  };
  // the A operands of a group, read from LDS while the group before it is multiplied
  struct Operands { i32x4_t a[2][2], sx; float4 xs; };
  auto read_a = [&](int g) __attribute__((always_inline)) {
    Operands o;
#pragma unroll
    for (int op = 0; op < 2; ++op)
#pragma unroll
      for (int dg = 0; dg < 2; ++dg) o.a[op][dg] = __builtin_bit_cast(i32x4_t, S.A[(g * 2 + op) * 2 + dg][lane]);
    o.sx = *(const i32x4_t*)&S.SX[g][4 * kb];
    o.xs = *(const float4*)&S.XS[g][4 * kb];
    return o;
  };
  Operands cur;
  float acc[NM][4];
  auto consume = [&](const Set& R, int s) __attribute__((always_inline)) {
    const int h0 = (s % Set::SPU) * Set::NH;
    if (s % Set::SPU == 0) {
#pragma unroll
      for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[m][i] = 0.f;
    }
    uint32_t sh[NM][Set::NS];
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int i = 0; i < Set::NS; ++i) sh[m][i] = STREAM ? R.s[m][i] >> (16 * (n & 1)) : R.s[m][i];
#pragma unroll
    for (int hh = 0; hh < Set::NH; ++hh) {
      // B operands of the two groups of the step: [group][op] of every matrix
      uint32_t w[NM][2][8];          // 2 bits: 2 words per group, 4 bits: 4, 8 bits: 8
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const uint4* t = &R.t[(hh * NM + m) * LPM];
        if constexpr (BITS == 2) {
          uint32_t a0 = t[0].x, a1 = t[0].y, a2 = t[0].z, a3 = t[0].w;
          swap32(a0, a1);
          swap32(a2, a3);
          w[m][0][0] = a0; w[m][1][0] = a1; w[m][0][1] = a2; w[m][1][1] = a3;
        } else if constexpr (!STREAM) {              // 4 bits: a load per group; 8 bits: two
#pragma unroll
          for (int part = 0; part < LPM; ++part) {
            const uint4 v = t[part];
            const int gs = part * 2 / LPM, at = (part % (LPM / 2 > 0 ? LPM / 2 : 1)) * 4;
            w[m][gs][at] = v.x; w[m][gs][at + 1] = v.y; w[m][gs][at + 2] = v.z; w[m][gs][at + 3] = v.w;
          }
        } else if constexpr (BITS == 4) {
          uint32_t a[4] = {t[0].x, t[0].y, t[0].z, t[0].w}, b[4] = {t[1].x, t[1].y, t[1].z, t[1].w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            swap32(a[j], b[j]);
            w[m][0][j] = a[j]; w[m][1][j] = b[j];
          }
        } else {
#pragma unroll
          for (int pr = 0; pr < 2; ++pr) {
            uint32_t a[4] = {t[2 * pr].x, t[2 * pr].y, t[2 * pr].z, t[2 * pr].w};
            uint32_t b[4] = {t[2 * pr + 1].x, t[2 * pr + 1].y, t[2 * pr + 1].z, t[2 * pr + 1].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              swap32(a[j], b[j]);
              w[m][0][4 * pr + j] = a[j]; w[m][1][4 * pr + j] = b[j];
            }
          }
        }
      }
#pragma unroll
      for (int gs = 0; gs < 2; ++gs) {
        const int gl = 2 * hh + gs, g = 2 * h0 + gl;
        __builtin_amdgcn_sched_barrier(0);        // one group's operands ahead, no more: bounds the live registers
        const Operands next = read_a((g + 1) & (kBGroups - 1));
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          i32x4_t B[2];
#pragma unroll
          for (int op = 0; op < 2; ++op) {
            if constexpr (BITS == 2) B[op] = codes16_2(w[m][gs][op]);
            else if constexpr (BITS == 4) B[op] = codes16_4(w[m][gs][2 * op], w[m][gs][2 * op + 1]);
            else B[op] = codes16_8(w[m][gs][4 * op], w[m][gs][4 * op + 1], w[m][gs][4 * op + 2], w[m][gs][4 * op + 3]);
          }
          i32x4_t dl = mfma_i8(cur.a[0][0], B[0], cur.sx);
          i32x4_t dh = mfma_i8(cur.a[0][1], B[0], (i32x4_t){0, 0, 0, 0});
          dl = mfma_i8(cur.a[1][0], B[1], dl);
          dh = mfma_i8(cur.a[1][1], B[1], dh);
          const float sc = f16_bits_to_f32((uint32_t)__builtin_amdgcn_ds_bpermute(4 * (n + 16 * (gl & 3)), (int)sh[m][gl >> 2]) & 0xffffu);
          const float xf[4] = {cur.xs.x, cur.xs.y, cur.xs.z, cur.xs.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[m][i] = fmaf((float)(dl[i] + (dh[i] << 8)) * sc, xf[i], acc[m][i]);
        }
        cur = next;
        // the sums are finished here: otherwise the compiler sinks them behind the loads and keeps every product alive
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
          for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(acc[m][i]));
      }
    }
  };
  Set R0, R1;
  issue(R0, 0);
  issue(R1, 1);
  S.XS[sg][sm] = sxs * (sm < TOK ? 1.f : 65536.f);
  S.SX[sg][sm] = -code_offset<BITS>() * sxsum;
  stage_wait<16>();                            // the operands have landed; the sixteen 16-byte loads behind them stay in flight
  __syncthreads();
  cur = read_a(0);
  for (int s = 0; s < total; s += 2) {         // (SPU is even: a unit ends with a pair of sets)
    consume(R0, s);
    issue(R0, s + 2);
    consume(R1, s + 1);
    issue(R1, s + 3);
    if ((s + 2) % Set::SPU == 0) {
      // ---- the unit is complete: its 128 rows are scale group `unit` of h
      const int unit = u0 + s / Set::SPU, hb = unit & 1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (PARTS == 2) {                // low and high part of a pair: lanes kb and kb + 2
#pragma unroll
          for (int m = 0; m < NM; ++m) acc[m][i] += __shfl_xor(acc[m][i], 32);
        }
        const float a = acc[0][i];
        float v;
        if constexpr (SWIGLU) v = a / (1.0f + __expf(-a)) * acc[NM - 1][i];
        else v = fmaxf(a, 0.f);
        S.H[hb][4 * kb + i][wave * 16 + n] = v;
      }
      __syncthreads();
      // half of the wavefronts, in turn, write the digits: 16 threads per pair, eight columns each
      if ((wave >> 2) == hb) {
        const int t8 = threadIdx.x & 255, m = t8 >> 4, seg = t8 & 15;
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = S.H[hb][m][8 * seg + i];
        int part[PARTS][8], sum[PARTS];
        const float hs = group_ints<PARTS, STREAM ? 8 : 16>(v, part, sum);
        const size_t pair = item.pair[m < item.n ? m : 0];
        const size_t at = (pair * NG + unit) * 2;           // of HS and HSUM
        if (m < item.n && (seg & 7) == 0) G.HS[at + (seg >> 3)] = hs;
#pragma unroll
        for (int p = 0; p < PARTS; ++p) {
          const int (&xi)[8] = part[p];
          uint32_t half[2][4];             // 2 bits: byte pairs (column q, q + 4 of the half word) of both digits
#pragma unroll
          for (int qd = 0; qd < 4; ++qd) {
            half[0][qd] = lo_byte(xi[qd]) | lo_byte(xi[qd + 4]) << 8;
            half[1][qd] = hi_byte(xi[qd]) | hi_byte(xi[qd + 4]) << 8;
          }
          uint32_t other[2][4];
          if constexpr (BITS == 2) {
#pragma unroll
            for (int dg = 0; dg < 2; ++dg)
#pragma unroll
              for (int qd = 0; qd < 4; ++qd) other[dg][qd] = (uint32_t)dppi<kDppXor1>((int)half[dg][qd]);
          }
          if (m >= item.n) continue;
          if (STREAM ? (seg & 7) == 0 : seg == 0) G.HSUM[at + (STREAM ? seg >> 3 : p)] = sum[p];
          uint8_t* dst = G.HQ + (pair * (size_t)(2 * G.L.d_ff) + (size_t)unit * 256) * PARTS + p * 128;
#pragma unroll
          for (int dg = 0; dg < 2; ++dg) {
            uint32_t by[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) by[i] = dg ? hi_byte(xi[i]) : lo_byte(xi[i]);
            const uint32_t lo4 = by[0] | by[1] << 8 | by[2] << 16 | by[3] << 24, hi4 = by[4] | by[5] << 8 | by[6] << 16 | by[7] << 24;
            const uint32_t even = by[0] | by[2] << 8 | by[4] << 16 | by[6] << 24, odds = by[1] | by[3] << 8 | by[5] << 16 | by[7] << 24;
            const bool cols = STREAM || G.out_columns != 0;
            // a piece (op, digit dg, kb) of the group lies at op * 128 * PARTS + dg * 64 + kb * 16
            if constexpr (BITS == 4) {           // the thread's columns are word `seg` of the group: operand, kb, half of the piece
              const int op = cols ? seg >> 3 : (seg >> 1) & 1, okb = cols ? seg & 3 : seg >> 2, hf = cols ? (seg >> 2) & 1 : seg & 1;
              *(uint2*)(dst + op * (128 * PARTS) + dg * 64 + okb * 16 + hf * 8) = make_uint2(even, odds);
            } else if constexpr (BITS == 2) {    // half of word seg >> 1: the even thread writes dwords 0, 1, the odd one 2, 3
              const int wd = seg >> 1, odd = seg & 1;
              const int op = cols ? wd >> 2 : (wd >> 1) & 1, okb = cols ? wd & 3 : (wd >> 2) | (wd & 1) << 1;
              const uint32_t d0 = odd ? (other[dg][2] | half[dg][2] << 16) : (half[dg][0] | other[dg][0] << 16);
              const uint32_t d1 = odd ? (other[dg][3] | half[dg][3] << 16) : (half[dg][1] | other[dg][1] << 16);
              *(uint2*)(dst + op * (128 * PARTS) + dg * 64 + okb * 16 + odd * 8) = make_uint2(d0, d1);
            } else if (cols) {                   // words 2 seg and 2 seg + 1
#pragma unroll
              for (int i = 0; i < 2; ++i) {
                const int wd = 2 * seg + i;
                *(uint32_t*)(dst + (wd >> 4) * (128 * PARTS) + dg * 64 + (wd & 3) * 16 + ((wd >> 2) & 3) * 4) = i ? hi4 : lo4;
              }
            } else {                             // half of a piece of sixteen columns
              *(uint2*)(dst + (seg >> 3) * (128 * PARTS) + dg * 64 + ((seg >> 1) & 3) * 16 + (seg & 1) * 8) = make_uint2(lo4, hi4);
            }
          }
        }
      }
    }
  }
}

// Grid: one workgroup per compute unit (the operands take most of its LDS). The units of all items form one list, cut
// into ranges of equal weight (a unit costs its bytes: the bitwidth, plus the scales), one per workgroup; a workgroup's
// range lies in one or two items.
template <bool SWIGLU, bool STREAM>
__global__ __launch_bounds__(512) void k_batch_in(BatchArgs G) {
  extern __shared__ __attribute__((aligned(16))) char bsmem[];
  BatchInLds& S = *(BatchInLds*)bsmem;
  constexpr int NM = SWIGLU ? 2 : 1;
  const int n_items = batch_items<batch_tok(STREAM)>(G, S.lists);
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < n_items * 2; i += 512) ((uint4*)G.items)[i] = ((const uint4*)S.lists.items)[i];
    if (threadIdx.x == 0) *G.n_items = n_items;
  }
  const int NU = G.L.d_ff / kBGroup;
  // 32 bits and a division only for the items the range meets: 64-bit ones for every item were 1-2 us ahead of the first load.
  // (256 items of weight 65: no overflow below d_ff 2^24)
  uint32_t total = 0;
  for (int i = 0; i < n_items; ++i) total += 8u * (uint32_t)S.lists.items[i].bits + 1u;
  total *= (uint32_t)NU;
  const uint32_t whole = total / gridDim.x, rest = total % gridDim.x;        // total * blockIdx.x / gridDim.x
  const uint32_t lo = __builtin_amdgcn_readfirstlane(whole * blockIdx.x + rest * blockIdx.x / gridDim.x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane(whole * (blockIdx.x + 1) + rest * (blockIdx.x + 1) / gridDim.x);
  uint32_t base = 0, end = 0;
  for (int i = 0; i < n_items && base < hi; ++i, base = end) {
    const int bits = __builtin_amdgcn_readfirstlane(S.lists.items[i].bits);
    const uint32_t c = 8u * (uint32_t)bits + 1u;
    end = base + c * (uint32_t)NU;
    if (end <= lo) continue;
    // units whose start weight lies in [lo, hi)
    const uint32_t a = lo > base ? (lo - base + c - 1) / c : 0, b = (hi - base + c - 1) / c;
    const int u0 = __builtin_amdgcn_readfirstlane((int)min(a, (uint32_t)NU)), u1 = __builtin_amdgcn_readfirstlane((int)min(b, (uint32_t)NU));
    if (u0 < u1) {
      const BatchItem& item = S.lists.items[i];
      if (bits == 2) batch_in_units<2, NM, SWIGLU, STREAM>(G, S, item, u0, u1);
      else if (bits == 4) batch_in_units<4, NM, SWIGLU, STREAM>(G, S, item, u0, u1);
      else batch_in_units<8, NM, SWIGLU, STREAM>(G, S, item, u0, u1);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// W_out in columns: word w of row r is the 32-bit word w * d_model + r. Lane (n, kb) loads word column 4 j + kb of the
// rows 4 n .. 4 n + 3 of its wavefront's 64 rows (four runs of 256 consecutive bytes per load); operand i of a load
// belongs to the rows 4 n + i.
template <int BITS>
struct BatchOutSet {
  static constexpr int LPG = BITS;                 // loads per scale group (128 columns: 4 * BITS word columns)
  static constexpr int GS = 8 / LPG;               // groups per set of eight loads
  uint4 t[8];
  uint2 s[GS];
};

struct BatchOutLds {
  uint4 A[kBOutGroups * 4][64];
  float XS[kBOutGroups][2][kBRows];        // [half of the group's columns] (other than stream layers: the first)
  int32_t SX[kBOutGroups][2][kBRows];
};

// A workgroup takes `blocks` blocks of 256 rows (out_blocks) with the same activations, its requests running on from one to the
// next. What lies past its end asks for a cached line: the next chunk's words, requested and dropped, were half as many bytes
// again at 4 bits. NT: words in columns are read with the non-temporal hint (stream_out). Three workgroups are resident per
// compute unit; with two, the rows form lost what the running requests gain (2 bits, d_ff 14336, 23 tokens 145 us, now 138).
// Canonical rows: the wavefront's 64 rows are four blocks of 16; lane (n, kb) loads 16-byte piece 4 j + kb of row 16 i + n
// (64 consecutive bytes of 16 rows: one scale group at 4 bits, two at 2, half of one at 8), operand i belongs to block i.
template <int BITS, bool COLS, bool STREAM, bool NT>
__device__ __forceinline__ void batch_out(const BatchArgs& G, BatchOutLds& S, const BatchItem& item, int blocks) {
  using Set = BatchOutSet<BITS>;
  constexpr int TOK = batch_tok(STREAM), PARTS = batch_parts(STREAM);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, kb = lane >> 4;
  const int NG = G.L.d_ff / kBGroup;
  const int g0 = blockIdx.y * kBOutGroups, ng = min(kBOutGroups, NG - g0);
  const int r0 = blockIdx.x * blocks * kBOutRows + wave * 64 + (COLS ? 4 * n : n);   // of the first block: operand i is row r0 + i, or r0 + 16 i
  const DevExpert* ex = G.table + item.e;
  const uint8_t* q = uniform_ptr(ex->q_out);
  const uint8_t* sc = (const uint8_t*)uniform_ptr(ex->s_out);
  // 256 threads = 8 groups x 2 halves x 16 rows: the operands' factors, stored behind the first weights' requests
  const int fg = threadIdx.x >> 5, fhalf = (threadIdx.x >> 4) & 1, fm = threadIdx.x & 15;
  const size_t fat = ((size_t)item.pair[fm % TOK < item.n ? fm % TOK : 0] * NG + min(g0 + fg, NG - 1)) * 2;
  const float fxs = G.HS[fat + fhalf];
  const int32_t fsum = G.HSUM[fat + (STREAM ? fhalf : fm / TOK)];
  {
    const int pm = item.pair[n % TOK < item.n ? n % TOK : 0];
    const uint8_t* src = G.HQ + ((size_t)pm * (size_t)(2 * G.L.d_ff) + (size_t)g0 * 256) * PARTS + (n / TOK) * 128 + kb * 16;
    const uint32_t a0 = (uint32_t)(uintptr_t)(MOEQ_LDS char*)&S.A[0][0];
    for (int i = 0; i < kBOutGroups; ++i) {
      const int o = wave + 4 * i;                  // operands of the groups that exist
      if (o < ng * 4) dma16(src + (o >> 1) * (PARTS * 128) + (o & 1) * 64, a0 + (uint32_t)o * 1024u);
    }
  }
  // sets of a block, an even number (the two register sets take turns); one past the chunk's groups is loaded from its last group
  const int n_sets = ((ng + Set::GS - 1) / Set::GS + 1) & ~1;
  const uint32_t col = (uint32_t)kBD * 4u;         // bytes of a word column
  const uint32_t lane_off = (uint32_t)kb * col + (uint32_t)r0 * 4u;
  const uint32_t row_bytes = (uint32_t)G.L.d_ff * BITS / 8u;
  // canonical rows: lane (n, kb) holds the chunk's scales of row 16 kb + n, two groups to a register
  uint32_t srow[kBOutGroups / 2] = {}, snext[kBOutGroups / 2] = {};
  int is = 0, ib = 0;                              // set and block the next request is for
  auto issue = [&](Set& R) __attribute__((always_inline)) {
    const bool live = ib < blocks;                 // past the end: cached bytes, so that every path issues the same loads
    const uint32_t rows = (uint32_t)ib * kBOutRows;
    const uint8_t* dead = G.HQ + lane * 16;
    if constexpr (COLS) {
#pragma unroll
      for (int gi = 0; gi < Set::GS; ++gi) {
        const int g = min(g0 + is * Set::GS + gi, g0 + ng - 1);
        const uint8_t* qg = q + (size_t)g * (4 * BITS) * col + (size_t)rows * 4u;
#pragma unroll
        for (int j = 0; j < Set::LPG; ++j) {
          const uint8_t* p = live ? qg + (size_t)(4 * j) * col + lane_off : dead;
          R.t[gi * Set::LPG + j] = NT ? load_stream16(p) : gload_u32x4(p);
        }
        R.s[gi] = gload_u32x2(live ? sc + (size_t)g * (kBD * 2) + (rows + (uint32_t)r0) * 2u : dead);
      }
    } else {
      // 64-byte steps of the rows: a set is two of them for the four blocks of 16
      const uint32_t step0 = (uint32_t)g0 * BITS / 4u + (uint32_t)is * 2u, last = (uint32_t)(g0 + ng) * BITS - 1u;
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          R.t[st * 4 + i] = gload_u32x4(live ? q + ((size_t)(rows + (uint32_t)(r0 + 16 * i)) * row_bytes + min((step0 + st) * 4u + kb, last) * 16u) : dead);
      if (is == 0) {
        const uint32_t row = live ? rows + (uint32_t)(blockIdx.x * blocks * kBOutRows + wave * 64 + 16 * kb + n) : 0u;
#pragma unroll
        for (int g = 0; g < kBOutGroups; g += 2) {
          const uint32_t a = gload_u16(sc + ((size_t)row * NG + min(g0 + g, NG - 1)) * 2), b = gload_u16(sc + ((size_t)row * NG + min(g0 + g + 1, NG - 1)) * 2);
          snext[g / 2] = a | b << 16;
        }
      }
    }
    if (++is == n_sets) { is = 0; ++ib; }
  };
  float acc[4][4];
  auto consume = [&](const Set& R, int s) __attribute__((always_inline)) {
    if (s == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
      if constexpr (!COLS) {
#pragma unroll
        for (int g = 0; g < kBOutGroups / 2; ++g) srow[g] = snext[g];
      }
    }
#pragma unroll
    for (int gi = 0; gi < Set::GS; ++gi) {
      const int g = s * Set::GS + gi;
      if (g < ng) {
        i32x4_t A[2][2];
#pragma unroll
        for (int op = 0; op < 2; ++op)
#pragma unroll
          for (int dg = 0; dg < 2; ++dg) A[op][dg] = __builtin_bit_cast(i32x4_t, S.A[(g * 2 + op) * 2 + dg][lane]);
        const i32x4_t sx = *(const i32x4_t*)&S.SX[g][0][4 * kb];
        const float4 xs = *(const float4*)&S.XS[g][0][4 * kb];
        const float xf[4] = {xs.x, xs.y, xs.z, xs.w};
        // (stream layers: the second operand's columns have an exponent of their own, as in k_moe_stream)
        const i32x4_t sx1 = STREAM ? *(const i32x4_t*)&S.SX[g][1][4 * kb] : (i32x4_t){0, 0, 0, 0};
        const float4 xs1 = STREAM ? *(const float4*)&S.XS[g][1][4 * kb] : xs;
        const float xf1[4] = {xs1.x, xs1.y, xs1.z, xs1.w};
        uint32_t s4[4];
        if constexpr (COLS) {
          s4[0] = R.s[gi].x & 0xffffu; s4[1] = R.s[gi].x >> 16; s4[2] = R.s[gi].y & 0xffffu; s4[3] = R.s[gi].y >> 16;
        } else {
          // (the group's register: s and gi select it; a set's groups have fixed places)
          const int gp = g >> 1;
          const uint32_t v = gp == 0 ? srow[0] : gp == 1 ? srow[1] : gp == 2 ? srow[2] : srow[3];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            s4[i] = ((uint32_t)__builtin_amdgcn_ds_bpermute(4 * (n + 16 * i), (int)v) >> (16 * (g & 1))) & 0xffffu;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          i32x4_t B[2];
          if constexpr (COLS) {
            const uint4* t = &R.t[gi * Set::LPG];
            auto word = [&](int j) { return i == 0 ? t[j].x : i == 1 ? t[j].y : i == 2 ? t[j].z : t[j].w; };
#pragma unroll
            for (int op = 0; op < 2; ++op) {
              if constexpr (BITS == 2) B[op] = codes16_2(word(op));
              else if constexpr (BITS == 4) B[op] = codes16_4(word(2 * op), word(2 * op + 1));
              else B[op] = codes16_8(word(4 * op), word(4 * op + 1), word(4 * op + 2), word(4 * op + 3));
            }
          } else if constexpr (BITS == 2) {
            const uint4 t = R.t[(gi >> 1) * 4 + i];
            uint32_t a0 = t.x, a1 = t.y, a2 = t.z, a3 = t.w;
            swap32(a0, a1);
            swap32(a2, a3);
            B[0] = codes16_2((gi & 1) ? a1 : a0);
            B[1] = codes16_2((gi & 1) ? a3 : a2);
          } else if constexpr (BITS == 4) {
            const uint4 t = R.t[gi * 4 + i];
            B[0] = codes16_4(t.x, t.y);
            B[1] = codes16_4(t.z, t.w);
          } else {
            const uint4 t0 = R.t[i], t1 = R.t[4 + i];
            B[0] = codes16_8(t0.x, t0.y, t0.z, t0.w);
            B[1] = codes16_8(t1.x, t1.y, t1.z, t1.w);
          }
          i32x4_t dl = mfma_i8(A[0][0], B[0], sx);
          i32x4_t dh = mfma_i8(A[0][1], B[0], (i32x4_t){0, 0, 0, 0});
          const i32x4_t dl1 = mfma_i8(A[1][0], B[1], STREAM ? sx1 : dl);
          const i32x4_t dh1 = mfma_i8(A[1][1], B[1], STREAM ? (i32x4_t){0, 0, 0, 0} : dh);
          const float scf = f16_bits_to_f32(s4[i]);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if constexpr (STREAM) acc[i][j] = fmaf((float)(dl[j] + (dh[j] << 8)) * scf, xf[j], acc[i][j]);
            acc[i][j] = fmaf((float)(dl1[j] + (dh1[j] << 8)) * scf, xf1[j], acc[i][j]);
          }
        }
      }
    }
  };
  Set R0, R1;
  issue(R0);
  issue(R1);
  S.XS[fg][fhalf][fm] = fxs * (fm < TOK ? 1.f : 65536.f);
  S.SX[fg][fhalf][fm] = -code_offset<BITS>() * fsum;
  stage_wait<16>();
  __syncthreads();
  for (int blk = 0; blk < blocks; ++blk) {
    for (int s = 0; s < n_sets; s += 2) {
      consume(R0, s);
      issue(R0);
      consume(R1, s + 1);
      issue(R1);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (PARTS == 2) {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][j] += __shfl_xor(acc[i][j], 32);
      }
      const int m = 4 * kb + j;                    // (the lanes of the high parts' rows, 8 .. 15, write nothing: item.n <= TOK)
      if (m < item.n) {
        float* o = G.part + ((size_t)blockIdx.y * (size_t)(G.T * G.k) + item.pair[m]) * kBD + blk * kBOutRows + r0;
        if constexpr (COLS) {
          *(float4*)o = make_float4(acc[0][j], acc[1][j], acc[2][j], acc[3][j]);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) o[16 * i] = acc[i][j];
        }
      }
    }
  }
}

// Grid (d_model / (blocks * 256), chunks of d_ff, upper bound of the items).
template <bool COLS, bool STREAM, bool NT>
__global__ __launch_bounds__(256, 3) void k_batch_out(BatchArgs G, int blocks) {
  __shared__ BatchOutLds S;
  __shared__ BatchItem item;
  if ((int)blockIdx.z >= *G.n_items) return;
  if (threadIdx.x < 2) ((uint4*)&item)[threadIdx.x] = ((const uint4*)(G.items + blockIdx.z))[threadIdx.x];
  __syncthreads();
  const int bits = __builtin_amdgcn_readfirstlane(item.bits);
  if (bits == 2) batch_out<2, COLS, STREAM, NT>(G, S, item, blocks);
  else if (bits == 4) batch_out<4, COLS, STREAM, NT>(G, S, item, blocks);
  else batch_out<8, COLS, STREAM, NT>(G, S, item, blocks);
}

// y[t][r] (+)= sum_j gate[t][j] * sum_c part[c][t k + j][r], chunks and choices in order. gate null: 1. Wavefront j sums the
// chunks of choice j, sixteen requested together; the first one adds the choices.
__global__ __launch_bounds__(512) void k_batch_combine(const float* __restrict__ part, const float* __restrict__ gate,
                                                       int n_chunks, int T, int k, int accumulate, float* __restrict__ y) {
  __shared__ float4 sums[8][64];
  const int t = blockIdx.y, lane = threadIdx.x & 63, j = threadIdx.x >> 6, r = (blockIdx.x * 64 + lane) * 4;
  const float* p = part + (size_t)(t * k + j) * kBD + r;
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int c0 = 0; c0 < n_chunks; c0 += 16) {
    float4 w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = *(const float4*)(p + (size_t)min(c0 + i, n_chunks - 1) * T * k * kBD);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const bool in = c0 + i < n_chunks;
      a.x += in ? w[i].x : 0.f; a.y += in ? w[i].y : 0.f; a.z += in ? w[i].z : 0.f; a.w += in ? w[i].w : 0.f;
    }
  }
  sums[j][lane] = a;
  __syncthreads();
  if (j) return;
  float* o = y + (size_t)t * kBD + r;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  if (accumulate)
    for (int i = 0; i < 4; ++i) v[i] = o[i];
  for (int q = 0; q < k; ++q) {
    const float g = gate ? gate[(size_t)t * k + q] : 1.0f;
    const float4 w = sums[q][lane];
    v[0] = fmaf(g, w.x, v[0]); v[1] = fmaf(g, w.y, v[1]); v[2] = fmaf(g, w.z, v[2]); v[3] = fmaf(g, w.w, v[3]);
  }
  for (int i = 0; i < 4; ++i) o[i] = v[i];
}

int batch_cus() {
  static const int cus = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    return n;
  }();
  return cus;
}

// Blocks of 256 rows that a k_batch_out workgroup takes one after the other, for so many (chunk, item) pairs of a call: two where
// that leaves about a workgroup per compute unit (in rows one and a half) and the arithmetic is not what they wait for. One expert of 4 or 8 bits, whose
// later items find its words in the caches, us one / two blocks: 8 bits in columns, d_ff 14336, 16 tokens 74 / 69, 32 tokens 130 /
// 111, 256 and more 988 / 877; 4 bits in rows 83 / 86 (24 tokens), 256 / 244 (128); a narrow one (d_ff 4096, 8 items) 45 / 50. Layer
// calls (8 experts, words in columns): 4 bits, d_ff 4096, 8 tokens 57 / 54, d_ff 8192 91 / 89, 2 and 4 bits, d_ff 14336, 23 tokens
// 177 / 170, 2, 4 and 8 bits in stream, d_ff 8192 152 / 145. 2 bits (bound by arithmetic: d_ff 14336 in rows 127 / 132), 8 bits alone
// (d_ff 4096, 23 tokens 133 / 137) and words in rows (4 bits, d_ff 14336, 8 tokens 171 / 176) take one.
int out_blocks(int pairs, int bits_mask, bool one_expert, bool columns) {
  const bool pays = one_expert ? bits_mask != 2 || pairs >= 200 : columns && bits_mask != 2 && bits_mask != 8;
  return pays && pairs * (kBD / kBOutRows / 2) * 8 >= (columns ? 7 : 12) * batch_cus() ? 2 : 1;
}
// Whether the words of W_out in columns are read with the non-temporal hint: where they are asked for once, or few experts of a
// layer call have a second item that would find them in a cache, and the loads are what the kernel waits for (not at 2 bits). us,
// without / with it, on several layers in turn: 4 bits, d_ff 8192, 16 tokens in stream 105 / 103, 8 bits 186 / 183, 4 bits in columns,
// d_ff 14336, 16 tokens 171 / 165; 2 bits in stream, d_ff 14336, 23 tokens 120 / 124; 4 bits in columns, d_ff 4096, 31 tokens 98 / 101.
// One expert in stream, 12 tokens, 4 bits, d_ff 14336 48.6 / 46.0, 8 bits, d_ff 9728 74 / 67; 300 tokens in columns 518 / 600.
bool stream_out(int P, int tok, int experts, bool one_expert, int bits_mask) {
  return bits_mask != 2 && (one_expert ? P <= tok : 2 * P <= tok * experts);
}

}  // namespace

// Byte offsets of the path's pieces in the workspace; k: choices per token (1 for a single expert's call).
BatchWs batch_ws(const LayerDims& L, int64_t T, int32_t k, int32_t bits_mask, bool in_stream) {
  BatchWs w{};
  const size_t parts = batch_parts(in_stream), P = (size_t)T * (size_t)k, NG = (size_t)L.d_ff / kBGroup;
  size_t off = 0;
  w.items = off;  off += up256(P * sizeof(BatchItem));
  w.n_items = off; off += 256;
  w.xq = off;     off += up256((size_t)__builtin_popcount((unsigned)bits_mask & 14u) * (size_t)T * parts * 2 * kBD);
  w.xs = off;     off += up256((size_t)T * kBGroups * 4);
  w.xsum = off;   off += up256((size_t)T * kBGroups * parts * 4);
  w.hq = off;     off += up256(P * parts * 2 * (size_t)L.d_ff);
  w.hs = off;     off += up256(P * NG * 8);
  w.hsum = off;   off += up256(P * NG * 8);
  w.part = off;   off += up256((NG + kBOutGroups - 1) / kBOutGroups * P * kBD * 4);
  w.total = off;
  return w;
}

bool batch_supported(const LayerDims& L) { return L.d_model == kBD && L.group == kBGroup && L.group_out == kBGroup && L.top_k <= 8; }
int batch_inline_router_max() { return kBInlineMaxE; }

hipError_t init_attrs_decode_batch() {
  (void)batch_cus();
  for (const void* kf : {(const void*)k_batch_in<true, true>, (const void*)k_batch_in<false, true>, (const void*)k_batch_in<true, false>,
                         (const void*)k_batch_in<false, false>})
    if (hipError_t e = hipFuncSetAttribute(kf, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(BatchInLds)); e != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_moe_batch(const LayerDims& L, const DevExpert* table, const float* router_w, const float* router_bias,
                            bool route_inline, int32_t fixed_expert, int32_t bits_mask, const void* x, int32_t T, int32_t* idx,
                            float* gate, const float* gate_out, int32_t accumulate, bool in_stream, bool out_columns, char* ws,
                            float* y, hipStream_t st, const Prof& prof) {
  const int k = fixed_expert >= 0 ? 1 : L.top_k;
  if (!batch_supported(L) || L.d_ff % kBGroup || T < 1 || (int64_t)T * k > kBatchMaxPairs || !(bits_mask & 14) || (in_stream && !out_columns))
    return hipErrorInvalidValue;
  if (route_inline && (fixed_expert >= 0 || L.n_experts > kBInlineMaxE)) return hipErrorInvalidValue;
  if (fixed_expert < 0 && (!idx || !gate)) return hipErrorInvalidValue;
  const BatchWs w = batch_ws(L, T, k, bits_mask, in_stream);
  BatchArgs G{L, table, router_w, router_bias, x, T, k, fixed_expert, bits_mask & 14, route_inline ? 1 : 0, out_columns ? 1 : 0, idx, gate,
              (uint8_t*)(ws + w.xq), (float*)(ws + w.xs), (int32_t*)(ws + w.xsum), (uint8_t*)(ws + w.hq),
              (float*)(ws + w.hs), (int32_t*)(ws + w.hsum), (BatchItem*)(ws + w.items), (int32_t*)(ws + w.n_items),
              (float*)(ws + w.part)};
  const int P = T * k;
  const int tok = batch_tok(in_stream), most = L.n_experts + P / tok, max_items = fixed_expert >= 0 ? (P + tok - 1) / tok : P < most ? P : most;
  const int chunks = (L.d_ff / kBGroup + kBOutGroups - 1) / kBOutGroups;
  prof_start(prof, MOEQ_KERNEL_FUSED, st);
  hipLaunchKernelGGL(in_stream ? k_batch_prep<true> : k_batch_prep<false>, dim3(T), dim3(512), 0, st, G);
  const bool sw = L.act == MOEQ_ACT_SWIGLU;
  auto kin = in_stream ? (sw ? k_batch_in<true, true> : k_batch_in<false, true>) : (sw ? k_batch_in<true, false> : k_batch_in<false, false>);
  prof_start(prof, MOEQ_KERNEL_FFN_IN, st);
  hipLaunchKernelGGL(kin, dim3(batch_cus()), dim3(512), sizeof(BatchInLds), st, G);
  prof_stop(prof, MOEQ_KERNEL_FFN_IN, st);
  prof_start(prof, MOEQ_KERNEL_FFN_OUT, st);
  const bool nt = stream_out(P, tok, L.n_experts, fixed_expert >= 0, bits_mask & 14);
  auto kout = in_stream ? (nt ? k_batch_out<true, true, true> : k_batch_out<true, true, false>)
                        : out_columns ? (nt ? k_batch_out<true, false, true> : k_batch_out<true, false, false>) : k_batch_out<false, false, false>;
  const int blocks = out_blocks(chunks * max_items, bits_mask & 14, fixed_expert >= 0, out_columns);
  hipLaunchKernelGGL(kout, dim3(kBD / kBOutRows / blocks, chunks, max_items), dim3(256), 0, st, G, blocks);
  prof_stop(prof, MOEQ_KERNEL_FUSED, st);
  hipLaunchKernelGGL(k_batch_combine, dim3(kBD / 256, T), dim3(64 * k), 0, st, G.part, gate_out, chunks, T, k, accumulate, y);
  prof_stop(prof, MOEQ_KERNEL_FFN_OUT, st);
  return hipGetLastError();
}

}  // namespace moeq
