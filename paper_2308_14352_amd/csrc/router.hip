// Router GEMV (Section 1; Section 2.1: a small router scores the experts for every token).
// logits[t][e] = router_w[e] . x[t] (+ bias[e]) in fp32.
// k_router_logits: one workgroup per (expert, group of up to 8 tokens): the expert's row is read once with 128-bit loads and
// dotted with each token of the group; partial sums are folded with DPP inside each wavefront, then across the wavefronts
// through LDS. The softmax and the top-k selection run where the result is needed (k_topk, the FFN kernels).
// k_route: logits and top-k of one to four tokens per workgroup in one kernel, with the same bits (launch_route chooses).
#include "decode_core.h"

namespace moeq {
namespace {

constexpr int kThreads = 256;
constexpr int kTokensPerWg = 8;

// TG tokens of a workgroup (of a group that has fewer, the last one stands in for the rest): their activations are requested
// together. With the loads behind a condition on the number of tokens they went one after the other, 4 us of a kernel's 4.7 at
// 8 tokens (128 experts of 1024 columns; now 1.6).
template <bool BF16, int TG>
__global__ __launch_bounds__(kThreads) void k_router_logits(LayerDims L, const float* __restrict__ Wr,
                                                            const float* __restrict__ bias,
                                                            const void* __restrict__ x, int32_t T,
                                                            float* __restrict__ logits) {
  __shared__ float part[kThreads / 64][TG];
  const int d = L.d_model, E = L.n_experts;
  const int e = blockIdx.x;
  const int t0 = blockIdx.y * TG;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* wr = Wr + (size_t)e * d;
  float acc[TG];
#pragma unroll
  for (int tt = 0; tt < TG; ++tt) acc[tt] = 0.f;
  for (int i = tid * 4; i < d; i += kThreads * 4) {
    const float4 w = *(const float4*)(wr + i);
    float4 v[TG];
#pragma unroll
    for (int tt = 0; tt < TG; ++tt) {
      const size_t at = (size_t)min(t0 + tt, T - 1) * d + i;
      if (BF16) {
        const ushort4 b = *(const ushort4*)((const uint16_t*)x + at);
        v[tt] = make_float4(bf16_bits_to_f32(b.x), bf16_bits_to_f32(b.y), bf16_bits_to_f32(b.z), bf16_bits_to_f32(b.w));
      } else {
        v[tt] = *(const float4*)((const float*)x + at);
      }
    }
#pragma unroll
    for (int tt = 0; tt < TG; ++tt) {
      acc[tt] = fmaf(w.x, v[tt].x, acc[tt]); acc[tt] = fmaf(w.y, v[tt].y, acc[tt]);
      acc[tt] = fmaf(w.z, v[tt].z, acc[tt]); acc[tt] = fmaf(w.w, v[tt].w, acc[tt]);
    }
  }
#pragma unroll
  for (int tt = 0; tt < TG; ++tt) {
    const float v = wave_sum(acc[tt]);
    if (lane == 0) part[wave][tt] = v;
  }
  __syncthreads();
  if (tid < TG && t0 + tid < T) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) v += part[w][tid];
    logits[(size_t)(t0 + tid) * E + e] = v + (bias ? bias[e] : 0.f);
  }
}

// Router and top-k of TG tokens in one workgroup: the calls of many tokens, where the logits in memory and a second kernel
// cost as much as the sums. The logits are those of k_router_logits, bit for bit, so that a token's routing does not depend on
// which of the two serves its call: the columns are four classes (256 columns in every 1024), a class is one chain of sums per
// lane, and lanes, quads, rows and classes are added in the same order. A wavefront's unit is EB experts x a class, or with many
// experts (WHOLE) EB experts x all four: the rows of all its experts are requested together, four steps of 256 columns at a time
// (WHOLE on four tokens: two, or the sums spill), and meet the TG tokens in registers. The folds of a class are as many
// instructions as its products at d_model 768, so they take all tokens' sums at once and leave out the classes without columns.
// us, with k_router_logits + k_topk before: 8 experts of 4096 columns 117 tokens 8.7 -> 4.3, 2048 tokens 48 -> 12.5; 64 of 768, 500
// tokens 11 -> 6; 128 of 768, 2100 tokens 66 -> 29.4.
constexpr int kRouteWaves = 8, kRouteClasses = 4;

template <bool BF16, int TG, int EB, bool WHOLE>
__global__ __launch_bounds__(kRouteWaves * 64) void k_route(LayerDims L, const float* __restrict__ Wr, const float* __restrict__ bias,
                                                            const void* __restrict__ x, int32_t T, int32_t* __restrict__ idx,
                                                            float* __restrict__ gate, float* __restrict__ probs) {
  extern __shared__ float rsm[];                 // [class][TG][experts, whole blocks of EB]
  constexpr int STEPS = WHOLE && TG == 4 ? 2 : 4, SETS = WHOLE ? kRouteClasses : 1;
  const int d = L.d_model, E = L.n_experts, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = (E + EB - 1) / EB, t0 = blockIdx.x * TG, stride = nb * EB;
  for (int u = wave; u < (WHOLE ? nb : nb * kRouteClasses); u += kRouteWaves) {
    const int eb = WHOLE ? u : u / kRouteClasses, cls = WHOLE ? 0 : u % kRouteClasses;
    float acc[SETS][TG * EB];
#pragma unroll
    for (int s = 0; s < SETS; ++s)
#pragma unroll
      for (int i = 0; i < TG * EB; ++i) acc[s][i] = 0.f;
    // steps of 256 columns: of all classes one after the other (step j of four is class j), of one class 1024 apart
    constexpr int STEP = WHOLE ? 256 : 1024;
    for (int c0 = 256 * cls; c0 < d; c0 += WHOLE ? 1024 : STEP * STEPS) {
#pragma unroll
      for (int j0 = 0; j0 < (WHOLE ? kRouteClasses : STEPS); j0 += STEPS) {
        float4 w[STEPS][EB], v[STEPS][TG];
        if (j0) __builtin_amdgcn_sched_barrier(0);           // (their registers are those of the steps before)
#pragma unroll
        for (int j = 0; j < STEPS; ++j)
          if (c0 + STEP * (j0 + j) < d) {
            const int c = min(c0 + STEP * (j0 + j) + lane * 4, d - 4);
#pragma unroll
            for (int t = 0; t < TG; ++t) {
              const size_t at = (size_t)min(t0 + t, T - 1) * d + c;
              if (BF16) {
                const uint2 b = *(const uint2*)((const uint16_t*)x + at);
                v[j][t] = make_float4(bf16_bits_to_f32(b.x & 0xffffu), bf16_bits_to_f32(b.x >> 16), bf16_bits_to_f32(b.y & 0xffffu), bf16_bits_to_f32(b.y >> 16));
              } else {
                v[j][t] = *(const float4*)((const float*)x + at);
              }
            }
#pragma unroll
            for (int i = 0; i < EB; ++i) w[j][i] = *(const float4*)(Wr + (size_t)min(eb * EB + i, E - 1) * d + c);     // rows past E repeat the last one
          }
#pragma unroll
        for (int j = 0; j < STEPS; ++j)
          if (c0 + STEP * (j0 + j) + lane * 4 < d) {
            const int s = WHOLE ? j0 + j : 0;
#pragma unroll
            for (int i = 0; i < EB; ++i)
#pragma unroll
              for (int t = 0; t < TG; ++t) {
                float& a = acc[s][t * EB + i];
                a = fmaf(w[j][i].x, v[j][t].x, a); a = fmaf(w[j][i].y, v[j][t].y, a);
                a = fmaf(w[j][i].z, v[j][t].z, a); a = fmaf(w[j][i].w, v[j][t].w, a);
              }
          }
      }
    }
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
      const float sum = 256 * (cls + s) < d ? route_fold(acc[s], lane) : 0.f;
      if (lane < TG * EB) rsm[((cls + s) * TG + lane / EB) * stride + eb * EB + lane % EB] = sum;
    }
  }
  __syncthreads();
  if (wave < TG && t0 + wave < T) {
    float* lg = rsm + wave * stride;
    for (int e = lane; e < E; e += 64) {
      float s = 0.f;
#pragma unroll
      for (int r = 0; r < kRouteClasses; ++r) s += lg[r * TG * stride + e];
      lg[e] = s + (bias ? bias[e] : 0.f);
    }
    const size_t t = (size_t)(t0 + wave);
    topk_from_logits(lg, E, L.top_k, L.renorm, lane, idx + t * L.top_k, gate + t * L.top_k, probs ? probs + t * E : nullptr);
  }
}

// Experts of a unit, and whether it takes all classes: units for the eight wavefronts.
template <bool BF16, int TG>
auto pick_route(const LayerDims& L) {
  return L.n_experts <= 8 ? k_route<BF16, TG, 4, false> : L.n_experts <= 32 ? k_route<BF16, TG, 8, false> : k_route<BF16, TG, 8, true>;
}

}  // namespace

// One kernel or two (logits through memory). A workgroup of k_route reads every expert's row, which in calls of up to a
// workgroup's tokens per compute unit takes as long as one of them; the two kernels spread the rows over the chip and read them
// once per eight tokens, but are two launches. us, one / two kernels: 8 experts of 4096 columns 4.2 / 8.7 (117 tokens), 64 of 768
// 5.0 / 6.5; 128 of 1536 9.8 / 7.0 (8 tokens), 128 of 4096 21.5 / 9.4 (8 tokens), 22 / 15.4 (117) and 26 / 37 (300); 1024 of 4096
// 176 / 13.5 (8 tokens), 168 / 208 (300); 33 of 4096 10.8 / 8.4 (8 tokens), 11.2 / 12.0 (117). The line is that of the two times as
// fitted to 700 calls; where it errs they are within 1.5 us.
static bool route_in_one(const LayerDims& L, int32_t T) {
  const double rows = (double)L.d_model * L.n_experts, wide = L.d_model / 2048.0;
  return T > 256 || 3.2 + rows / 27000.0 < 6.3 + 0.25 * wide * wide * (T < 8 ? T / 8.0 : 1.0) + rows * T / 8e6;
}

hipError_t launch_route(const LayerDims& L, const float* router_w, const float* router_bias, const void* x, int32_t T,
                        float* logits, int32_t* idx, float* gate, float* probs, hipStream_t st) {
  if (!route_in_one(L, T)) {
    if (hipError_t e = launch_router_logits(L, router_w, router_bias, x, T, logits, st); e != hipSuccess) return e;
    return launch_topk(L, logits, T, idx, gate, probs, st);
  }
  // tokens of a workgroup: one round of workgroups where that does it (600 tokens on 128 experts of 768 columns with two / four
  // 16.8 / 10.9 us); four take 64 KB of LDS at 1024 experts
  const int tg = T > 512 && L.n_experts <= 512 ? 4 : T > 256 ? 2 : 1, eb = L.n_experts <= 8 ? 4 : 8;
  const size_t lds = (size_t)kRouteClasses * tg * ((L.n_experts + eb - 1) / eb * eb) * sizeof(float);
  auto k = L.x_bf16 ? (tg == 4 ? pick_route<true, 4>(L) : tg == 2 ? pick_route<true, 2>(L) : pick_route<true, 1>(L))
                    : (tg == 4 ? pick_route<false, 4>(L) : tg == 2 ? pick_route<false, 2>(L) : pick_route<false, 1>(L));
  hipLaunchKernelGGL(k, dim3((T + tg - 1) / tg), dim3(kRouteWaves * 64), lds, st, L, router_w, router_bias, x, T, idx, gate, probs);
  return hipGetLastError();
}

hipError_t launch_router_logits(const LayerDims& L, const float* router_w, const float* router_bias, const void* x,
                                int32_t T, float* logits, hipStream_t st) {
  auto launch = [&](auto tg_tag) {
    constexpr int TG = decltype(tg_tag)::value;
    hipLaunchKernelGGL((L.x_bf16 ? k_router_logits<true, TG> : k_router_logits<false, TG>), dim3(L.n_experts, (T + TG - 1) / TG),
                       dim3(kThreads), 0, st, L, router_w, router_bias, x, T, logits);
    return hipGetLastError();
  };
  if (T == 1) return launch(std::integral_constant<int, 1>{});
  if (T <= 4) return launch(std::integral_constant<int, 4>{});
  return launch(std::integral_constant<int, kTokensPerWg>{});
}

}  // namespace moeq
