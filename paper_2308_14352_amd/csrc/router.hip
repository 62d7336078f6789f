// Router GEMV (Section 1; Section 2.1: a small router scores the experts for every token).
// logits[t][e] = router_w[e] . x[t] (+ bias[e]) in fp32. One workgroup per (expert, group of up to 8
// tokens): the expert's row is read once with 128-bit loads and dotted with each token of the group;
// partial sums are folded with DPP inside each wavefront, then across the wavefronts through LDS.
// The softmax and the top-k selection run where the result is needed (see the FFN kernels).
#include "decode_core.h"

namespace moeq {
namespace {

constexpr int kThreads = 256;
constexpr int kTokensPerWg = 8;

template <bool BF16>
__global__ __launch_bounds__(kThreads) void k_router_logits(LayerDims L, const float* __restrict__ Wr,
                                                            const float* __restrict__ bias,
                                                            const void* __restrict__ x, int32_t T,
                                                            float* __restrict__ logits) {
  __shared__ float part[kThreads / 64][kTokensPerWg];
  const int d = L.d_model, E = L.n_experts;
  const int e = blockIdx.x;
  const int t0 = blockIdx.y * kTokensPerWg;
  const int nt = min(kTokensPerWg, T - t0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* wr = Wr + (size_t)e * d;
  float acc[kTokensPerWg];
#pragma unroll
  for (int tt = 0; tt < kTokensPerWg; ++tt) acc[tt] = 0.f;
  for (int i = tid * 4; i < d; i += kThreads * 4) {
    const float4 w = *(const float4*)(wr + i);
#pragma unroll
    for (int tt = 0; tt < kTokensPerWg; ++tt) {
      if (tt < nt) {
        float4 v;
        if (BF16) {
          const ushort4 b = *(const ushort4*)((const uint16_t*)x + (size_t)(t0 + tt) * d + i);
          v = make_float4(bf16_bits_to_f32(b.x), bf16_bits_to_f32(b.y), bf16_bits_to_f32(b.z), bf16_bits_to_f32(b.w));
        } else {
          v = *(const float4*)((const float*)x + (size_t)(t0 + tt) * d + i);
        }
        acc[tt] = fmaf(w.x, v.x, acc[tt]); acc[tt] = fmaf(w.y, v.y, acc[tt]);
        acc[tt] = fmaf(w.z, v.z, acc[tt]); acc[tt] = fmaf(w.w, v.w, acc[tt]);
      }
    }
  }
#pragma unroll
  for (int tt = 0; tt < kTokensPerWg; ++tt) {
    if (tt < nt) {   // uniform over the workgroup
      const float v = wave_sum(acc[tt]);
      if (lane == 0) part[wave][tt] = v;
    }
  }
  __syncthreads();
  if (tid < nt) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) v += part[w][tid];
    logits[(size_t)(t0 + tid) * E + e] = v + (bias ? bias[e] : 0.f);
  }
}

// Router and top-k of TG tokens in one workgroup: the calls of many tokens, where the logits in memory and a second kernel
// cost as much as the sums. A wavefront's unit is eight experts x a range of the columns: all experts' rows are requested
// together, four steps of 256 columns at a time, and meet the TG tokens in registers; a transposing fold leaves the sum of
// expert l % 8 in lane l. With few experts the eight wavefronts split the columns as well. us, with k_router_logits + k_topk
// before: Mixtral layer (8 experts, d_model 4096) 117 tokens 16.4 + 4.7 -> 6.3, 2048 tokens 22.7 + 4.8 -> 15.0; 64 experts,
// d_model 768, 500 tokens 12.8 + 4.7 -> 6. A workgroup reads every expert's row, so it takes two tokens from 256 on and four
// from 1024 on, where all compute units have several workgroups all the same.
constexpr int kRouteWaves = 8, kRouteSteps = 4;
template <bool BF16, int TG>
__global__ __launch_bounds__(kRouteWaves * 64) void k_route(LayerDims L, const float* __restrict__ Wr, const float* __restrict__ bias,
                                                            const void* __restrict__ x, int32_t T, int32_t* __restrict__ idx,
                                                            float* __restrict__ gate) {
  extern __shared__ float rsm[];                 // [column ranges][TG][experts, whole blocks of eight]
  const int d = L.d_model, E = L.n_experts, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = (E + 7) / 8, t0 = blockIdx.x * TG;
  const int cs = nb == 1 ? 8 : nb == 2 ? 4 : nb <= 4 ? 2 : 1;              // column ranges
  const int seg = (d / cs + 255) / 256 * 256;
  for (int u = wave; u < nb * cs; u += kRouteWaves) {
    const int eb = u / cs, c_begin = (u - eb * cs) * seg, c_end = min(d, c_begin + seg);
    float acc[TG][8];
#pragma unroll
    for (int t = 0; t < TG; ++t)
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[t][i] = 0.f;
    for (int c0 = c_begin + lane * 4; c0 < c_end; c0 += 256 * kRouteSteps) {
      float4 w[kRouteSteps][8], v[kRouteSteps][TG];
#pragma unroll
      for (int j = 0; j < kRouteSteps; ++j) {
        const int c = c0 + 256 * j;
#pragma unroll
        for (int t = 0; t < TG; ++t) v[j][t] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (c < c_end) {
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
          for (int i = 0; i < 8; ++i) w[j][i] = *(const float4*)(Wr + (size_t)min(eb * 8 + i, E - 1) * d + c);     // rows past E repeat the last one
        }
      }
#pragma unroll
      for (int j = 0; j < kRouteSteps; ++j)
        if (c0 + 256 * j < c_end)
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int t = 0; t < TG; ++t) {
              acc[t][i] = fmaf(w[j][i].x, v[j][t].x, acc[t][i]); acc[t][i] = fmaf(w[j][i].y, v[j][t].y, acc[t][i]);
              acc[t][i] = fmaf(w[j][i].z, v[j][t].z, acc[t][i]); acc[t][i] = fmaf(w[j][i].w, v[j][t].w, acc[t][i]);
            }
    }
#pragma unroll
    for (int t = 0; t < TG; ++t) {
      float a[4], b[2];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float lo = acc[t][2 * i], hi = acc[t][2 * i + 1];
        a[i] = ((lane & 1) ? hi : lo) + dpp<kDppXor1>((lane & 1) ? lo : hi);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) b[i] = ((lane & 2) ? a[2 * i + 1] : a[2 * i]) + dpp<kDppXor2>((lane & 2) ? a[2 * i] : a[2 * i + 1]);
      float s = ((lane & 4) ? b[1] : b[0]) + __shfl_xor((lane & 4) ? b[0] : b[1], 4);
      s += dpp<kDppRor8>(s);
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      if (lane < 8) rsm[((u - eb * cs) * TG + t) * (nb * 8) + eb * 8 + lane] = s;
    }
  }
  __syncthreads();
  if (wave < TG && t0 + wave < T) {
    float* lg = rsm + wave * (nb * 8);
    for (int e = lane; e < E; e += 64) {
      float s = lg[e];
      for (int r = 1; r < cs; ++r) s += lg[r * TG * (nb * 8) + e];
      lg[e] = s + (bias ? bias[e] : 0.f);
    }
    topk_from_logits(lg, E, L.top_k, L.renorm, lane, idx + (size_t)(t0 + wave) * L.top_k, gate + (size_t)(t0 + wave) * L.top_k, nullptr);
  }
}

}  // namespace

hipError_t launch_route(const LayerDims& L, const float* router_w, const float* router_bias, const void* x, int32_t T,
                        int32_t* idx, float* gate, hipStream_t st) {
  const int nb = (L.n_experts + 7) / 8, cs = nb == 1 ? 8 : nb == 2 ? 4 : nb <= 4 ? 2 : 1;
  const int tg = T >= 1024 ? 4 : T >= 256 ? 2 : 1;
  const size_t lds = (size_t)cs * tg * nb * 8 * sizeof(float);
  auto k = L.x_bf16 ? (tg == 4 ? k_route<true, 4> : tg == 2 ? k_route<true, 2> : k_route<true, 1>)
                    : (tg == 4 ? k_route<false, 4> : tg == 2 ? k_route<false, 2> : k_route<false, 1>);
  hipLaunchKernelGGL(k, dim3((T + tg - 1) / tg), dim3(kRouteWaves * 64), lds, st, L, router_w, router_bias, x, T, idx, gate);
  return hipGetLastError();
}

hipError_t launch_router_logits(const LayerDims& L, const float* router_w, const float* router_bias, const void* x,
                                int32_t T, float* logits, hipStream_t st) {
  const dim3 grid(L.n_experts, (T + kTokensPerWg - 1) / kTokensPerWg);
  if (L.x_bf16)
    hipLaunchKernelGGL(k_router_logits<true>, grid, dim3(kThreads), 0, st, L, router_w, router_bias, x, T, logits);
  else
    hipLaunchKernelGGL(k_router_logits<false>, grid, dim3(kThreads), 0, st, L, router_w, router_bias, x, T, logits);
  return hipGetLastError();
}

}  // namespace moeq
