// Device side of a decode step's input (embedding row and first RMSNorm), shared by the kernel of its own
// (elementwise.hip) and the sampler that goes on to it (attention.hip).
#pragma once

#include "common.h"
#include "kernels.h"

namespace vla {

// Block-wide sum over 256 threads.
__device__ __forceinline__ float block_sum256(float v, float* sh) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  return sh[0] + sh[1] + sh[2] + sh[3];
}

constexpr int kMaxPerThread = 32;  // d <= 8192

// Row b from token `id`, by a 256-thread workgroup (sh: 4 floats of LDS); the gain is loaded with the embedding row.
__device__ __forceinline__ void embed_token_row(const EmbedTokenArgs& a, int id, int b, float* sh) {
  const bool ok = id >= 0 && id < a.vocab;
  const int d = a.d;
  if (!ok && threadIdx.x == 0) atomicOr(a.flags, 1u);
  uint2 e[kMaxPerThread / 4];
  float4 gv[kMaxPerThread / 4];
  float v[kMaxPerThread];
  float ss = 0.f;
  const int n = (d / 4 + 255) / 256;  // groups of 4 columns per thread
#pragma unroll
  for (int t = 0; t < kMaxPerThread / 4; ++t) {
    if (t >= n) break;
    const int c = 4 * (threadIdx.x + 256 * t);
    if (c >= d) continue;
    e[t] = ok ? *reinterpret_cast<const uint2*>(a.emb + (size_t)id * d + c) : make_uint2(0, 0);
    gv[t] = *reinterpret_cast<const float4*>(a.g + c);
  }
#pragma unroll
  for (int t = 0; t < kMaxPerThread / 4; ++t) {
    if (t >= n) break;
    const int c = 4 * (threadIdx.x + 256 * t);
    if (c >= d) {
      v[4 * t] = v[4 * t + 1] = v[4 * t + 2] = v[4 * t + 3] = 0.f;
      continue;
    }
    v[4 * t] = __uint_as_float(e[t].x << 16);
    v[4 * t + 1] = __uint_as_float(e[t].x & 0xffff0000u);
    v[4 * t + 2] = __uint_as_float(e[t].y << 16);
    v[4 * t + 3] = __uint_as_float(e[t].y & 0xffff0000u);
    ss += v[4 * t] * v[4 * t] + v[4 * t + 1] * v[4 * t + 1] + v[4 * t + 2] * v[4 * t + 2] +
          v[4 * t + 3] * v[4 * t + 3];
  }
  ss = block_sum256(ss, sh);
  const float r = rsqrtf(ss / (float)d + a.eps);
#pragma unroll
  for (int t = 0; t < kMaxPerThread / 4; ++t) {
    if (t >= n) break;
    const int c = 4 * (threadIdx.x + 256 * t);
    if (c >= d) break;
    *reinterpret_cast<float4*>(a.x + (size_t)b * d + c) = make_float4(v[4 * t], v[4 * t + 1], v[4 * t + 2], v[4 * t + 3]);
    *reinterpret_cast<uint2*>(a.u + frag_index(b, c, d)) =
        make_uint2(pack2bf(v[4 * t] * r * gv[t].x, v[4 * t + 1] * r * gv[t].y),
                   pack2bf(v[4 * t + 2] * r * gv[t].z, v[4 * t + 3] * r * gv[t].w));
  }
}

}  // namespace vla
