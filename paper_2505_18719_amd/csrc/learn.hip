// Learning-phase kernels of VLA-RL (Alg. 1 after the rollout loop, Eq. 2):
// generalised advantage estimation over a window of steps, the PPO-clip
// surrogate with its gradient w.r.t. the token log-probabilities, and the
// gradient of those log-probabilities w.r.t. the action logits.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace vla {
namespace {

constexpr int kGaeChunks = 16;  // waves per workgroup; each takes one slice of the time axis

// Steps t1 - 1 .. t0 of environment n, last first: step(t, delta_t, gamma lam (1 - d_{t+1}), V_t).  The recursion is
// serial but its inputs are not, so AHEAD steps' loads go out together (a window has few waves to cover a load's latency).
template <int AHEAD, class F>
__device__ __forceinline__ void gae_steps(const GaeArgs& a, int n, int t0, int t1, F step) {
  const size_t N = a.n_env;
  const float gl = a.gamma * a.lam;
  float vn = a.values[t1 * N + n];
  for (int t = t1 - 1; t >= t0; t -= AHEAD) {
    float r[AHEAD], v[AHEAD];
    uint8_t d[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
      if (t - u >= t0) {
        r[u] = a.rewards[(t - u) * N + n];
        v[u] = a.values[(t - u) * N + n];
        d[u] = a.dones[(t - u + 1) * N + n];
      }
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
      if (t - u >= t0) {
        const float c = d[u] ? 0.f : 1.f;
        step(t - u, r[u] + a.gamma * c * vn - v[u], gl * c, v[u]);
        vn = v[u];
      }
  }
}

// One workgroup per 64 environments, wave w the time slice [t0_w, t1_w).
// The recursion A_t = delta_t + k_t A_{t+1} (k_t = gamma lam (1 - d_{t+1}))
// is affine in A_{t+1}, so a slice maps the advantage after it to the one at
// its start as A_{t0} = P + Q A_{t1}.  Pass 1 composes each slice's map, the
// slice maps are chained backwards from A_M = 0 in LDS, and pass 2 replays
// each slice from its true incoming advantage, writing A_t and A_t + V_t.
// Every wave reads rows t of 64 consecutive environments (coalesced).
template <int AHEAD>
__global__ __launch_bounds__(64 * kGaeChunks) void gae_kernel(GaeArgs a) {
  __shared__ float P[kGaeChunks][64], Q[kGaeChunks][64], Ain[kGaeChunks][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int n = blockIdx.x * 64 + lane;
  const int N = a.n_env, M = a.n_steps;
  const int L = (M + kGaeChunks - 1) / kGaeChunks;
  const int t0 = min(M, w * L), t1 = min(M, t0 + L);
  const bool live = n < N;
  float p = 0.f, q = 1.f;
  if (live) {
    gae_steps<AHEAD>(a, n, t0, t1, [&](int, float delta, float kc, float) {
      p = delta + kc * p;
      q = kc * q;
    });
  }
  P[w][lane] = p;
  Q[w][lane] = q;
  __syncthreads();
  if (w == 0) {
    float nxt = 0.f;  // A_M
    for (int c = kGaeChunks - 1; c >= 0; --c) {
      Ain[c][lane] = nxt;
      nxt = P[c][lane] + Q[c][lane] * nxt;
    }
  }
  __syncthreads();
  if (!live) return;
  float adv = Ain[w][lane];
  gae_steps<AHEAD>(a, n, t0, t1, [&](int t, float delta, float kc, float v) {
    adv = delta + kc * adv;
    a.advantages[(size_t)t * N + n] = adv;
    if (a.returns) a.returns[(size_t)t * N + n] = adv + v;
  });
}

// The surrogate of action t: its term and clip flag are added to (surr, clip), its token gradient is returned.  The
// token loads are unrolled to MAX >= n_tokens, so that they are in flight together (0: a plain loop, for one or two tokens).
constexpr int kPpoMaxTokens = 16;
template <int MAX>
__device__ __forceinline__ float ppo_action(const PpoArgs& a, int t, float& surr, float& clip) {
  const float* ln = a.logp_new + (size_t)t * a.n_tokens;
  const float* lo = a.logp_old + (size_t)t * a.n_tokens;
  const float A = a.advantages[t];
  float sn = 0.f, so = 0.f;
  if constexpr (MAX == 0) {
    for (int i = 0; i < a.n_tokens; ++i) {
      sn += ln[i];
      so += lo[i];
    }
  } else {
    float vn[MAX], vo[MAX];
#pragma unroll
    for (int i = 0; i < MAX; ++i)
      if (i < a.n_tokens) {
        vn[i] = ln[i];
        vo[i] = lo[i];
      }
#pragma unroll
    for (int i = 0; i < MAX; ++i)
      if (i < a.n_tokens) {
        sn += vn[i];
        so += vo[i];
      }
  }
  const float rho = expf(sn - so);
  const float rc = fminf(fmaxf(rho, 1.f - a.eps), 1.f + a.eps);
  const bool clipped = ((A > 0.f) & (rho > 1.f + a.eps)) | ((A < 0.f) & (rho < 1.f - a.eps));  // no branches
  surr += fminf(rho * A, rc * A);
  clip += clipped ? 1.f : 0.f;
  return clipped ? 0.f : -rho * A / (float)a.n;
}

// Sums over a workgroup of NT threads by fixed wave and LDS trees; the totals are in threads 0 .. 63.
template <int NT>
__device__ __forceinline__ void ppo_block_sum(float& surr, float& clip) {
  __shared__ float red[2][NT / 64];
  const int tid = threadIdx.x;
  surr = wave_sum(surr);
  clip = wave_sum(clip);
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = surr;
    red[1][tid >> 6] = clip;
  }
  __syncthreads();
  if (tid < 64) {
    surr = wave_sum(tid < NT / 64 ? red[0][tid] : 0.f);
    clip = wave_sum(tid < NT / 64 ? red[1][tid] : 0.f);
  }
}

// PPO-clip over n actions in one workgroup: thread i takes actions i, i + 1024,
// ... in order, the partial sums are combined by fixed wave and LDS trees, so
// the loss is the same bits on every run.
constexpr int kPpoThreads = 1024;
template <int MAX>
__global__ __launch_bounds__(kPpoThreads) void ppo_clip_kernel(PpoArgs a) {
  float surr = 0.f, clip = 0.f;
  for (int t = threadIdx.x; t < a.n; t += kPpoThreads) {
    const float g = ppo_action<MAX>(a, t, surr, clip);
    float* dl = a.dlogp + (size_t)t * a.n_tokens;
    for (int i = 0; i < a.n_tokens; ++i) dl[i] = g;
  }
  ppo_block_sum<kPpoThreads>(surr, clip);
  if (threadIdx.x == 0) {
    a.stats[0] = -surr / (float)a.n;
    a.stats[1] = clip / (float)a.n;
  }
}

// The same over many workgroups, each a contiguous run of `per` actions (bound by one workgroup's load latency per
// pass of 1024 actions otherwise: 65536 actions 417 -> 10 us, 4096 actions 21.1 -> 7.6).  The entry point takes no scratch, so a workgroup
// leaves its sums, and the gradient that belongs there, in the first three token gradients of its first action
// (n_tokens >= 3); ppo_finish_kernel adds the sums in order and puts that action's gradient in place.  An action's
// inputs are read by its own thread before any of its gradients is written, as in the one-workgroup kernel.
constexpr int kPpoSplitThreads = 256;
__global__ __launch_bounds__(kPpoSplitThreads) void ppo_split_kernel(PpoArgs a, int per) {
  const int t0 = blockIdx.x * per, t1 = t0 + min(per, a.n - t0), tid = threadIdx.x;
  float surr = 0.f, clip = 0.f, g0 = 0.f;
  for (int t = t0 + tid; t < t1; t += kPpoSplitThreads) {
    const float g = ppo_action<kPpoMaxTokens>(a, t, surr, clip);
    if (t == t0) {
      g0 = g;
      continue;
    }
    float* dl = a.dlogp + (size_t)t * a.n_tokens;
    for (int i = 0; i < a.n_tokens; ++i) dl[i] = g;
  }
  ppo_block_sum<kPpoSplitThreads>(surr, clip);
  if (tid == 0) {
    float* dl = a.dlogp + (size_t)t0 * a.n_tokens;
    dl[0] = surr;
    dl[1] = clip;
    dl[2] = g0;
  }
}

constexpr long long kPpoSplitWork = 160 << 10;  // actions x tokens x (tokens + 1)
constexpr int kPpoMaxSplit = 1024;  // workgroups of ppo_split_kernel: one thread of ppo_finish_kernel each
__global__ __launch_bounds__(kPpoMaxSplit) void ppo_finish_kernel(PpoArgs a, int per, int groups) {
  const int b = threadIdx.x;
  float surr = 0.f, clip = 0.f;
  if (b < groups) {
    float* dl = a.dlogp + (size_t)b * per * a.n_tokens;
    surr = dl[0];
    clip = dl[1];
    const float g = dl[2];
    for (int i = 0; i < a.n_tokens; ++i) dl[i] = g;
  }
  ppo_block_sum<kPpoMaxSplit>(surr, clip);
  if (b == 0) {
    a.stats[0] = -surr / (float)a.n;
    a.stats[1] = clip / (float)a.n;
  }
}

// d log softmax(z / T)[k] / dz_j = (1[j = k] - p_j) / T, scaled by the
// arriving gradient; one wave per row, bins j = lane + 64 u.
__global__ __launch_bounds__(256) void logprob_backward_kernel(LogprobBwdArgs a) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= a.rows) return;
  const float* z = a.logits + (size_t)row * a.bins;
  float zt[4];
  float m = -INFINITY;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = lane + 64 * u;
    zt[u] = j < a.bins ? z[j] / a.temperature : -INFINITY;
    m = fmaxf(m, zt[u]);
  }
  m = wave_max(m);
  float e[4], se = 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    e[u] = lane + 64 * u < a.bins ? expf(zt[u] - m) : 0.f;
    se += e[u];
  }
  se = wave_sum(se);
  const int k = a.tokens[row] - a.action_begin;
  const float g = (k >= 0 && k < a.bins) ? a.dlogp[row] / a.temperature : __builtin_nanf("");
  const float inv = 1.f / se;
  float* dz = a.dlogits + (size_t)row * a.bins;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = lane + 64 * u;
    if (j < a.bins) dz[j] = g * ((j == k ? 1.f : 0.f) - e[u] * inv);
  }
}

// The same with 16 lanes per row and float4 loads and stores (bins % 4 == 0, 16-byte aligned rows): 4 KB of logits in
// flight per wave, 4-step trees for four rows at once where the kernel above runs 6-step ones for one, and (z - max) times
// 1 / T where it divides (the division's and expf's instructions, not memory, bounded it: 458752 x 256 305 us = 3.1 TB/s
// -> 157 us = 6.0 TB/s).  The maximum is taken off before the scaling: its exponent is 0 whatever max / T is, where a fused
// z / T - round(max / T) leaves the rounding error of max / T, which past |max / T| = 2^31 is more than expf's range.
__global__ __launch_bounds__(256) void logprob_backward4_kernel(LogprobBwdArgs a) {
  const int row = blockIdx.x * 16 + (threadIdx.x >> 4);
  const int l = threadIdx.x & 15, lim4 = a.bins / 4;
  const bool in = row < a.rows;
  const float4* z = reinterpret_cast<const float4*>(a.logits + (size_t)(in ? row : 0) * a.bins);
  const float inv_t = 1.f / a.temperature;
  float v[4][4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const float4 q = l + 16 * u < lim4 ? z[l + 16 * u] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    v[u][0] = q.x; v[u][1] = q.y; v[u][2] = q.z; v[u][3] = q.w;
  }
  const int tok = a.tokens[in ? row : 0];
  const float dl = a.dlogp[in ? row : 0];
  float m = -INFINITY;
#pragma unroll
  for (int u = 0; u < 4; ++u) m = fmaxf(m, fmaxf(fmaxf(v[u][0], v[u][1]), fmaxf(v[u][2], v[u][3])));
  m = row_max16(m);
  float su[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const bool live = l + 16 * u < lim4;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[u][e] = live ? expf((v[u][e] - m) * inv_t) : 0.f;
    su[u] = (v[u][0] + v[u][1]) + (v[u][2] + v[u][3]);
  }
  const float se = row_sum16((su[0] + su[1]) + (su[2] + su[3]));
  const int k = tok - a.action_begin;
  const float g = (k >= 0 && k < a.bins) ? dl / a.temperature : __builtin_nanf("");
  const float inv = 1.f / se;
  if (!in) return;
  float4* dz = reinterpret_cast<float4*>(a.dlogits + (size_t)row * a.bins);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = 4 * (l + 16 * u);
    if (j < a.bins)
      dz[l + 16 * u] = make_float4(g * ((j == k ? 1.f : 0.f) - v[u][0] * inv), g * ((j + 1 == k ? 1.f : 0.f) - v[u][1] * inv),
                                   g * ((j + 2 == k ? 1.f : 0.f) - v[u][2] * inv), g * ((j + 3 == k ? 1.f : 0.f) - v[u][3] * inv));
  }
}

}  // namespace

hipError_t launch_gae(const GaeArgs& a, hipStream_t s) {
  if (a.n_env <= 0 || a.n_steps <= 0) return hipSuccess;
  const dim3 grid((a.n_env + 63) / 64), block(64 * kGaeChunks);
  // Eight steps' loads together where a slice has more than four steps and the rows of its steps are not in one cache line
  // (inputs not in the caches, us, one by one / eight: 64 x 512 26.6 / 16.0, 256 x 256 14.6 / 10.0, 16 x 512 24.6 / 15.1;
  // in the caches 4096 x 512 22.5 / 16.6, 64 x 512 13.7 / 13.7).  Otherwise the loads that a window has no steps for only
  // cost (in the caches 64 x 16 2.1 / 2.7, 64 x 64 3.4 / 3.6; one environment, 512 steps, 15.6 / 16.9).
  if (a.n_steps > 4 * kGaeChunks && a.n_env >= 16) hipLaunchKernelGGL(gae_kernel<8>, grid, block, 0, s, a);
  else hipLaunchKernelGGL(gae_kernel<1>, grid, block, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_ppo_clip(const PpoArgs& a, hipStream_t s) {
  if (a.n <= 0) return hipErrorInvalidValue;
  // One workgroup where that takes less than the second launch costs: its time goes with the actions and about the square
  // of their tokens (strided loads), and it meets the 12 us of a call of two launches at 3000 actions of 7 tokens (13.5 / 11.9
  // us a call), 9000 of 3 (11.6 / 12), 600 of 16 (13.7 / 12); 4096 of 7 17.7 / 12.1, 2048 of 7 9.8 / 11.9; 8 tokens take
  // twice as long as the others would have it (2048 actions 21 us).  And below 3 tokens, where an action's gradients have no
  // room for a workgroup's sums.  The loads are unrolled to little more than the tokens: 20000 actions of one token take 10.0
  // us, with 16 loads unrolled 19.5.
  const long long work = (long long)a.n * a.n_tokens * (a.n_tokens + 1) * (a.n_tokens == 8 ? 2 : 1);
  if (a.n_tokens < 3 || work < kPpoSplitWork) {
    const dim3 block(kPpoThreads);
    if (a.n_tokens <= 2) hipLaunchKernelGGL(ppo_clip_kernel<0>, dim3(1), block, 0, s, a);
    else if (a.n_tokens <= 4) hipLaunchKernelGGL(ppo_clip_kernel<4>, dim3(1), block, 0, s, a);
    else if (a.n_tokens <= 8) hipLaunchKernelGGL(ppo_clip_kernel<8>, dim3(1), block, 0, s, a);
    else hipLaunchKernelGGL(ppo_clip_kernel<kPpoMaxTokens>, dim3(1), block, 0, s, a);
  } else {
    const int per = std::max(kPpoSplitThreads, (a.n - 1) / kPpoMaxSplit + 1), groups = (a.n - 1) / per + 1;
    hipLaunchKernelGGL(ppo_split_kernel, dim3(groups), dim3(kPpoSplitThreads), 0, s, a, per);
    hipLaunchKernelGGL(ppo_finish_kernel, dim3(1), dim3(kPpoMaxSplit), 0, s, a, per, groups);
  }
  return hipGetLastError();
}

hipError_t launch_logprob_backward(const LogprobBwdArgs& a, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  if (a.bins <= 0 || a.bins > 256) return hipErrorInvalidValue;
  // float4 rows, and a temperature whose reciprocal is a normal number and so small that where z - max overflows to -inf,
  // its exponential is 0 anyway
  const uintptr_t align = reinterpret_cast<uintptr_t>(a.logits) | reinterpret_cast<uintptr_t>(a.dlogits);
  if (a.bins % 4 == 0 && align % 16 == 0 && a.temperature >= 0x1p-100f && a.temperature <= 0x1p100f)
    hipLaunchKernelGGL(logprob_backward4_kernel, dim3((a.rows + 15) / 16), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(logprob_backward_kernel, dim3((a.rows + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace vla
