// Memory-bound kernels of the VLA rollout path on gfx950: input assembly,
// RMSNorm (one wave per row, fp32 statistics), the consumers of the decode
// GEMM's split-K partials (residual add + RMSNorm, SwiGLU, RoPE + KV append,
// logits), and one-time weight repacking.  All loads and stores are 16-byte
// vectors where the layout allows.
#include <algorithm>

#include "common.h"
#include "embed_dev.h"
#include "kernels.h"
#include "lds_limit.h"

namespace vla {

namespace {

// ------------------------------------------------------------------ embed
// x^0 rows of each environment: n_visual projected visual embeddings, then the
// embedding rows of its prompt ids, then (teacher-forced pass) its actions.
__global__ __launch_bounds__(256) void embed_kernel(EmbedArgs a) {
  const int row = blockIdx.x;
  const int env = a.row_env[row], pos = a.row_pos[row];
  const bf16_t* src;
  if (pos < a.n_visual) {
    src = a.vis + ((size_t)env * a.n_visual + pos) * a.d;
  } else {
    int id;
    if (pos < a.env_prefix[env]) id = a.prompt_ids[a.env_prompt_off[env] + pos - a.n_visual];
    else id = a.actions[env * a.n_actions + pos - a.env_prefix[env]];
    if (id < 0 || id >= a.vocab) {
      if (threadIdx.x == 0) atomicOr(a.flags, 1u);
      src = nullptr;
    } else {
      src = a.emb + (size_t)id * a.d;
    }
  }
  float* dst = a.x + (size_t)row * a.d;
  for (int c = threadIdx.x * 8; c < a.d; c += 256 * 8) {
    float f[8];
    if (src) unpack8(*reinterpret_cast<const uint4*>(src + c), f);
    else
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = 0.f;
    reinterpret_cast<float4*>(dst + c)[0] = make_float4(f[0], f[1], f[2], f[3]);
    reinterpret_cast<float4*>(dst + c)[1] = make_float4(f[4], f[5], f[6], f[7]);
  }
}

// ------------------------------------------------------------------ RMSNorm
// One wave per row: u = bf16(x * rsqrt(mean(x^2) + eps) * g), row-major (row stride ldu).
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float* __restrict__ x, int ldx,
                                                      const int32_t* __restrict__ rows,
                                                      const float* __restrict__ g, float eps,
                                                      bf16_t* __restrict__ u, int ldu, int M, int d) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= M) return;
  const int src = rows ? rows[i] : i;
  const float* xr = x + (size_t)src * ldx;
  float ss = 0.f;
  for (int c = lane * 4; c < d; c += 256) {
    const float4 v = *reinterpret_cast<const float4*>(xr + c);
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  ss = wave_sum(ss);
  const float r = rsqrtf(ss / (float)d + eps);
  bf16_t* ur = u + (size_t)i * ldu;
  for (int c = lane * 4; c < d; c += 256) {
    const float4 v = *reinterpret_cast<const float4*>(xr + c);
    const float4 w = *reinterpret_cast<const float4*>(g + c);
    uint2 o;
    o.x = pack2bf(v.x * r * w.x, v.y * r * w.y);
    o.y = pack2bf(v.z * r * w.z, v.w * r * w.w);
    *reinterpret_cast<uint2*>(ur + c) = o;
  }
}

// RMSNorm into frag layout.  A workgroup of RPW waves normalises RPW rows of
// one 16-row frag block (RPW = 16: the whole block; 8: one half), one wave per
// row: the wave reads its row once into registers (NJ float4 per lane, 1 KB
// per load instruction), reduces the mean square, and writes the scaled bf16
// row into LDS, row-major with a 16-byte pad per row; the workgroup then reads
// LDS in frag order (the pad puts the 8 rows of one 16-lane read phase on
// distinct banks) and writes each 1 KB block as one contiguous store per 64
// (or 32) lanes.  Rows past M are written as zeros.
template <int NJ, int RPW>
__global__ __launch_bounds__(64 * RPW) void rmsnorm_frag_kernel(const float* __restrict__ x, int ldx,
                                                                const int32_t* __restrict__ rows,
                                                                const float* __restrict__ g, float eps,
                                                                bf16_t* __restrict__ u, int M, int d) {
  extern __shared__ uint4 norm_lds[];
  char* ls = reinterpret_cast<char*>(norm_lds);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = blockIdx.x * RPW, nj = d / 256;
  const int lrow = 2 * d + 16;  // LDS bytes per row
  char* lr = ls + wave * lrow + 8 * lane;
  if (r0 + wave < M) {  // wave-uniform
    const int i = r0 + wave;
    const float* xr = x + (size_t)(rows ? rows[i] : i) * ldx + 4 * lane;
    float4 v[NJ];
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      if (j < nj) v[j] = *reinterpret_cast<const float4*>(xr + 256 * j);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      if (j < nj) ss += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
    ss = wave_sum(ss);
    const float r = rsqrtf(ss / (float)d + eps);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      if (j < nj) {
        const float4 gv = *reinterpret_cast<const float4*>(g + 4 * lane + 256 * j);
        *reinterpret_cast<uint2*>(lr + 512 * j) =
            make_uint2(pack2bf(v[j].x * r * gv.x, v[j].y * r * gv.y), pack2bf(v[j].z * r * gv.z, v[j].w * r * gv.w));
      }
  } else {
    for (int j = 0; j < nj; ++j) *reinterpret_cast<uint2*>(lr + 512 * j) = make_uint2(0, 0);
  }
  __syncthreads();
  // block kb of the 16-row block: lane l = row % 16 + 16 (k % 32 / 8) holds 16 bytes
  constexpr int LPB = 4 * RPW;  // lanes of a block this workgroup writes
  const int idx = threadIdx.x % LPB, rr = idx % RPW, q = idx / RPW;
  const int ro = r0 & 15, l = ro + rr + 16 * q;
  bf16_t* ub = u + frag_index(r0 & ~15, 0, d) + 8 * l;
  const char* src = ls + rr * lrow + 16 * q;
  for (int kb = threadIdx.x / LPB; kb < d / 32; kb += 16)
    *reinterpret_cast<uint4*>(ub + (size_t)kb * 512) = *reinterpret_cast<const uint4*>(src + 64 * kb);
}

__global__ __launch_bounds__(256) void embed_token_norm_kernel(const int32_t* tok, EmbedTokenArgs a) {
  __shared__ float sh[4];
  embed_token_row(a, tok[blockIdx.x], blockIdx.x, sh);
}

// One workgroup per row: 4 consecutive columns per thread and pass (1024 threads in two passes cover d <= 8192, smaller
// rows take d / 4 threads), the partial slots' float4s and the gain in flight together.  Two waits bound it (the loads,
// the sum over the waves); the gain's load after them was a third.  d = 256: 2.7 -> 2.6 us, d = 1024: 3.9 -> 3.7.
__global__ __launch_bounds__(1024) void reduce_residual_norm_kernel(const float* __restrict__ part, SkinnyPlan p,
                                                                    float* __restrict__ x, bf16_t* __restrict__ u,
                                                                    const float* __restrict__ g, float eps, int M,
                                                                    int d) {
  __shared__ float sh[16];
  const int m = blockIdx.x;
  float4 v[2], gv[2];
  float ss = 0.f;
#pragma unroll
  for (int t = 0; t < 2; ++t) {  // d <= 8192
    const int c = 4 * (threadIdx.x + 1024 * t);
    if (c >= d) break;
    gv[t] = *reinterpret_cast<const float4*>(g + c);
    const float4 a = sum_slots4(part + (size_t)m * d + c, (size_t)M * d, skinny_slots(p, c >> 6),
                                *reinterpret_cast<const float4*>(x + (size_t)m * d + c));
    v[t] = a;
    ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w)
    if (w < (int)blockDim.x / 64) ss += sh[w];
  const float r = rsqrtf(ss / (float)d + eps);
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int c = 4 * (threadIdx.x + 1024 * t);
    if (c >= d) break;
    *reinterpret_cast<float4*>(x + (size_t)m * d + c) = v[t];
    *reinterpret_cast<uint2*>(u + frag_index(m, c, d)) =
        make_uint2(pack2bf(v[t].x * r * gv[t].x, v[t].y * r * gv[t].y),
                   pack2bf(v[t].z * r * gv[t].z, v[t].w * r * gv[t].w));
  }
}

__global__ __launch_bounds__(256) void reduce_sum_kernel(const float* __restrict__ part, SkinnyPlan p,
                                                         float* __restrict__ z, int M, int N,
                                                         float* __restrict__ z2) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)M * N) return;
  const int m = (int)(i / N), n = (int)(i % N);
  const float v = skinny_sum(part, p, M, p.tiles * 64, m, n);
  z[i] = v;
  if (z2) z2[i] = v;
}

__global__ __launch_bounds__(256) void reduce_swiglu_kernel(const float* __restrict__ part, SkinnyPlan p,
                                                            bf16_t* __restrict__ h, int ldh, int M, int F) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;  // group of 4 consecutive j
  if (i >= (size_t)M * (F / 4)) return;
  const int m = (int)(i / (F / 4)), j = 4 * (int)(i % (F / 4));
  const int N = p.tiles * 64;
  const int cg = 64 * (j >> 5) + (j & 31);  // gate columns cg .. cg+3, up columns 32 further (one 64-column tile)
  const int ns = skinny_slots(p, cg >> 6);
  const float* pr = part + (size_t)m * N + cg;
  const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
  const float4 gs = sum_slots4(pr, (size_t)M * N, ns, z), us = sum_slots4(pr + 32, (size_t)M * N, ns, z);
  auto sw = [](float a, float b) { return a / (1.f + expf(-a)) * b; };
  *reinterpret_cast<uint2*>(h + frag_index(m, j, ldh)) =
      make_uint2(pack2bf(sw(gs.x, us.x), sw(gs.y, us.y)), pack2bf(sw(gs.z, us.z), sw(gs.w, us.w)));
}

// ------------------------------------------------------------------ repacking
// One 16-byte chunk (8 K elements) of destination row r per thread, written in
// frag layout.  The source row (or a zero row) follows the packing mode:
//  kPackRows:   source row r, rows >= src_rows zero, K elements >= src_cols zero
//  kPackQk:     q/k rows of each head reordered so that each 64-row block holds
//               rotary pairs 32 rows apart: block b = rows [32b, 32b+32) then
//               [half+32b, half+32b+32)
//  kPackGateUp: [gate; up] interleaved in blocks of 32 rows, zero rows past src_rows
__global__ __launch_bounds__(256) void pack_frag_kernel(PackArgs a) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int kc = a.K / 8;
  if (i >= (size_t)a.rows * kc) return;
  const int r = (int)(i / kc), k = (int)(i % kc) * 8;
  int part;
  const int j = pack_src_row(a.mode, r, a.head_dim, a.src_rows, part);
  const bf16_t* src = j < 0 ? nullptr : (part ? a.src2 : a.src) + (size_t)j * a.src_ld;
  bf16_t v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (src && k + e < a.src_cols) ? src[k + e] : (bf16_t)0;
  uint4 o;
  o.x = v[0] | (uint32_t(v[1]) << 16);
  o.y = v[2] | (uint32_t(v[3]) << 16);
  o.z = v[4] | (uint32_t(v[5]) << 16);
  o.w = v[6] | (uint32_t(v[7]) << 16);
  *reinterpret_cast<uint4*>(a.dst + frag_index(r, k, a.K)) = o;
}

// a[r, i] = lo_i + (k + 1/2) (hi_i - lo_i) / bins for bin k = tokens[r, i] - action_begin,
// NaN outside the bins; one thread per element.
__global__ void extract_actions_kernel(const int32_t* __restrict__ tokens, int n_elems, int n_dims, int action_begin,
                                       int bins, const float* __restrict__ lo, const float* __restrict__ hi,
                                       float* __restrict__ out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n_elems) return;
  const int dim = i % n_dims;
  const int k = tokens[i] - action_begin;
  const float l = lo[dim];
  out[i] = (k >= 0 && k < bins) ? l + ((float)k + 0.5f) * (hi[dim] - l) / (float)bins : __builtin_nanf("");
}

// Row i of the compact buffers takes row rows[i]: the fp32 residual row and the
// bf16 frag-layout row (8 elements = 16 bytes per thread step).
__global__ void gather_rows_kernel(const float* __restrict__ x, const bf16_t* __restrict__ o,
                                   const int32_t* __restrict__ rows, int d, float* __restrict__ xc,
                                   bf16_t* __restrict__ oc) {
  const int i = blockIdx.x, r = rows[i];
  for (int k = 8 * threadIdx.x; k < d; k += 8 * 256) {
    const float4* xs = reinterpret_cast<const float4*>(x + (size_t)r * d + k);
    float4* xd = reinterpret_cast<float4*>(xc + (size_t)i * d + k);
    xd[0] = xs[0];
    xd[1] = xs[1];
    *reinterpret_cast<uint4*>(oc + frag_index(i, k, d)) = *reinterpret_cast<const uint4*>(o + frag_index(r, k, d));
  }
}

__global__ void bf16_to_f32_kernel(float* dst, const bf16_t* src, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = bf2f(src[i]);
}

// dst = src, 4 x 16 bytes per thread; the stores bypass the caches (404 MB: 5.0 -> 5.6 TB/s, the runtime's copy
// before; smaller copies: launch_copy).  Only vla_debug_read copies so.
__global__ __launch_bounds__(256) void copy_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, size_t n16) {
  const size_t i0 = (size_t)blockIdx.x * 1024 + threadIdx.x;
  u32x4 v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (i0 + 256 * u < n16) v[u] = src[i0 + 256 * u];
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (i0 + 256 * u < n16) __builtin_nontemporal_store(v[u], dst + i0 + 256 * u);
}

__global__ void fill_zero_kernel(uint4* dst, size_t n16) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256)
    dst[i] = make_uint4(0, 0, 0, 0);
}

}  // namespace

hipError_t launch_embed(const EmbedArgs& a, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.d % 8 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(embed_kernel, dim3(a.M), dim3(256), 0, s, a);
  return hipGetLastError();
}

namespace {
template <int NJ, int RPW>
hipError_t launch_norm_frag(const float* x, int ldx, const int32_t* rows, const float* g, float eps, bf16_t* u,
                            int M, int d, hipStream_t s) {
  const size_t lds = (size_t)RPW * (2 * d + 16);
  static LdsLimit limit;
  const hipError_t e = limit.allow(reinterpret_cast<const void*>(&rmsnorm_frag_kernel<NJ, RPW>), RPW * (2 * 256 * NJ + 16));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((rmsnorm_frag_kernel<NJ, RPW>), dim3((M + RPW - 1) / RPW), dim3(64 * RPW), lds, s, x, ldx, rows,
                     g, eps, u, M, d);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_rmsnorm(const float* x, int ldx, const int32_t* rows, const float* g, float eps, bf16_t* u,
                          int ldu, int M, int d, hipStream_t s, bool frag) {
  if (M <= 0) return hipSuccess;
  if (d % 4 != 0 || (frag && d % 32 != 0)) return hipErrorInvalidValue;
  if (frag) {
    if (d % 256 != 0 || d > 8192) return hipErrorInvalidValue;
    if (d <= 4096) return launch_norm_frag<16, 8>(x, ldx, rows, g, eps, u, M, d, s);
    return launch_norm_frag<32, 8>(x, ldx, rows, g, eps, u, M, d, s);
  }
    hipLaunchKernelGGL(rmsnorm_kernel, dim3((M + 3) / 4), dim3(256), 0, s, x, ldx, rows, g, eps, u, ldu, M, d);
  return hipGetLastError();
}

hipError_t launch_embed_token_norm(const int32_t* tok, const bf16_t* emb, float* x, bf16_t* u, const float* g,
                                   float eps, int B, int d, int vocab, uint32_t* flags, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  if (d > 256 * kMaxPerThread || d % 32 != 0) return hipErrorInvalidValue;
  const EmbedTokenArgs a{emb, x, u, g, eps, d, vocab, flags};
  hipLaunchKernelGGL(embed_token_norm_kernel, dim3(B), dim3(256), 0, s, tok, a);
  return hipGetLastError();
}

hipError_t launch_reduce_residual_norm(const float* part, const SkinnyPlan& p, float* x, bf16_t* u, const float* g,
                                       float eps, int M, int d, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (d > 8192 || d % 64 != 0 || p.tiles * 64 != d) return hipErrorInvalidValue;
  hipLaunchKernelGGL(reduce_residual_norm_kernel, dim3(M), dim3(std::min(1024, (d / 4 + 63) / 64 * 64)), 0, s, part, p, x, u, g, eps, M, d);
  return hipGetLastError();
}

hipError_t launch_reduce_sum(const float* part, const SkinnyPlan& p, float* z, int M, int N, hipStream_t s,
                             float* z2) {
  const size_t n = (size_t)M * N;
  if (n == 0) return hipSuccess;
  if (N > p.tiles * 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(reduce_sum_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, part, p, z, M, N,
                     z2);
  return hipGetLastError();
}

hipError_t launch_reduce_swiglu(const float* part, const SkinnyPlan& p, bf16_t* h, int ldh, int M, int F,
                                hipStream_t s) {
  const size_t n = (size_t)M * (F / 4);
  if (n == 0) return hipSuccess;
  if (2 * F > p.tiles * 64 || F % 32 != 0 || ldh < F) return hipErrorInvalidValue;
  hipLaunchKernelGGL(reduce_swiglu_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, part, p, h, ldh, M, F);
  return hipGetLastError();
}

// LoRA merge, one 256-thread workgroup per kMergeRows rows x COLS K columns.  Rows are
// the projection's own rows in packed order: for the interleaved [gate; up]
// weight only the 32-row halves of `part`, so no workgroup computes rows it
// does not write.  The update is taken transposed, A^T B^T on MFMA, a 16-row block of the projection in the columns of
// the product and K columns 8 (i / 4) + 4 t + i % 4 of a 32-column block in row i of its tiles t = 0, 1: lane (row
// l % 16, K elements 8 (l / 16) ..) then holds the update of the 16 bytes that it holds in frag layout, so the original
// weights are loaded to that layout, the update is added in registers, and every store is a whole 1 KB block.  A^T of the
// tile's columns is staged in LDS; B's rows are MFMA operands as they lie.  The merge is a copy with an update, its tiles
// taken along the rows of the original weights; NT stores bypass the caches.  Width and stores: launch_lora_merge_batch.
constexpr int kMergeRows = 64;

// Rows of the projection a merge computes (for [gate; up], the part's half of the packed rows).
__host__ __device__ inline int merge_rows(const MergeArgs& a) { return a.mode == kPackGateUp ? a.rows / 2 : a.rows; }

// Tile (rows kMergeRows rb .., columns COLS cb ..) of one merge.
template <int COLS, bool NT>
__device__ __forceinline__ void merge_tile(const MergeArgs& a, int rb, int cb) {
  constexpr int RB = kMergeRows / 64, CB = COLS / 32;              // 16-row blocks of a wave, 32-column blocks
  __shared__ __attribute__((aligned(16))) bf16_t at[COLS][72];  // A^T: [column][rank], padded rows
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int c0 = cb * COLS, nblk = min(COLS, a.K - c0) / 32;
  const int RK = (a.rank + 31) / 32 * 32;
  const bool gu = a.mode == kPackGateUp;
  const int nrows = merge_rows(a);
  // this lane's rows: packed row and source row (-1: a zero row), their original weights and B's rank columns 8 g ..
  int row[RB], src[RB];
  uint4 w0[RB][CB], bv[RB][2];
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int l = rb * kMergeRows + 16 * (wave + 4 * i) + r16;
    row[i] = gu ? 64 * (l >> 5) + 32 * a.part + (l & 31) : l;
    int part;
    src[i] = l < nrows ? pack_src_row(a.mode, row[i], a.head_dim, a.src_rows, part) : -1;
    if (l >= nrows) row[i] = -1;
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int col = c0 + 32 * c + 8 * g;
      w0[i][c] = make_uint4(0, 0, 0, 0);  // zero rows and columns of the packed layout
      if (src[i] >= 0 && col < a.src_cols)  // src_cols % 8 == 0: a chunk is wholly in or out
        w0[i][c] = *reinterpret_cast<const uint4*>(a.w0 + (size_t)src[i] * a.src_ld + col);
    }
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      const int k = 32 * kc + 8 * g;
      bv[i][kc] = make_uint4(0, 0, 0, 0);
      if (src[i] >= 0 && k < a.rank) bv[i][kc] = *reinterpret_cast<const uint4*>(a.b + (size_t)src[i] * a.rank + k);
    }
  }
  // A^T of the tile's columns, zero past the rank and past the source columns: 8 columns of one rank row per
  // 16-byte load
  for (int e = tid; e < RK * (COLS / 8); e += 256) {
    const int kr = e / (COLS / 8), c = 8 * (e % (COLS / 8));
    uint4 v = make_uint4(0, 0, 0, 0);
    if (kr < a.rank && c0 + c < a.src_cols) v = *reinterpret_cast<const uint4*>(a.a + (size_t)kr * a.src_cols + c0 + c);
    const uint32_t vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int x = 0; x < 8; ++x) at[c + x][kr] = (bf16_t)(vv[x >> 1] >> (16 * (x & 1)));
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    if (c >= nblk) break;
    bf16x8 av[2][2];  // [t][kc]
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int kc = 0; kc < 2; ++kc)
        if (kc < RK / 32)
          av[t][kc] = as_bf16x8(*reinterpret_cast<const uint4*>(&at[32 * c + 8 * (r16 >> 2) + 4 * t + (r16 & 3)][32 * kc + 8 * g]));
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      f32x4 acc[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kc = 0; kc < 2; ++kc)
          if (kc < RK / 32) acc[t] = mfma16(av[t][kc], as_bf16x8(bv[i][kc]), acc[t]);
      }
      if (row[i] < 0) continue;
      const int col = c0 + 32 * c + 8 * g;
      float w[8];
      unpack8(w0[i][c], w);
      if (src[i] >= 0 && col < a.src_cols) {
#pragma unroll
        for (int x = 0; x < 8; ++x) w[x] += a.scale * acc[x >> 2][x & 3];
      }
      const u32x4 ov = {pack2bf(w[0], w[1]), pack2bf(w[2], w[3]), pack2bf(w[4], w[5]), pack2bf(w[6], w[7])};
      u32x4* const dst = reinterpret_cast<u32x4*>(a.dst + frag_index(row[i], col, a.K));
      if constexpr (NT) __builtin_nontemporal_store(ov, dst);
      else *dst = ov;
    }
  }
}

// One workgroup per tile of each item, the items' tiles one after the other, along the rows of the original weights.
template <int COLS, bool NT>
__global__ __launch_bounds__(256) void lora_merge_kernel(MergeBatch b) {
  int i = 0;
  while (i + 1 < b.n && (int)blockIdx.x >= b.wg0[i + 1]) ++i;
  const MergeArgs& a = b.item[i];
  const int local = (int)blockIdx.x - b.wg0[i];
  const int ncb = (a.K + COLS - 1) / COLS;
  merge_tile<COLS, NT>(a, local / ncb, local % ncb);
}

static bool merge_ok(const MergeArgs& a) {
  return a.K % 64 == 0 && a.rank >= 8 && a.rank <= 64 && a.rank % 8 == 0 && a.src_ld % 8 == 0 && a.src_cols % 8 == 0 &&
         (a.mode != kPackGateUp || (a.part >= 0 && a.part <= 1 && a.rows % 64 == 0));
}

// Sets the first workgroup of each item for tiles of COLS columns; returns the launch's workgroups.
static int merge_tiles(MergeBatch& b, int cols) {
  int wg = 0;
  for (int i = 0; i < b.n; ++i) {
    b.wg0[i] = wg;
    wg += (merge_rows(b.item[i]) + kMergeRows - 1) / kMergeRows * ((b.item[i].K + cols - 1) / cols);
  }
  return b.wg0[b.n] = wg;
}

// The stores go past the caches where the merged weights and the original ones together do not fit the last-level cache
// (`stream`, decided for the whole model: see vla_create).  A merge of one layer and a prefill of one environment, past the
// caches / through them: d = 2560 (157 MB) 202 / 218 us, d = 4096 424 / 445; d = 2048 (101 MB) 145 / 139, d = 1536 112 / 110.
// The merge of the 7B layer at rank 32 (810 MB) takes 158 us so = 5.1 TB/s, what a plain copy reaches.
//
// 128 columns instead of 64 (with such stores, us, 128 / 64):
// - up to rank 32; above, a workgroup's staging of A^T costs more than the longer pieces of rows save (rank 64: d = 4096
//   205 / 207, d = 3072 117 / 84, d = 1024 20 / 15);
// - from 4096 workgroups on, or from 1024 on where the rows of an original weight are a multiple of 2 KB: there the 128 bytes
//   of consecutive rows that 64 columns take presumably lie on few memory channels.  Merge of all layers and a prefill at rank 8:
//   d = 4096, two layers 786 / 803, d = 3072 517 / 531, d = 1024, eight layers 647 / 662, but d = 1280 803 / 792.  Too few
//   workgroups (the projections of d = 1024 one by one): 906 / 826.
// Before, every merge ran 64 columns down the rows through an LDS tile with cached stores: d = 256 4.9 us (now 4.3), 1024
// 13.5 (12.3), 2048 39 (35), 4096 180 (154) at rank 8.
constexpr int kMergeWide = 4096, kMergeWideEven = 1024;
hipError_t launch_lora_merge_batch(MergeBatch b, hipStream_t s) {
  if (b.n < 1 || b.n > kMergeBatchMax) return hipErrorInvalidValue;
  int rank = 0;
  bool even = false;
  for (int i = 0; i < b.n; ++i) {
    if (b.item[i].rows < 0 || !merge_ok(b.item[i])) return hipErrorInvalidValue;
    rank = std::max(rank, b.item[i].rank);
    even |= b.item[i].src_ld % 1024 == 0;
  }
  if (b.stream && rank <= 32) {
    const int wg = merge_tiles(b, 128);
    if (wg >= (even ? kMergeWideEven : kMergeWide)) {
      hipLaunchKernelGGL((lora_merge_kernel<128, true>), dim3(wg), dim3(256), 0, s, b);
      return hipGetLastError();
    }
  }
  const int wg = merge_tiles(b, 64);
  if (wg == 0) return hipSuccess;
  if (b.stream) hipLaunchKernelGGL((lora_merge_kernel<64, true>), dim3(wg), dim3(256), 0, s, b);
  else hipLaunchKernelGGL((lora_merge_kernel<64, false>), dim3(wg), dim3(256), 0, s, b);
  return hipGetLastError();
}

hipError_t launch_lora_merge(const MergeArgs& a, bool stream, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  MergeBatch b{};
  b.item[0] = a;
  b.n = 1;
  b.stream = stream;
  return launch_lora_merge_batch(b, s);
}

// One wave per row: 16-byte chunks of 8 consecutive K elements (contiguous in
// frag layout), lane l taking chunks l, l + 64, ..., then a butterfly sum.
__global__ __launch_bounds__(256) void value_head_kernel(const bf16_t* __restrict__ u, int R, int d,
                                                         const bf16_t* __restrict__ head, float* __restrict__ values) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= R) return;
  float acc = 0.f;
  for (int c = lane; c < d / 8; c += 64) {
    float uf[8], hf[8];
    unpack8(*reinterpret_cast<const uint4*>(u + frag_index(r, 8 * c, d)), uf);
    unpack8(*reinterpret_cast<const uint4*>(head + 8 * c), hf);
#pragma unroll
    for (int x = 0; x < 8; ++x) acc += uf[x] * hf[x];
  }
  acc = wave_sum(acc);
  if (lane == 0) values[r] = acc;
}

hipError_t launch_value_head(const bf16_t* u, int R, int d, const bf16_t* head, float* values, hipStream_t s) {
  if (R <= 0) return hipSuccess;
  if (d % 8 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(value_head_kernel, dim3((R + 3) / 4), dim3(256), 0, s, u, R, d, head, values);
  return hipGetLastError();
}

hipError_t launch_pack_frag(const PackArgs& a, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  if (a.K % 32 != 0 || a.src_cols > a.K || !a.dst || !a.src || (a.mode == kPackGateUp && !a.src2))
    return hipErrorInvalidValue;
  const size_t n = (size_t)a.rows * (a.K / 8);
  hipLaunchKernelGGL(pack_frag_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bf16_to_f32(float* dst, const bf16_t* src, int n, hipStream_t s) {
  hipLaunchKernelGGL(bf16_to_f32_kernel, dim3((n + 255) / 256), dim3(256), 0, s, dst, src, n);
  return hipGetLastError();
}

hipError_t launch_extract_actions(const int32_t* tokens, int n, int n_dims, int action_begin, int bins,
                                  const float* lo, const float* hi, float* actions, hipStream_t s) {
  const int n_elems = n * n_dims;
  if (n_elems <= 0) return hipSuccess;
  hipLaunchKernelGGL(extract_actions_kernel, dim3((n_elems + 255) / 256), dim3(256), 0, s, tokens, n_elems, n_dims,
                     action_begin, bins, lo, hi, actions);
  return hipGetLastError();
}

hipError_t launch_gather_rows(const float* x, const bf16_t* o, const int32_t* rows, int R, int d, float* xc,
                              bf16_t* oc, hipStream_t s) {
  if (R <= 0) return hipSuccess;
  if (d % 8 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gather_rows_kernel, dim3(R), dim3(256), 0, s, x, o, rows, d, xc, oc);
  return hipGetLastError();
}

hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  // The runtime's copy below 8 MB: it writes through the caches (0.1 to 2 MB 2.0-2.2 us, copy_kernel 3.6-4.4).  The four
  // packed weights of a layer read back, runtime / kernel: d = 1536 (4.7 to 26 MB) 26.9 / 27.2 us, d = 2560 (13 to 71 MB)
  // 69 / 50, d = 4096 (34 to 182 MB) 157 / 144.
  if (bytes < (8u << 20) || ((uintptr_t)dst | (uintptr_t)src | bytes) % 16 != 0)
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, s);
  const size_t n16 = bytes / 16;
  hipLaunchKernelGGL(copy_kernel, dim3((unsigned)((n16 + 1023) / 1024)), dim3(256), 0, s, static_cast<const u32x4*>(src),
                     static_cast<u32x4*>(dst), n16);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* dst, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  if (bytes % 16 != 0) return hipErrorInvalidValue;
  const size_t n16 = bytes / 16;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, reinterpret_cast<uint4*>(dst), n16);
  return hipGetLastError();
}

}  // namespace vla
