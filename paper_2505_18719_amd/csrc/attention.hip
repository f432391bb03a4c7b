// Causal attention over the paged KV cache on gfx950.
//
// Prefill: one 512-thread workgroup per (environment, head); the head's whole
// K and V^T are copied into LDS once, then 16-query tiles are dealt to the 8
// waves.  Scores are computed transposed so that P stays in registers in the
// layout the P*V MFMA consumes, and a whole score row (<= 320 keys, the
// longest sequence of one environment) stays in registers, so the softmax is
// exact.
//
// Decode: one workgroup per (environment, head) and one query; scores and
// P*V in fp32 on the vector ALUs, streaming K rows and transposed V pages with
// 16-byte loads.
#include "common.h"
#include "embed_dev.h"
#include "kernels.h"

namespace vla {

namespace {

// Prefill attention: one 512-thread workgroup (8 waves) per (environment,
// head).  The environment's whole K (key rows) and V^T (feature rows) for
// this head, <= 320 keys, are copied once into LDS with buffer_load ... lds
// (80 KB each at head_dim 128), then every wave takes 16-query tiles of the
// causal triangle in a balanced order.  Per tile, scores are computed
// transposed, S^T = K Q^T, with the keys of each 32-key chunk assigned to MFMA
// rows so that lane group g ends up holding keys 8g .. 8g+7 of the chunk for
// its query: exactly the B-operand fragment of P^T in O^T = V^T P^T.  P never
// leaves registers and enters the MFMA as P_hi + P_lo (two bf16 products,
// ~16 significant bits).  The whole score row (<= 320 keys) is kept, so the
// softmax is exact (true maximum, no online rescaling).
//
// LDS layouts (both conflict-free for the 16-byte operand reads, no padding):
//  K: row R holds key kperm(R), with the 32 keys of a chunk ordered as the
//     MFMA rows of its two 16-key tiles; 16-byte feature chunk j of row R is
//     stored at slot j ^ kswz(R).
//  V^T: the cache's own page layout, one 16-key page after the other (feature
//     f of a page: 16 keys, two 16-byte halves); half h of feature f is stored
//     at 16-byte unit 2f + (h ^ ((f >> 3) & 1)) of its page.
constexpr int kMaxKeys = 320;
constexpr int kMaxChunks = kMaxKeys / 32;
constexpr int kMaxPages = kMaxKeys / kPage;

// key held by LDS row R of K: MFMA row i of 16-key tile t of chunk c is key 32c + 8(i/4) + 4t + i%4
__device__ __forceinline__ int kperm(int R) {
  const int i = R & 15, t = (R >> 4) & 1, c = R >> 5;
  return 32 * c + 8 * (i >> 2) + 4 * t + (i & 3);
}
template <int HD>
__device__ __forceinline__ int kswz(int R) {
  return HD == 128 ? (R & 15) : ((R >> 1) & 7);
}

// One 16-query tile (queries 16 qt .. 16 qt + 15 of the environment) whose
// keys span NC 32-key chunks; only the last chunk holds keys that some query
// of the tile must not see (ncq = qt / 2 + 1 for every tile of a sequence).
// Straight-line code for a compile-time chunk count, so the scheduler can
// overlap the LDS reads of one chunk with the MFMAs of another.
template <int HD, int NC>
__device__ __forceinline__ void attn_tile(const PrefillAttnArgs& a, const char* klds, const char* vlds, int qt, int L,
                                          int row0, int head, int lane) {
  constexpr int KROW = HD * 2, VPAGE = HD * kPage * 2;
  constexpr int KS = HD / 32, NB = HD / 16;
  const int r16 = lane & 15, g = lane >> 4;
  const int qpos = qt * 16 + r16;
  uint4 qf[KS];  // B operand: query qpos, features 32 ks + 8g .. +8
  {
    const bf16_t* qp = a.q + (size_t)(row0 + min(qpos, L - 1)) * a.d + head * HD + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const uint4*>(qp + ks * 32);
  }
  // scores: lane holds S(query qpos, key 32c + 8g + 4t + r) in sc[2c + t][r]
  f32x4 sc[2 * NC];
#pragma unroll
  for (int t = 0; t < 2 * NC; ++t) sc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
    for (int ct = 0; ct < 2 * NC; ++ct) {
      // LDS row 16 ct + r16 (chunk ct / 2, tile ct % 2); its swizzle is kswz<HD>(r16)
      const char* kr = klds + (16 * ct + r16) * KROW + 16 * ((4 * ks + g) ^ kswz<HD>(r16));
      sc[ct] = mfma16(as_bf16x8(*reinterpret_cast<const uint4*>(kr)), as_bf16x8(qf[ks]), sc[ct]);
    }
  }
  const int klim = min(qpos, L - 1);  // last key this lane's query sees
  float mx = -INFINITY;
#pragma unroll
  for (int ct = 0; ct < 2 * NC; ++ct)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float v = sc[ct][r] * a.scale;
      if (ct >= 2 * NC - 2) {
        const int key = 32 * (ct >> 1) + 8 * g + 4 * (ct & 1) + r;
        v = key <= klim ? v : -INFINITY;
      }
      sc[ct][r] = v;
      mx = fmaxf(mx, v);
    }
  mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
  mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
  float sum = 0.f;
#pragma unroll
  for (int ct = 0; ct < 2 * NC; ++ct)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float pv = expf(sc[ct][r] - mx);  // masked: expf(-inf) = 0
      sc[ct][r] = pv;
      sum += pv;
    }
  sum += __shfl_xor(sum, 16, kWave);
  sum += __shfl_xor(sum, 32, kWave);
  if (a.lse && g == 0 && qpos < L) a.lse[((size_t)(row0 + qpos) * a.n_heads + head) * 2] = mx + logf(sum);

  // O^T = V^T P^T: A operand = V^T rows (feature nb*16 + r16), keys 32c + 8g .. +8,
  // i.e. page 2c + g/2, half g%2; (f >> 3) & 1 of feature 16nb + r16 is r16 >> 3
  f32x4 o[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) o[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const char* vp0 = vlds + (g >> 1) * VPAGE + 16 * (2 * r16 + ((g & 1) ^ (r16 >> 3)));
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    bf16x8 phi, plo;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float pv = sc[2 * c + t][r];
        const __bf16 h = (__bf16)pv;
        phi[4 * t + r] = h;
        plo[4 * t + r] = (__bf16)(pv - (float)h);
      }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const uint4 vv = *reinterpret_cast<const uint4*>(vp0 + 2 * c * VPAGE + nb * 16 * 32);
      o[nb] = mfma16(as_bf16x8(vv), phi, o[nb]);
      o[nb] = mfma16(as_bf16x8(vv), plo, o[nb]);
    }
  }
  // o[nb][r] = O(query qpos, feature nb*16 + 4g + r)
  if (qpos < L) {
    const float inv = 1.f / sum;
    // frag layout (the O projection's A operand): 4 consecutive features stay contiguous
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      *reinterpret_cast<uint2*>(a.o + frag_index(row0 + qpos, head * HD + nb * 16 + 4 * g, a.d)) =
          make_uint2(pack2bf(o[nb][0] * inv, o[nb][1] * inv), pack2bf(o[nb][2] * inv, o[nb][3] * inv));
  }
}

// Tiles qt_lo .. qt_hi - 1, most expensive first, dealt to the 8 waves in snake order.
template <int HD>
__device__ __forceinline__ void attn_tiles(const PrefillAttnArgs& a, const char* klds, const char* vlds, int qt_lo,
                                           int qt_hi, int L, int row0, int head, int wave, int lane) {
  const int n = qt_hi - qt_lo;
  for (int p0 = 0; p0 < n; p0 += 8) {
    const int p = p0 + (((p0 >> 3) & 1) ? 7 - wave : wave);
    if (p >= n) continue;
    const int qt = qt_hi - 1 - p;
    switch (qt / 2 + 1) {  // live 32-key chunks
      case 1: attn_tile<HD, 1>(a, klds, vlds, qt, L, row0, head, lane); break;
      case 2: attn_tile<HD, 2>(a, klds, vlds, qt, L, row0, head, lane); break;
      case 3: attn_tile<HD, 3>(a, klds, vlds, qt, L, row0, head, lane); break;
      case 4: attn_tile<HD, 4>(a, klds, vlds, qt, L, row0, head, lane); break;
      case 5: attn_tile<HD, 5>(a, klds, vlds, qt, L, row0, head, lane); break;
      case 6: attn_tile<HD, 6>(a, klds, vlds, qt, L, row0, head, lane); break;
      case 7: attn_tile<HD, 7>(a, klds, vlds, qt, L, row0, head, lane); break;
      case 8: attn_tile<HD, 8>(a, klds, vlds, qt, L, row0, head, lane); break;
      case 9: attn_tile<HD, 9>(a, klds, vlds, qt, L, row0, head, lane); break;
      default: attn_tile<HD, 10>(a, klds, vlds, qt, L, row0, head, lane); break;
    }
  }
}

template <int HD>
__global__ __launch_bounds__(512, 1) void attn_prefill_kernel(PrefillAttnArgs a) {
  constexpr int KROW = HD * 2;           // bytes per K row
  constexpr int KCH = HD / 8;            // 16-byte chunks per K row
  constexpr int VPAGE = HD * kPage * 2;  // bytes per V^T page
  __shared__ __attribute__((aligned(1024))) char lds[kMaxKeys * KROW + kMaxPages * VPAGE];
  char* const klds = lds;
  char* const vlds = lds + kMaxKeys * KROW;
  const int env = blockIdx.x, head = blockIdx.y;
  const int L = a.env_len[env], row0 = a.env_row0[env];
  const int H = a.n_heads;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nch = (L + 31) / 32;
  const int32_t* pt = a.page_table + env * a.max_pages;
  const int last_page = a.max_pages - 1;

  // ---- copy the K rows and V^T pages of the nch chunks into LDS, chunk by
  // chunk: copy i moves 1 KB of chunk i / CP (K rows first, then V^T pages);
  // wave w issues copies w, w + 8, ..., i.e. CP / 8 per chunk
  constexpr int KC = 32 * KROW / 1024, VC = 2 * VPAGE / 1024, CP = KC + VC;
  constexpr int KROWS_PER_KB = 1024 / KROW;
  static_assert(CP % 8 == 0, "copies per chunk must divide among the 8 waves");
  {
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)a.kv.k, (short)0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)a.kv.v, (short)0, 0x7fffffff, 0x00020000);
    const uint32_t kbase = (uint32_t)(uintptr_t)((lds_ptr_t*)klds), vbase = (uint32_t)(uintptr_t)((lds_ptr_t*)vlds);
    // the environment's page table, one entry per lane, read once: a copy must
    // not wait on a load of its own (the wait would also drain every copy
    // issued before it)
    int ptv = pt[min(lane, last_page)];
    // the copies below use ptv; passing it through an empty asm ends the load's
    // lifetime here, so the compiler waits for it once and not before each copy
    asm volatile("" : "+v"(ptv));
    for (int i = wave; i < CP * nch; i += 8) {
      const int c = i / CP, sub = i % CP;
      if (sub < KC) {
        const int kcopy = c * KC + sub;  // 1 KB of K rows, all in one 16-key page
        const int R = kcopy * KROWS_PER_KB + lane / KCH, slot = lane % KCH;
        const int key = kperm(R);
        const int page = __builtin_amdgcn_readlane(ptv, min(kperm(kcopy * KROWS_PER_KB) / kPage, last_page));
        const uint32_t off = (uint32_t)((((page * H + head) * kPage + key % kPage) * HD + 8 * (slot ^ kswz<HD>(R))) * 2);
        lds_dma16(kbase + kcopy * 1024, off, rk, 0);
      } else {
        const int vcopy = c * VC + (sub - KC);  // 1 KB of V^T pages
        const int pg = vcopy / (VPAGE / 1024);
        const int unit = (vcopy % (VPAGE / 1024)) * 64 + lane;  // 16-byte unit of the page
        const int f = unit >> 1, h = (unit & 1) ^ ((f >> 3) & 1);
        const int page = __builtin_amdgcn_readlane(ptv, min(pg, last_page));
        const uint32_t off = (uint32_t)((((page * H + head) * HD + f) * kPage + 8 * h) * 2);
        lds_dma16(vbase + vcopy * 1024, off, rv, 0);
      }
    }
  }
  // phase 1: the tiles whose keys lie in the first h1 chunks start as soon as
  // those chunks have landed, while the rest are still being copied
  const int h1 = min(nch, kMaxChunks / 2);
  const int nq = (L + 15) / 16;
  const int q1 = min(nq, 2 * h1);  // tiles 0 .. q1-1 need chunks < h1
  switch ((nch - h1) * (CP / 8)) {  // this wave's copies of the later chunks may stay in flight
    case 0: WAIT_VMCNT(0); break;
    case 1: WAIT_VMCNT(1); break;
    case 2: WAIT_VMCNT(2); break;
    case 3: WAIT_VMCNT(3); break;
    case 4: WAIT_VMCNT(4); break;
    case 5: WAIT_VMCNT(5); break;
    case 6: WAIT_VMCNT(6); break;
    case 7: WAIT_VMCNT(7); break;
    case 8: WAIT_VMCNT(8); break;
    case 9: WAIT_VMCNT(9); break;
    default: WAIT_VMCNT(10); break;
  }
  __syncthreads();
  // query tiles below the first needed row are skipped (their keys are still loaded: later rows see them)
  const int qlo = a.env_q0 ? min(max(a.env_q0[env], 0), L - 1) / 16 : 0;
  if (qlo < q1) attn_tiles<HD>(a, klds, vlds, qlo, q1, L, row0, head, wave, lane);
  if (q1 < nq) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    attn_tiles<HD>(a, klds, vlds, max(qlo, q1), nq, L, row0, head, wave, lane);
  }
}

// One 256-thread workgroup per (environment, head).  Scores: HD / 8 lanes per key row, KPP keys a pass.  P V: thread
// (feature, group of pages).
//
// The work is 150 KB of reads and almost no arithmetic.  With few workgroups what counts is that the reads do not wait on
// each other: KP passes of K rows and VP pages of V go into registers before the token's own q, k, v have been summed
// from the QKV projection's partials (all of a sequence with KP = NK, VP = NV), the rest KC passes and VC pages at a time.
// With many, the workgroups of a CU cover each other's waits, and registers that limit their number cost more (the rule
// is in launch_attn_decode).
// The order of every sum depends on the sequence length alone.
template <int HD>
struct DecodeShape {
  static constexpr int LPK = HD / 8;                  // lanes per key row
  static constexpr int KPP = 256 / LPK;               // keys per pass
  static constexpr int G = 256 / HD;                  // page groups in P*V
  static constexpr int NK = kMaxKeys / KPP, NV = kMaxPages / G;
};

// Sum over the LPK lanes of a key row: xor 8 (16 lanes), 4, 2, 1.
template <int LPK>
__device__ __forceinline__ float key_sum(float v) {
  if constexpr (LPK == 16) return row_sum16(v);
  v += dpp_mov<0x114, 0xA>(dpp_mov<0x104, 0x5>(v, v), v);  // xor 4: row_shl 4 into even banks, row_shr 4 into odd ones
  v += dpp_mov<0x4E>(v, v);                                // quad_perm 2 3 0 1
  return v + dpp_mov<0xB1>(v, v);                          // quad_perm 1 0 3 2
}

template <int HD, int KP, int VP, int KC, int VC>
__global__ __launch_bounds__(256) void attn_decode_kernel(DecodeAttnArgs a) {
  using S = DecodeShape<HD>;
  constexpr int LPK = S::LPK, KPP = S::KPP, G = S::G, HALF = HD / 2;
  __shared__ __attribute__((aligned(16))) float sc[kMaxKeys];
  __shared__ __attribute__((aligned(16))) bf16_t q16[HD], k16[HD];  // this token's rotated q and k
  __shared__ float vn[HD];                                           // and its v (a bf16 value)
  __shared__ float red[2][4];
  __shared__ float op[G][HD];
  const int head = blockIdx.x, b = blockIdx.y;
  const int H = a.n_heads, tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pos = a.env_prefix[b] + a.step - 1;  // this step's token; the keys are 0 .. pos
  const int n = pos + 1, last = pos / kPage;
  const int32_t* pt = a.page_table + b * a.max_pages;

  // ---- q, k, v of the token for this head: one thread per rotary pair of
  // q and k (columns permuted per head as for the prefill GEMM's epilogue:
  // pair (32 blk + c, HALF + 32 blk + c) sits in columns 64 blk + c and
  // 64 blk + c + 32 of the head) and per pair of v features (e, e + HALF).
  // Their partials are loaded ahead of the pages.
  const bool qkv = tid < 3 * HALF;
  const int region = tid / HALF, e = tid % HALF, N = 3 * a.d;
  float p1[kSlotsAhead], p2[kSlotsAhead];
  float2 cs = make_float2(1.f, 0.f);
  const float *c1 = nullptr, *c2 = nullptr;
  int ns1 = 0, ns2 = 0;
  const size_t stride = (size_t)a.B * N;
  if (qkv) {
    const int col1 = region * a.d + head * HD + (region < 2 ? 64 * (e / 32) + e % 32 : e);
    const int col2 = col1 + (region < 2 ? 32 : HALF);
    ns1 = skinny_slots(a.plan, col1 >> 6);
    ns2 = skinny_slots(a.plan, col2 >> 6);
    c1 = a.part + (size_t)b * N + col1;
    c2 = a.part + (size_t)b * N + col2;
#pragma unroll
    for (int s = 0; s < kSlotsAhead; ++s) {
      if (s < ns1) p1[s] = c1[s * stride];
      if (s < ns2) p2[s] = c2[s * stride];
    }
    if (region < 2) cs = a.rope[pos * HALF + e];
  }

  // ---- the pages (past the last one, it again: nothing of those is used); a wave's keys of a pass lie in one page
  const int key0 = tid / LPK, part = tid % LPK;
  const int i = tid % HD, grp = __builtin_amdgcn_readfirstlane(tid / HD);
  auto k_row = [&](int it) {  // this lane's 8 features of key KPP it + key0
    // with many workgroups memory bounds it, and the keys past the sequence in its last page are not read
    if (KP == 0 && KPP * it + key0 >= pos) return make_uint4(0, 0, 0, 0);
    const int page = pt[min(KPP / kPage * it + wave * (64 / LPK) / kPage, last)];
    return *reinterpret_cast<const uint4*>(a.kv.k + (((size_t)page * H + head) * kPage + key0 % kPage) * HD + part * 8);
  };
  auto v_page = [&](int it, uint4 (&v)[2]) {  // the 16 keys of page grp + G it for feature i
    const uint4* vp = reinterpret_cast<const uint4*>(a.kv.v + (((size_t)pt[min(grp + G * it, last)] * H + head) * HD + i) * kPage);
    v[0] = vp[0];
    v[1] = vp[1];
  };
  uint4 kf[KP > 0 ? KP : 1], vf[VP > 0 ? VP : 1][2];
#pragma unroll
  for (int it = 0; it < KP; ++it) kf[it] = k_row(it);
#pragma unroll
  for (int it = 0; it < VP; ++it) v_page(it, vf[it]);
  __builtin_amdgcn_sched_barrier(0);  // the loads above go out before the first wait

  if (qkv) {
    float x1 = 0.f, x2 = 0.f;  // as skinny_sum: slots added in order
#pragma unroll
    for (int s = 0; s < kSlotsAhead; ++s) {
      if (s < ns1) x1 += p1[s];
      if (s < ns2) x2 += p2[s];
    }
    for (int s = kSlotsAhead; s < ns1; ++s) x1 += c1[s * stride];
    for (int s = kSlotsAhead; s < ns2; ++s) x2 += c2[s * stride];
    const size_t at = (size_t)pt[last] * H + head;
    const int slot = pos % kPage;
    if (region == 2) {
      const bf16_t v1 = f2bf(x1), v2 = f2bf(x2);
      bf16_t* vb = a.kv.v + at * HD * kPage + slot;
      vb[(size_t)e * kPage] = v1;
      vb[(size_t)(e + HALF) * kPage] = v2;
      vn[e] = bf2f(v1);
      vn[e + HALF] = bf2f(v2);
    } else {
      // the fused multiply-adds of the prefill GEMM's epilogue
      const bf16_t r1 = f2bf(fmaf(x1, cs.x, -(x2 * cs.y))), r2 = f2bf(fmaf(x2, cs.x, x1 * cs.y));
      bf16_t* t16 = region == 0 ? q16 : k16;
      t16[e] = r1;
      t16[e + HALF] = r2;
      if (region == 1) {
        bf16_t* kr = a.kv.k + (at * kPage + slot) * HD;
        kr[e] = r1;
        kr[e + HALF] = r2;
      }
    }
  }
  __syncthreads();

  // ---- scores: one key row per LPK lanes
  float qv[8];
  unpack8(*reinterpret_cast<const uint4*>(q16 + part * 8), qv);
  auto score = [&](int it, uint4 kr) {
    const int key = KPP * it + key0;
    if (KPP * (it + 1) > pos && key == pos) kr = *reinterpret_cast<const uint4*>(k16 + part * 8);  // this step's token
    float kv8[8];
    unpack8(kr, kv8);
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) acc += qv[j] * kv8[j];
    acc = key_sum<LPK>(acc);
    if (part == 0 && key < n) sc[key] = acc * a.scale;
  };
#pragma unroll
  for (int it = 0; it < KP; ++it)
    if (KPP * it < n) score(it, kf[it]);
  for (int it = KP; KPP * it < n; it += KC) {
    uint4 kc[KC];
#pragma unroll
    for (int u = 0; u < KC; ++u) kc[u] = k_row(it + u);
#pragma unroll
    for (int u = 0; u < KC; ++u)
      if (KPP * (it + u) < n) score(it + u, kc[u]);
  }
  __syncthreads();

  float m = -INFINITY;
  for (int t = tid; t < n; t += 256) m = fmaxf(m, sc[t]);
  m = wave_max(m);
  if ((tid & 63) == 0) red[0][wave] = m;
  __syncthreads();
  m = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
  float s = 0.f;
  for (int t = tid; t < n; t += 256) {
    const float p = expf(sc[t] - m);
    sc[t] = p;
    s += p;
  }
  s = wave_sum(s);
  if ((tid & 63) == 0) red[1][wave] = s;
  __syncthreads();
  s = red[1][0] + red[1][1] + red[1][2] + red[1][3];

  const float vnew = vn[i];
  float acc = 0.f;
  auto pv = [&](int it, const uint4 (&v)[2]) {
    const int pg = grp + G * it;
    float v16[16], p16[16];
    unpack8(v[0], v16);
    unpack8(v[1], v16 + 8);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float4 p = *reinterpret_cast<const float4*>(sc + pg * kPage + 4 * j);
      p16[4 * j] = p.x; p16[4 * j + 1] = p.y; p16[4 * j + 2] = p.z; p16[4 * j + 3] = p.w;
    }
    if (pg < last) {
#pragma unroll
      for (int j = 0; j < kPage; ++j) acc += p16[j] * v16[j];
    } else {  // the token's v from LDS; slots past it hold no key
#pragma unroll
      for (int j = 0; j < kPage; ++j)
        if (pg * kPage + j <= pos) acc += p16[j] * (pg * kPage + j == pos ? vnew : v16[j]);
    }
  };
#pragma unroll
  for (int it = 0; it < VP; ++it)
    if (grp + G * it <= last) pv(it, vf[it]);
  for (int it = VP; grp + G * it <= last; it += VC) {
    uint4 vc[VC][2];
#pragma unroll
    for (int u = 0; u < VC; ++u) v_page(it + u, vc[u]);
#pragma unroll
    for (int u = 0; u < VC; ++u)
      if (grp + G * (it + u) <= last) pv(it + u, vc[u]);
  }
  op[grp][i] = acc;
  __syncthreads();
  if (grp == 0) {
    float t = 0.f;
#pragma unroll
    for (int gg = 0; gg < G; ++gg) t += op[gg][i];
    a.o[frag_index(b, head * HD + i, a.d)] = f2bf(t / s);  // frag layout: A operand of the O projection
  }
}

// ------------------------------------------------------------------ sampler
// One wave per row over A <= 256 bins (4 per lane).  Gumbel-max: the sampled
// bin maximises z/T + g (lowest bin on exact ties); log-probability and
// entropy are those of softmax(z/T).
// Row `row` by one wave; returns the scored bin.  `write`: this wave stores the outputs.
__device__ __forceinline__ int sample_row(const SamplerArgs& a, int row, int lane, bool write) {
  float zv[4], zt[4], gm[4];
  float m = -INFINITY;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int j = lane + 64 * t;
    if (a.gumbel) gm[t] = j < a.A ? a.gumbel[((size_t)row * a.n_actions + a.step) * a.A + j] : 0.f;
    zv[t] = 0.f;
    if (j < a.A) zv[t] = a.z ? a.z[(size_t)row * a.A + j] : skinny_sum(a.part, a.plan, a.rows, a.plan.tiles * 64, row, j);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    zt[t] = lane + 64 * t < a.A ? zv[t] / a.temperature : -INFINITY;
    m = fmaxf(m, zt[t]);
  }
  m = wave_max(m);
  float se = 0.f, sz = 0.f;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    if (lane + 64 * t < a.A) {
      const float e = expf(zt[t] - m);
      se += e;
      sz += e * (zt[t] - m);
    }
  }
  se = wave_sum(se);
  sz = wave_sum(sz);
  const float lse = m + logf(se);
  const float ent = logf(se) - sz / se;

  int out;    // index into [B, n_actions] outputs
  int kbin;   // scored bin
  if (a.gumbel) {
    const int b = row, i = a.step;
    float best = -INFINITY;
    int bi = 0x7fffffff;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int j = lane + 64 * t;
      if (j < a.A) {
        float s = zt[t] + gm[t];
        if (s != s) s = -INFINITY;
        if (s > best || (s == best && j < bi)) { best = s; bi = j; }
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float ob = __shfl_xor(best, o, kWave);
      const int oi = __shfl_xor(bi, o, kWave);
      if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
    }
    if (bi >= a.A) bi = 0;  // every score was NaN
    kbin = bi;
    out = b * a.n_actions + i;
    if (write && lane == 0) {
      a.tokens[out] = a.action_begin + kbin;
      a.next_tok[b] = a.action_begin + kbin;
    }
  } else {
    out = row;
    kbin = a.given[row] - a.action_begin;
    if (kbin < 0 || kbin >= a.A) {
      if (write && lane == 0) atomicOr(a.flags, 2u);
      kbin = -1;
    }
  }
  // z/T at the chosen bin, read from the lane that holds it
  const int src_lane = kbin < 0 ? 0 : (kbin & 63), src_t = kbin < 0 ? 0 : (kbin >> 6);
  float mine = zt[0];
#pragma unroll
  for (int t = 1; t < 4; ++t)
    if (t == src_t) mine = zt[t];
  const float ztk = __shfl(mine, src_lane, kWave);
  if (write && lane == 0) {
    a.logp[out] = kbin < 0 ? __builtin_nanf("") : ztk - lse;
    if (a.entropy) a.entropy[out] = ent;
  }
  if (write && a.logits_out) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int j = lane + 64 * t;
      if (j < a.A) a.logits_out[(size_t)out * a.A + j] = zv[t];
    }
  }
  return kbin;
}

__global__ __launch_bounds__(256) void sampler_kernel(SamplerArgs a) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row < a.rows) sample_row(a, row, threadIdx.x & 63, true);
}

// One workgroup per row: every wave samples the row's token, then all of them write the next step's input from it.
// (Head sum, sampler and embedding were three launches at a decode step: 9 us at d = 256, 17 us at d = 4096, now 6.3 and 10.7.)
__global__ __launch_bounds__(256) void sampler_embed_kernel(SamplerArgs a, EmbedTokenArgs e) {
  __shared__ float sh[4];
  const int kbin = sample_row(a, blockIdx.x, threadIdx.x & 63, threadIdx.x < 64);
  embed_token_row(e, a.action_begin + kbin, blockIdx.x, sh);
}

}  // namespace

hipError_t launch_attn_prefill(const PrefillAttnArgs& a, hipStream_t s) {
  if (a.n_env <= 0) return hipSuccess;
  const dim3 grid(a.n_env, a.n_heads), block(512);
  if (a.head_dim == 128) hipLaunchKernelGGL(attn_prefill_kernel<128>, grid, block, 0, s, a);
  else if (a.head_dim == 64) hipLaunchKernelGGL(attn_prefill_kernel<64>, grid, block, 0, s, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

namespace {
template <int HD, int KP, int VP, int KC, int VC>
void launch_decode(const DecodeAttnArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((attn_decode_kernel<HD, KP, VP, KC, VC>), dim3(a.n_heads, a.B), dim3(256), 0, s, a);
}
}  // namespace

hipError_t launch_attn_decode(const DecodeAttnArgs& a, hipStream_t s) {
  if (a.B <= 0) return hipSuccess;
  if (a.max_pages < 1 || a.max_pages > kMaxPages) return hipErrorInvalidValue;
  if (a.head_dim != 128 && a.head_dim != 64) return hipErrorInvalidValue;
  // By workgroups per CU, which is what covers a workgroup's waits (us, all of a sequence ahead / 4 passes and 2 pages
  // at a time / one by one; a workgroup that looked up its pages in LDS and read one by one before): head_dim 128, at
  // most one per CU 11.1 / 14.9 / 19.9 (28.0), 2 22.2 / 19.7 / 25.6, 4 42.4 / 32.7 / 34.6, 8 75 / 69.7 / 60.7 (59.0), and
  // without the last page's keys past the sequence 58.6 (58.5), 12 91.8 (94.2), 14 104.6 (105.2), 16 124.7 (122);
  // head_dim 64, one 8.9 / 10.9 / 11.8 (19.2), 4 19.7 / 17.5 / 17.2, 8 41.9 / 37.4 / 32.7.
  const long long wgs = (long long)a.B * a.n_heads;
  const bool few = wgs <= a.cus, some = wgs <= 4ll * a.cus;
  if (a.head_dim == 128) {
    if (few) launch_decode<128, DecodeShape<128>::NK, DecodeShape<128>::NV, 1, 1>(a, s);
    else if (some) launch_decode<128, 0, 0, 4, 2>(a, s);
    else launch_decode<128, 0, 0, 1, 1>(a, s);
  } else {
    if (few) launch_decode<64, DecodeShape<64>::NK, DecodeShape<64>::NV, 1, 1>(a, s);
    else if (some) launch_decode<64, 0, 0, 4, 2>(a, s);
    else launch_decode<64, 0, 0, 1, 1>(a, s);
  }
  return hipGetLastError();
}

hipError_t launch_sampler(const SamplerArgs& a, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  if (a.A > 256) return hipErrorInvalidValue;
  hipLaunchKernelGGL(sampler_kernel, dim3((a.rows + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_sampler_embed(const SamplerArgs& a, const EmbedTokenArgs& e, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  if (a.A > 256 || !a.gumbel || e.d > 256 * kMaxPerThread || e.d % 32 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(sampler_embed_kernel, dim3(a.rows), dim3(256), 0, s, a, e);
  return hipGetLastError();
}

}  // namespace vla
