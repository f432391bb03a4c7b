// Prefill GEMM with smaller tiles than gemm_prefill.hip's 256 x 256 (same operands, epilogues and arguments), for
// products whose 256 x 256 tiles leave most CUs idle or end in a nearly empty round: few environments, or a narrow
// decoder.  Every output element is the same sequence of v_mfma_f32_16x16x32_bf16 over K and goes through the same
// epilogue arithmetic as there, so the results are the same bits whichever tile shape runs.
//
// A workgroup copies both operands' 1 KB frag blocks into an LDS ring with buffer_load ... lds; while a wave's MFMAs
// of one stage run, its fragments of the next stage are being read into a second register set and the copies of the
// stages after it are in flight (a ring slot is refilled as soon as its fragments are in registers, one workgroup
// barrier per stage).
//
// What bounds it: the copies.  With the LDS reads and the MFMAs left out a 96 x 64 tile of K = 11008 takes 56 of its
// 60 us; deeper rings than these change nothing, because the columns of W that are in flight at one time are those of
// N / TN tiles only and a CU's misses are served at 30-50 GB/s (256 CUs on distinct lines: 6.2 TB/s).  So a shape is
// worth what it fills, and gemm_plan picks by the time that each would take (below).
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "lds_limit.h"

namespace vla {

namespace {

#define TILE_PIN() __builtin_amdgcn_sched_barrier(0)

// One tile shape: WVM x WVN waves, each owning WMB x WNB 16 x 16 blocks; KS K steps of 32 per stage, S stages.
template <int WMB_, int WNB_, int WVM_, int WVN_, int KS_, int S_>
struct TileShape {
  static constexpr int WMB = WMB_, WNB = WNB_, WVM = WVM_, WVN = WVN_, KS = KS_, S = S_;
  static constexpr int NW = WVM * WVN, NT = 64 * NW;
  static constexpr int TM = 16 * WMB * WVM, TN = 16 * WNB * WVN;
  static constexpr int NA = TM / 16 * KS, NB = TN / 16 * KS;  // 1 KB blocks of A and W per stage
  static constexpr int CA = NA / NW, CW = NB / NW, CPW = CA + CW;
  static constexpr int STAGE = (NA + NB) * 1024;
  // the ring, and in its place for the epilogue the fp32 tile
  static constexpr int LDS = S * STAGE > TM * TN * 4 ? S * STAGE : TM * TN * 4;
  // the epilogue's units of 16 rows x 64 columns, dealt to the waves
  static constexpr int GR = TN / 64, UNITS = GR * (TM / 16), NU = (UNITS + NW - 1) / NW;
  static_assert(NA % NW == 0 && NB % NW == 0, "every wave issues the same number of copies");
  static_assert(TN % 64 == 0 && LDS <= 160 * 1024, "whole 64-column groups; the LDS of a CU");
};

// Tile of workgroup pid: each XCD runs a contiguous run of the tiles, ordered group_m tile rows high, so that the
// workgroups that share columns of W (and rows of A) share an L2.
__device__ __forceinline__ void map_tiles_xcd(int pid, int G, int group_m, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int per = G / 8;
  int L = pid;
  if (pid < per * 8) L = (pid & 7) * per + (pid >> 3);
  const int group = group_m * tiles_n;
  const int g = L / group;
  const int first_m = g * group_m;
  const int gm = min(tiles_m - first_m, group_m);
  const int r = L - g * group;
  tm = first_m + r % gm;
  tn = r / gm;
}

template <int N>
__device__ __forceinline__ void wait_vm() {
  if constexpr (N <= 0) WAIT_VMCNT(0);
  else if constexpr (N < 64) WAIT_VMCNT(N);
  else WAIT_VMCNT(63);
}

// Waits until at most `stages_in_flight` stages' copies of this wave are in flight (the ring's start and tail).
template <int CPW>
__device__ __forceinline__ void wait_vm_rt(int stages_in_flight) {
  switch (stages_in_flight) {
    case 1: wait_vm<CPW>(); break;
    case 2: wait_vm<2 * CPW>(); break;
    case 3: wait_vm<3 * CPW>(); break;
    case 4: wait_vm<4 * CPW>(); break;
    case 5: wait_vm<5 * CPW>(); break;
    case 6: wait_vm<6 * CPW>(); break;
    case 7: wait_vm<7 * CPW>(); break;
    default: wait_vm<0>(); break;
  }
}

template <class T, int EPI>
__global__ __launch_bounds__(T::NT) void gemm_tiles_kernel(GemmArgs a, int tiles_m, int tiles_n, int group_m) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  constexpr int TM = T::TM, TN = T::TN;
  int tm, tn;
  map_tiles_xcd(blockIdx.x, tiles_m * tiles_n, group_m, tiles_m, tiles_n, tm, tn);
  const int M = a.M, N = a.N, K = a.K, m0 = tm * TM, n0 = tn * TN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % T::WVM, wn = wave / T::WVM;
  const int nk = K / 32, nst = (nk + T::KS - 1) / T::KS;

  const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc((void*)a.A, (short)0, 0x7fffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc((void*)a.W, (short)0, 0x7fffffff, 0x00020000);
  const int KBA = frag_kb(a.ka ? a.ka : K), KBW = frag_kb(a.kw ? a.kw : K);
  const int last_rb_a = (M + 15) / 16 - 1, last_rb_w = N / 16 - 1;
  const uint32_t voff = lane * 16;
  const uint32_t lbase = (uint32_t)(uintptr_t)((lds_ptr_t*)lds);
  // copy j of this wave: block wave * CA + j of A's NA (then W's NB), row block b / KS, K step b % KS of the stage
  int sa[T::CA], sw[T::CW];
#pragma unroll
  for (int j = 0; j < T::CA; ++j) sa[j] = min((m0 >> 4) + (wave * T::CA + j) / T::KS, last_rb_a) * KBA * 1024;
#pragma unroll
  for (int j = 0; j < T::CW; ++j) sw[j] = min((n0 >> 4) + (wave * T::CW + j) / T::KS, last_rb_w) * KBW * 1024;
  auto copy_stage = [&](int st, int it) {
    const uint32_t sb = lbase + st * T::STAGE;
#pragma unroll
    for (int j = 0; j < T::CA; ++j) {
      const int b = wave * T::CA + j;
      lds_dma16(sb + b * 1024, voff, rsA, sa[j] + min(it * T::KS + b % T::KS, nk - 1) * 1024);
    }
#pragma unroll
    for (int j = 0; j < T::CW; ++j) {
      const int b = wave * T::CW + j;
      lds_dma16(sb + (T::NA + b) * 1024, voff, rsW, sw[j] + min(it * T::KS + b % T::KS, nk - 1) * 1024);
    }
  };

  f32x4 acc[T::WMB][T::WNB];
#pragma unroll
  for (int i = 0; i < T::WMB; ++i)
#pragma unroll
    for (int j = 0; j < T::WNB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // QKV: the positions and pages of the rows that this lane will store (q, k: row lane / 4 of each of its units, v: rows
  // lane / 8 and 8 + lane / 8) are loaded here, so that the dependent loads run under the main loop (they are in
  // front of the first copies or newer than them: the loop's waits only become stricter)
  int pos[T::NU][2], page[T::NU][2];
  auto unit_c0 = [&](int i) { return n0 + 64 * ((wave + i * T::NW) % T::GR); };
  auto unit_r0 = [&](int i) { return 16 * ((wave + i * T::NW) / T::GR); };
  auto unit_row = [&](int i, int j) {
    return min(m0 + unit_r0(i) + (unit_c0(i) + a.col0 < 2 * a.d_model ? lane >> 2 : 8 * j + (lane >> 3)), M - 1);
  };
  if constexpr (EPI == kEpiQkvRope) {
#pragma unroll
    for (int i = 0; i < T::NU; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        pos[i][j] = a.meta.row_pos[unit_row(i, j)];
        page[i][j] = a.meta.row_env[unit_row(i, j)];
      }
  }
#pragma unroll
  for (int st = 0; st < T::S; ++st)
    if (st < nst) copy_stage(st, st);
  if constexpr (EPI == kEpiQkvRope) {
#pragma unroll
    for (int i = 0; i < T::NU; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) page[i][j] = a.meta.page_table[page[i][j] * a.meta.max_pages + pos[i][j] / kPage];
  }
  struct Frags {
    bf16x8 a[T::KS][T::WMB], w[T::KS][T::WNB];
  } f0, f1;
  int cur = 0;  // ring slot of the stage whose fragments are in registers
  auto read = [&](int slot, Frags& f) {
    const char* sp = lds + slot * T::STAGE + lane * 16;
#pragma unroll
    for (int ks = 0; ks < T::KS; ++ks) {
#pragma unroll
      for (int i = 0; i < T::WMB; ++i)
        f.a[ks][i] = as_bf16x8(*reinterpret_cast<const uint4*>(sp + ((wm * T::WMB + i) * T::KS + ks) * 1024));
#pragma unroll
      for (int j = 0; j < T::WNB; ++j)
        f.w[ks][j] = as_bf16x8(*reinterpret_cast<const uint4*>(sp + (T::NA + (wn * T::WNB + j) * T::KS + ks) * 1024));
    }
  };
  auto step = [&](int it, Frags& f, Frags& fn) {
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this step's fragments are in registers, its slot is free
    if (it + T::S - 1 < nst) wait_vm<T::CPW * (T::S - 2)>();
    else wait_vm_rt<T::CPW>(nst - 2 - it);
    TILE_PIN();
    __builtin_amdgcn_s_barrier();
    TILE_PIN();
    if (it + T::S < nst) copy_stage(cur, it + T::S);
    cur = cur + 1 == T::S ? 0 : cur + 1;
    if (it + 1 < nst) read(cur, fn);
    TILE_PIN();
#pragma unroll
    for (int ks = 0; ks < T::KS; ++ks) {
      if (T::KS > 1 && ks > 0 && it * T::KS + ks >= nk) break;  // K an odd multiple of 32: the last stage is short
#pragma unroll
      for (int i = 0; i < T::WMB; ++i)
#pragma unroll
        for (int j = 0; j < T::WNB; ++j) acc[i][j] = mfma16(f.a[ks][i], f.w[ks][j], acc[i][j]);
    }
    TILE_PIN();
  };
  wait_vm_rt<T::CPW>(min(T::S, nst) - 1);
  __builtin_amdgcn_s_barrier();
  TILE_PIN();
  read(0, f0);
  for (int it = 0; it < nst; it += 2) {
    step(it, f0, f1);
    if (it + 1 < nst) step(it + 1, f1, f0);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // ---- the tile through LDS, row-major, 16-byte chunks XOR-swizzled by row
  float* st = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int i = 0; i < T::WMB; ++i)
#pragma unroll
    for (int j = 0; j < T::WNB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rl = (wm * T::WMB + i) * 16 + 4 * (lane >> 4) + r, cl = (wn * T::WNB + j) * 16 + (lane & 15);
        st[rl * TN + (((cl >> 2) ^ (rl & 15)) << 2) + (cl & 3)] = acc[i][j][r];
      }
  __syncthreads();
  auto chunk = [&](int rl, int q) { return *reinterpret_cast<const float4*>(st + rl * TN + ((q ^ (rl & 15)) << 2)); };
  if constexpr (EPI == kEpiStoreF32 || EPI == kEpiResidual) {
    constexpr int QPR = TN / 4, N4 = TM * QPR / T::NT;
    constexpr int U = N4 < 8 ? N4 : 8;
    for (int e0 = 0; e0 < N4; e0 += U) {
      float4 res[U];
      if constexpr (EPI == kEpiResidual) {
        const float* src = a.R ? a.R : a.C;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int e = tid + (e0 + u) * T::NT, row = m0 + e / QPR, col = n0 + 4 * (e % QPR);
          if (e0 + u < N4 && row < M && col < N) res[u] = *reinterpret_cast<const float4*>(src + (size_t)row * a.ldc + col);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = tid + (e0 + u) * T::NT, rl = e / QPR, q = e % QPR, row = m0 + rl, col = n0 + 4 * q;
        if (e0 + u >= N4 || row >= M || col >= N) continue;
        const float4 v = chunk(rl, q);
        float4* p = reinterpret_cast<float4*>(a.C + (size_t)row * a.ldc + col);
        if constexpr (EPI == kEpiResidual) *p = make_float4(res[u].x + v.x, res[u].y + v.y, res[u].z + v.z, res[u].w + v.w);
        else *p = v;
      }
    }
  } else {
    // a wave takes 16 rows of one 64-column group at a time
#pragma unroll
    for (int i = 0; i < T::NU; ++i) {
      const int c0 = unit_c0(i), cl = (c0 - n0) / 4, r0 = unit_r0(i);  // cl: the group's first float4
      if (wave + i * T::NW >= T::UNITS || c0 >= N || m0 + r0 >= M) continue;
      if constexpr (EPI == kEpiSwiGlu || EPI == kEpiSwiGluKeep) {
        // lane: row lane % 16, features 8 (lane / 16) .. + 8 of the group's 32: one whole 1 KB frag block of H
        const int rl = r0 + (lane & 15), oct = lane >> 4, row = m0 + rl;
        float x1[8], x2[8], o[8];
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
          const float4 v1 = chunk(rl, cl + 2 * oct + h2), v2 = chunk(rl, cl + 8 + 2 * oct + h2);
          x1[4 * h2] = v1.x; x1[4 * h2 + 1] = v1.y; x1[4 * h2 + 2] = v1.z; x1[4 * h2 + 3] = v1.w;
          x2[4 * h2] = v2.x; x2[4 * h2 + 1] = v2.y; x2[4 * h2 + 2] = v2.z; x2[4 * h2 + 3] = v2.w;
          if (EPI == kEpiSwiGluKeep && row < M) {
            float* cr = a.C + (size_t)row * a.ldc + c0 + 8 * oct + 4 * h2;
            *reinterpret_cast<float4*>(cr) = v1;
            *reinterpret_cast<float4*>(cr + 32) = v2;
          }
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) o[t] = x1[t] / (1.f + expf(-x1[t])) * x2[t];
        if (row < M)
          *reinterpret_cast<uint4*>(a.H + frag_index(row, c0 / 2 + 8 * oct, a.ldh)) =
              make_uint4(pack2bf(o[0], o[1]), pack2bf(o[2], o[3]), pack2bf(o[4], o[5]), pack2bf(o[6], o[7]));
      } else {  // kEpiQkvRope: as in gemm_prefill.hip
        const int d = a.d_model, hd = a.head_dim, H = a.n_heads, half = hd / 2;
        const int region = (c0 + a.col0) / d, cc0 = c0 + a.col0 - region * d, head = cc0 / hd, blk = (cc0 % hd) / 64;
        if (region < 2) {
          const int q8 = lane & 3, rl = r0 + (lane >> 2), row = m0 + rl, ai = 32 * blk + 8 * q8;
          const int2 pp = make_int2(pos[i][0], page[i][0]);
          float4 cs[4];
          const float4* rp = reinterpret_cast<const float4*>(a.rope + pp.x * half + ai);
#pragma unroll
          for (int t = 0; t < 4; ++t) cs[t] = rp[t];
          float x1[8], x2[8], o1[8], o2[8];
#pragma unroll
          for (int h2 = 0; h2 < 2; ++h2) {
            const float4 v1 = chunk(rl, cl + 2 * q8 + h2), v2 = chunk(rl, cl + 8 + 2 * q8 + h2);
            x1[4 * h2] = v1.x; x1[4 * h2 + 1] = v1.y; x1[4 * h2 + 2] = v1.z; x1[4 * h2 + 3] = v1.w;
            x2[4 * h2] = v2.x; x2[4 * h2 + 1] = v2.y; x2[4 * h2 + 2] = v2.z; x2[4 * h2 + 3] = v2.w;
          }
          if (row >= M) continue;
#pragma unroll
          for (int t = 0; t < 8; ++t) {  // the rotation, with its fused multiply-adds spelled out
            const float c = (t & 1) ? cs[t >> 1].z : cs[t >> 1].x;
            const float sn = (t & 1) ? cs[t >> 1].w : cs[t >> 1].y;
            o1[t] = fmaf(x1[t], c, -(x2[t] * sn));
            o2[t] = fmaf(x2[t], c, x1[t] * sn);
          }
          bf16_t* dst = region == 0 ? a.q + (size_t)row * a.ldq + head * hd
                                    : a.kv.k + (((size_t)pp.y * H + head) * kPage + pp.x % kPage) * hd;
          *reinterpret_cast<uint4*>(dst + ai) =
              make_uint4(pack2bf(o1[0], o1[1]), pack2bf(o1[2], o1[3]), pack2bf(o1[4], o1[5]), pack2bf(o1[6], o1[7]));
          *reinterpret_cast<uint4*>(dst + half + ai) =
              make_uint4(pack2bf(o2[0], o2[1]), pack2bf(o2[2], o2[3]), pack2bf(o2[4], o2[5]), pack2bf(o2[6], o2[7]));
        } else {
          const int q = lane & 7, i1 = cc0 % hd + 4 * q;
#pragma unroll
          for (int it2 = 0; it2 < 2; ++it2) {
            const int rl = r0 + 8 * it2 + (lane >> 3), row = m0 + rl;
            const int2 pp = make_int2(pos[i][it2], page[i][it2]);
            const float4 v1 = chunk(rl, cl + q), v2 = chunk(rl, cl + q + 8);
            if (row >= M) continue;
            const float x1[4] = {v1.x, v1.y, v1.z, v1.w}, x2[4] = {v2.x, v2.y, v2.z, v2.w};
            bf16_t* vb = a.kv.v + ((size_t)pp.y * H + head) * hd * kPage + pp.x % kPage;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              vb[(size_t)(i1 + t) * kPage] = f2bf(x1[t]);
              vb[(size_t)(i1 + t + 32) * kPage] = f2bf(x2[t]);
            }
          }
        }
      }
    }
  }
}

template <class T, int EPI>
hipError_t launch_shape_epi(const GemmArgs& a, hipStream_t s) {
  static LdsLimit limit;
  const hipError_t e = limit.allow(reinterpret_cast<const void*>(&gemm_tiles_kernel<T, EPI>), T::LDS);
  if (e != hipSuccess) return e;
  const int tm = (a.M + T::TM - 1) / T::TM, tn = (a.N + T::TN - 1) / T::TN;
  const int gm = std::max(1, std::min(tm, 1024 / T::TM));
  hipLaunchKernelGGL((gemm_tiles_kernel<T, EPI>), dim3(tm * tn), dim3(T::NT), T::LDS, s, a, tm, tn, gm);
  return hipGetLastError();
}

template <class T>
hipError_t launch_shape(const GemmArgs& a, GemmEpilogue epi, hipStream_t s) {
  switch (epi) {
    case kEpiStoreF32: return launch_shape_epi<T, kEpiStoreF32>(a, s);
    case kEpiResidual: return launch_shape_epi<T, kEpiResidual>(a, s);
    case kEpiSwiGlu: return launch_shape_epi<T, kEpiSwiGlu>(a, s);
    case kEpiQkvRope: return launch_shape_epi<T, kEpiQkvRope>(a, s);
    case kEpiSwiGluKeep: return launch_shape_epi<T, kEpiSwiGluKeep>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// The shapes, and a fit to their measured times over M = 1 .. 9216 of the projections and input gradients at d = 256 ..
// 4096 (rms error 7-14 %): ns of one K step of 32 with one tile on a CU and with two (two rings fit one CU's LDS up to
// 96 x 128, 128 x 128 and 160 x 128), then us of a launch's first tile outside the main loop and of each later one.
// Shape 0 is gemm_prefill.hip's 256 x 256 tile.
namespace {
struct ShapeCost {
  int tm, tn;
  float t1, t2, first, more;
};
constexpr ShapeCost kShapes[kGemmShapes] = {
    {256, 256, 468.f, 1160.f, 10.8f, 14.1f}, {64, 64, 122.f, 226.f, 3.8f, 0.1f},
    {96, 64, 153.f, 268.f, 4.0f, 0.6f},      {160, 64, 216.f, 438.f, 4.8f, 3.8f},
    {96, 128, 332.f, 379.f, 3.4f, 1.6f},     {128, 128, 364.f, 423.f, 4.2f, 3.0f},
    {160, 128, 392.f, 505.f, 5.4f, 3.7f},    {96, 192, 312.f, 620.f, 6.7f, 6.0f},
    {160, 192, 432.f, 888.f, 9.2f, 7.7f},
};
}  // namespace

// Estimated us of a product on one shape: the CU with the most tiles decides, and two tiles that share a CU cost less
// than twice one.
static float shape_cost(const ShapeCost& c, int M, int N, int K, int cus) {
  const long long tiles = (long long)((M + c.tm - 1) / c.tm) * ((N + c.tn - 1) / c.tn);
  const long long q = (tiles + cus - 1) / cus;
  const float step = (float)(q / 2) * c.t2 + (float)(q % 2) * c.t1;
  return c.first + c.more * (float)(q - 1) + 1e-3f * step * (float)(K / 32);
}

// The shape with the least estimated time.  Over the measured sizes of less than one full round of 256 x 256 tiles (one per
// CU) the choice is 1 % slower than the best shape of each on average (24 % at worst); always 256 x 256 is 69 %.  Measured
// with each product's own epilogue (us, 256 x 256 -> chosen): M = 277, d = 4096: QKV 81 -> 52, O 68 -> 25, gate/up 85 -> 67,
// down 163 -> 58; M = 1088, K = 256, N = 768: 11.6 -> 4.2.
//
// From one full round on the 256 x 256 tile, which does the most work per byte moved, is left only where its last round is
// less than half full:
// - a smaller shape takes the whole product up to kWholeRounds rounds (QKV of d = 256, 22000 rows, 1.02 rounds 49 -> 30 us;
//   O of d = 3072, 6600 rows, 1.22 rounds 152 -> 141).  The estimate, whose steps have the operands in the caches, is too
//   good for smaller tiles in many rounds: by it alone QKV of d = 512, 44000 rows, 4.05 rounds took 136 us for 126, gate/up
//   of d = 256, 55000 rows, 5.1 rounds 137 for 82;
// - or it is cut by rows or columns: its first part the whole rounds that fit (or one round less), the rest on a smaller
//   shape after it.  The estimate, with cut_us for the second launch and the drain before it, has to be 3 % better than one
//   shape's.  M = 2304, d = 4096: gate/up 353 -> 315; M = 4720: O and down together 582 -> 524, the four input gradients of
//   a layer 1530 -> 1380; M = 37760: O and down 3480 -> 3290.  With a last round at least half full every cut measured was
//   slower (1.51 to 1.62 rounds: QKV of d = 3072 158 -> 179, O and down of d = 4096 676 -> 699); so was one of the SwiGLU
//   epilogue, whose 256 x 256 tile hides its stores under the next tile, at K = 256 (2.04 rounds 42 -> 49), and of QKV there
//   in many rounds (3.25 85 -> 101).
// Over about 200 products of 1 to 17 rounds at d = 256 to 4096 the choice is 4.6 % faster than always 256 x 256, none by more
// than 1.5 % slower.
constexpr float kWholeRounds = 1.25f, kWholeRoundsQkv = 1.2f;
GemmPlan gemm_plan(int M, int N, int K, int cus, GemmEpilogue epi) {
  const bool swiglu = epi == kEpiSwiGlu || epi == kEpiSwiGluKeep;
  const float whole = epi == kEpiQkvRope ? kWholeRoundsQkv : kWholeRounds, cut_us = swiglu ? 10.f : 7.f;
  const ShapeCost& big = kShapes[0];
  const int tm = (M + big.tm - 1) / big.tm, tn = (N + big.tn - 1) / big.tn;
  const long long tiles = (long long)tm * tn, rounds = tiles / cus;
  GemmPlan best{};
  float tb = 0.f;
  for (int i = 0; i < kGemmShapes; ++i) {
    const float t = shape_cost(kShapes[i], M, N, K, cus);
    if (i == 0) {
      tb = 0.95f * t;  // a smaller shape has to gain 5 %
    } else if (t < tb && (float)tiles <= whole * (float)cus) {
      tb = t;
      best.first = i;
    }
  }
  if (rounds < 1 || 2 * (tiles % cus) >= cus || (K < 512 && (swiglu || rounds > 2))) return best;
  tb = 0.97f * shape_cost(kShapes[best.first], M, N, K, cus);
  for (long long r = rounds; r >= 1 && r >= rounds - 1; --r) {
    const int cut_n = (int)(r * cus / tm), cut_m = (int)(r * cus / tn);  // tile columns, tile rows in r rounds
    for (int by_rows = 0; by_rows < 2; ++by_rows) {
      const int rows = by_rows ? cut_m * big.tm : 0, cols = by_rows ? 0 : cut_n * big.tn;
      if (rows >= M || cols >= N || rows + cols == 0) continue;
      const float t0 = cut_us + (by_rows ? shape_cost(big, rows, N, K, cus) : shape_cost(big, M, cols, K, cus));
      for (int i = 1; i < kGemmShapes; ++i) {
        const float t = t0 + (by_rows ? shape_cost(kShapes[i], M - rows, N, K, cus)
                                      : shape_cost(kShapes[i], M, N - cols, K, cus));
        if (t < tb) {
          tb = t;
          best = GemmPlan{0, i, rows, cols};
        }
      }
    }
  }
  return best;
}

hipError_t launch_gemm_shape(const GemmArgs& a, GemmEpilogue epi, int shape, hipStream_t s) {
  switch (shape) {
    case 1: return launch_shape<TileShape<2, 2, 2, 2, 2, 4>>(a, epi, s);
    case 2: return launch_shape<TileShape<3, 2, 2, 2, 2, 4>>(a, epi, s);
    case 3: return launch_shape<TileShape<5, 2, 2, 2, 2, 3>>(a, epi, s);
    case 4: return launch_shape<TileShape<3, 4, 2, 2, 2, 2>>(a, epi, s);
    case 5: return launch_shape<TileShape<4, 4, 2, 2, 2, 2>>(a, epi, s);
    case 6: return launch_shape<TileShape<5, 4, 2, 2, 2, 2>>(a, epi, s);
    case 7: return launch_shape<TileShape<3, 6, 2, 2, 2, 3>>(a, epi, s);
    case 8: return launch_shape<TileShape<5, 6, 2, 2, 2, 3>>(a, epi, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace vla
