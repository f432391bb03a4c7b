// Decode-time skinny GEMM on gfx950: C = A * W^T for M <= 128 rows (one per
// environment), A [M, K] bf16, W [N, K] bf16, fp32 accumulation.
//
// Decode streams every weight once per step, so the kernel is shaped for HBM
// bandwidth and for balance over the CUs:
//  - One persistent 256-thread workgroup per CU.  The work is cut into units
//    of 64 output columns x 256 K.  Whole column tiles are dealt out one per
//    workgroup per round; the tiles left over after the last full round are
//    split into their units, and each workgroup takes an equal contiguous run
//    of those (stream-K), so every workgroup streams the same weight bytes.
//  - Every tile segment a workgroup finishes is written as an fp32 partial
//    sum into a slot of a partial buffer; the consumer kernel adds a tile's
//    slots in slot order, so results are bitwise deterministic.  The slot of
//    a segment and a tile's slot count follow from the plan in closed form.
//  - Within a unit the four waves take one 64-wide K step each, as two
//    v_mfma_f32_16x16x32_bf16 k-steps.  Weights and activations are both in
//    frag layout, so every load instruction reads one contiguous 1 KB block
//    that leaves each lane holding its MFMA fragment (the number of memory
//    requests per byte is what bounds this kernel).  The next unit's weights
//    are in flight while a unit's MFMAs run (32 KB per CU; deeper rings only
//    queued more loads), its activations are loaded in the step that uses
//    them, pinned in issue order.
//  - The activations (<= 128 x K bf16) are read through L2, where every
//    workgroup of an XCD shares them.  Per unit a wave loads 8 weight blocks
//    and 2 MB activation blocks (MB = 16-row blocks of A), so at 64 rows the
//    activation loads equal the weight loads in count; they hit in L2 and cost
//    about a tenth of the kernel's time (measured by leaving them out).
//  The device code is in skinny_dev.h, shared with the persistent decode
//  layer kernel.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "lds_limit.h"
#include "skinny_dev.h"

namespace vla {

namespace {

using skinny::COLS;
using skinny::NW;
using skinny::UNIT_K;

template <int MB, bool T, bool S>
__global__ __launch_bounds__(64 * NW, 1) void skinny_kernel(SkinnyArgs a, SkinnyPlan p) {
  extern __shared__ __attribute__((aligned(1024))) float red[];  // [NW][MB*16][COLS], T: then the waves' weight blocks
  const skinny::Sched sc = skinny::make_sched(p, blockIdx.x);
  skinny::Ring<MB> r;
  skinny::run<MB, false, T, S>(sc, a, p, r, red, false);
}

template <int MB, bool T, bool S>
hipError_t launch_mb(const SkinnyArgs& a, const SkinnyPlan& p, hipStream_t st) {
  const size_t lds = skinny::red_bytes<MB>() + (T ? skinny::kTransposeBytes : 0);
  static LdsLimit limit;
  const hipError_t e = limit.allow(reinterpret_cast<const void*>(&skinny_kernel<MB, T, S>), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((skinny_kernel<MB, T, S>), dim3(p.G), dim3(64 * NW), lds, st, a, p);
  return hipGetLastError();
}

template <bool T, bool S>
hipError_t launch_rows(const SkinnyArgs& a, const SkinnyPlan& p, hipStream_t st) {
  const int mb = (a.M + 15) / 16;
  if (mb <= 1) return launch_mb<1, T, S>(a, p, st);
  if (mb <= 2) return launch_mb<2, T, S>(a, p, st);
  if (S || mb <= 4) return launch_mb<4, T, S>(a, p, st);  // S: at most 64 rows
  if constexpr (!S) return launch_mb<8, T, S>(a, p, st);
}

}  // namespace

SkinnyPlan skinny_plan(int N, int K, int workgroups, int max_slots) {
  SkinnyPlan p{};
  p.tiles = N / COLS;
  p.chunks = K / UNIT_K;
  for (int G = std::min(workgroups, kSkinnyMaxGroups); G >= 1; --G) {
    p.G = G;
    p.dp_tiles = (p.tiles / G) * G;
    const int U = (p.tiles - p.dp_tiles) * p.chunks;
    if (U > 0 && U < G) continue;  // every workgroup of a stream-K run needs at least one unit
    p.slots = 1;
    for (int t = p.dp_tiles; t < p.tiles; ++t) p.slots = std::max(p.slots, skinny_slots(p, t));
    if (p.slots <= max_slots) break;
  }
  return p;
}

constexpr long long kStreamElems = 24 << 20, kStreamElemsFew = 14 << 20;
hipError_t launch_skinny(const SkinnyArgs& a, const SkinnyPlan& p, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (a.M > 128 || !skinny_plan_ok(p, a.N, a.K) || (long long)frag_elems(a.N, a.K) * 2 >= (1ll << 31))
    return hipErrorInvalidValue;
  // Past the caches where the model asks for it (its weights do not fit the last-level cache): up to 32 rows from 28 MB a
  // product on, up to 64 rows from 48 MB on.  One product, us, one row, through the caches / past them: 180 MB 33.7 / 31.5,
  // 104 MB 20.2 / 19.3, 52 MB 12.2 / 11.7, 46 MB 10.6 / 10.8, 34 MB 8.7 / 8.6, 19 MB 6.6 / 7.1, 12 MB 5.4 / 5.7.  What a
  // product of 28 to 48 MB leaves in the caches displaces the smaller ones' weights, and counts up to 32 rows.  Whole rollout
  // steps, us, every product past the caches / from 28 MB / from 48 MB: d = 2048, four layers, 1, 16, 24, 32 environments
  // 1589 / 1527 / 1574, 2032 / 1977 / 2015, 2521 / 2468 / 2493, - / 2626 / 2637; d = 2816, four layers, 1, 16, 24
  // 1803 / 1804 / 1830, 2549 / 2540 / 2580, 3077 / 3075 / 3124; but from 28 MB / from 48 MB with 64 environments
  // d = 2048, eight layers 7654 / 7592, d = 2304, five layers 5201 / 5150, d = 2560, four layers 4357 / 4319.  Above 64 rows
  // (all products of a decode, 128 rows, through the caches / every one past them): d = 4096, eight layers 6878 / 6861, d =
  // 2048, eight layers 3319 / 3547.
  const bool stream = a.stream && a.M <= 64 && (long long)a.N * a.K >= (a.M <= 32 ? kStreamElemsFew : kStreamElems);
  return stream ? launch_rows<false, true>(a, p, st) : launch_rows<false, false>(a, p, st);
}

// C = A W with W [kt, ldw] as it lies (the gradients' products over the rows of an activation matrix): the same units, slots
// and sums as launch_skinny with a transposed copy of W, which cost a pass of its own (the twelve of a 4720-row layer's
// gradients at d = 4096 225 us), at the time of the untransposed product (64 rows x 22016, 4720 rows: 46 us for 47).
hipError_t launch_skinny_t(const SkinnyArgs& a, const SkinnyPlan& p, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (a.M > 128 || !skinny_plan_ok(p, a.N, a.K) || a.kt < 1 || a.kt > a.K || a.ldw % 32 != 0 || a.col0 < 0 ||
      a.col0 % 32 != 0 || a.col0 + a.N > a.ldw ||
      (long long)frag_elems(a.kt, a.ldw) * 2 >= (1ll << 31) || (long long)frag_elems(a.M, a.K) * 2 >= (1ll << 31))
    return hipErrorInvalidValue;
  return launch_rows<true, false>(a, p, st);
}

}  // namespace vla
