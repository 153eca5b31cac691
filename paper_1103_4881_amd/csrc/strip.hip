// Strip kernel instances of a plan (one filter pair, up to kMaxPlanes planes).
#include "strip_body.h"
#include "strip_host.h"

namespace aol {

namespace {

// Workgroup x of the launch, with the workgroups of one XCD (dispatched to
// the 8 XCDs in turn) taking consecutive items: neighbouring strips and
// segments share the lines at their borders through that XCD's L2.
__device__ __forceinline__ int strip_item(int x, int total) {
  const int per = total >> 3, rem = total & 7, xcd = x & 7;
  return xcd * per + min(xcd, rem) + (x >> 3);
}

// The same in runs of 2^s consecutive items per XCD: neighbours in a row share
// their lines, and all XCDs stay in the same frames.
__device__ __forceinline__ int strip_run(int x, int total, int s) {
  const int block = 8 << s;
  if ((x | (block - 1)) >= total) return x;  // the launch's last items in order
  return (x & ~(block - 1)) + ((x & 7) << s) + ((x & (block - 1)) >> 3);
}

}  // namespace

// Waves per SIMD the registers are held to: four (128 registers) where the
// instance fits without spilling, else three (168), or two.
constexpr int strip_occ(int elem, bool split, int kh, int kv, bool edges) {
  if (edges && split && kv == 2) return 2;
  return !edges && !split && (kh * kv == 1 || (elem != kU8 && kv == 2)) ? 4 : 3;
}

template <int ELEM, bool SPLIT, int KH, int KV, int NB, int W, int D, bool EDGES>
__global__ __launch_bounds__(64 * W, strip_occ(ELEM, SPLIT, KH, KV, EDGES)) void k_strip(StripLaunch L) {
  constexpr int ES = ELEM == kU8 ? 1 : 2, OES = ELEM == kU8 ? 1 : 4;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const STRIP_CONST StripLaunch* A = (const STRIP_CONST StripLaunch*)__builtin_amdgcn_kernarg_segment_ptr();
  const int item = L.by_xcd < 0 ? strip_item(blockIdx.x, gridDim.x) : strip_run(blockIdx.x, gridDim.x, L.by_xcd) + L.first;
  const int frame = div_by(item, L.wgs_per_frame, L.mg_wgs);
  int r = item - frame * L.wgs_per_frame;
  int pl = 0;
  for (int j = 1; j < L.n_planes; ++j)
    if (r >= A->st[j].wg_base) pl = j;
  const StripStream S = load_const(&A->st[pl]);
  r -= S.wg_base;
  const int seg = div_by(r, S.wgx, S.mg_wgx), wx = r - seg * S.wgx;
  const gsrc_t src = (gsrc_t)(uint64_t)A->ptrs[2 * pl] + (int64_t)frame * A->fstride[2 * pl] * ES;
  const gdst_t dst = (gdst_t)(uint64_t)A->ptrs[2 * pl + 1] + (int64_t)frame * A->fstride[2 * pl + 1] * OES;
  strip_body<ELEM, SPLIT, KH, KV, NB, W, D, EDGES>(S, &A->filter, src, dst, wx * S.wnb, min(S.wnb, S.nbh - wx * S.wnb),
                                                   seg * S.segb, min(S.nbv, (seg + 1) * S.segb), lds);
}

using StripFn = void (*)(StripLaunch);

template <int ELEM, bool SPLIT, int KH, int KV, int NB>
static StripFn strip_pick_form(int form, bool edges) {
  if constexpr (!SPLIT && KH * KV == (ELEM == kU8 ? 1 : 4))
    if (form == kStripWide) return k_strip<ELEM, SPLIT, KH, KV, NB, 8, 2, false>;
  return edges ? k_strip<ELEM, SPLIT, KH, KV, NB, 4, 1, true> : k_strip<ELEM, SPLIT, KH, KV, NB, 4, 2, false>;
}

template <int ELEM>
static StripFn strip_pick_f(int cls, int form, bool edges) {
  switch (cls) {
    case 0: return strip_pick_form<ELEM, false, 2, 2, 2>(form, edges);
    case 2: return strip_pick_form<ELEM, false, 2, 3, 2>(form, edges);
    default: return strip_pick_form<ELEM, false, 4, 5, 1>(form, edges);
  }
}

static StripFn strip_pick(int elem, int cls, int form, bool edges) {
  if (elem == kBF16) return strip_pick_f<kBF16>(cls, form, edges);
  if (elem == kFP16) return strip_pick_f<kFP16>(cls, form, edges);
  switch (cls) {
    case 0: return strip_pick_form<kU8, false, 1, 1, 4>(form, edges);
    case 1: return strip_pick_form<kU8, true, 1, 1, 4>(form, edges);
    case 2: return strip_pick_form<kU8, false, 1, 2, 4>(form, edges);
    case 3: return strip_pick_form<kU8, true, 1, 2, 4>(form, edges);
    case 4: return strip_pick_form<kU8, false, 2, 2, 2>(form, edges);
    case 5: return strip_pick_form<kU8, true, 2, 2, 2>(form, edges);
    case 6: return strip_pick_form<kU8, false, 4, 4, 1>(form, edges);
    default: return strip_pick_form<kU8, true, 4, 4, 1>(form, edges);
  }
}

hipError_t strip_prepare(int elem, int cls, int form, bool edges, size_t lds_bytes) {
  return hipFuncSetAttribute((const void*)strip_pick(elem, cls, form, edges),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
}

hipError_t strip_launch(int elem, int cls, int form, bool edges, const StripLaunch& L, int grid, size_t lds_bytes,
                        hipStream_t stream) {
  hipLaunchKernelGGL(strip_pick(elem, cls, form, edges), dim3(grid), dim3(64 * strip_waves(form)), lds_bytes, stream,
                     L);
  return hipGetLastError();
}

}  // namespace aol
