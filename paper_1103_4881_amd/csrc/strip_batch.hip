// Strip kernel instances of a batch (streams of any sizes and filters).
#include "strip_body.h"
#include "strip_host.h"

namespace aol {

// One workgroup per unit of a batch. Every class of filter is in one kernel, so
// that streams of different filters share the device in one launch; it holds
// the registers of its largest class (three workgroups a compute unit). 64
// uint8 streams of 640x480 to 3840x2160, 237 MB, take 66 us, 3.6 TB/s (one
// persistent workgroup per compute unit with a band of columns in LDS: 76 us):
// about two rounds of workgroups, each with its chain of descriptor loads
// before its first lines. Its waves wait on memory or LDS 44 % of their cycles
// and for an issue slot 28 %; 13 % issue vector instructions.
template <int ELEM, bool EDGES>
__global__ __launch_bounds__(256, EDGES && ELEM == kU8 ? 2 : 3) void k_strip_batch(StripBatch L) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const StripUnit U = load_const((const STRIP_CONST StripUnit*)(uint64_t)L.units + blockIdx.x);
  const StripStream S = load_const((const STRIP_CONST StripStream*)(uint64_t)L.streams + U.stream);
  const STRIP_CONST uint64_t* ptr = (const STRIP_CONST uint64_t*)(uint64_t)L.ptr_table + 2 * U.stream;
  const cfilt_t F = (cfilt_t)(uint64_t)U.filter;
  const gsrc_t src = (gsrc_t)ptr[0];
  const gdst_t dst = (gdst_t)ptr[1];
  constexpr int D = EDGES ? 1 : 2;
#define STRIP_UNIT(CLS, SPLIT, KH, KV, NB)                                                                  \
  case CLS:                                                                                                 \
    strip_body<ELEM, SPLIT, KH, KV, NB, 4, D, EDGES>(S, F, src, dst, U.wb0, U.wnb, U.B0, U.B1, lds);        \
    break;
  if constexpr (ELEM == kU8) {
    switch (U.cls) {
      STRIP_UNIT(0, false, 1, 1, 4)
      STRIP_UNIT(1, true, 1, 1, 4)
      STRIP_UNIT(2, false, 1, 2, 4)
      STRIP_UNIT(3, true, 1, 2, 4)
      STRIP_UNIT(4, false, 2, 2, 2)
      STRIP_UNIT(5, true, 2, 2, 2)
      STRIP_UNIT(6, false, 4, 4, 1)
      STRIP_UNIT(7, true, 4, 4, 1)
    }
  } else {
    switch (U.cls) {
      STRIP_UNIT(0, false, 2, 2, 2)
      STRIP_UNIT(2, false, 2, 3, 2)
      STRIP_UNIT(4, false, 4, 5, 1)
    }
  }
#undef STRIP_UNIT
}

static void (*strip_batch_pick(int elem, bool edges))(StripBatch) {
  if (elem == kBF16) return edges ? k_strip_batch<kBF16, true> : k_strip_batch<kBF16, false>;
  if (elem == kFP16) return edges ? k_strip_batch<kFP16, true> : k_strip_batch<kFP16, false>;
  return edges ? k_strip_batch<kU8, true> : k_strip_batch<kU8, false>;
}

hipError_t strip_batch_prepare(int elem, bool edges, size_t lds_bytes) {
  return hipFuncSetAttribute((const void*)strip_batch_pick(elem, edges), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)lds_bytes);
}

hipError_t strip_batch_launch(int elem, bool edges, const StripBatch& L, int grid, size_t lds_bytes, hipStream_t stream) {
  hipLaunchKernelGGL(strip_batch_pick(elem, edges), dim3(grid), dim3(256), lds_bytes, stream, L);
  return hipGetLastError();
}

}  // namespace aol
