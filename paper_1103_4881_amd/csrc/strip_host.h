// Host-side construction of the strip kernel's descriptors.
#pragma once
#include <hip/hip_runtime.h>

#include <vector>

#include "common.h"
#include "strip.h"

namespace aol {

// One filter pair's device tables for the strip kernel.
struct StripTables {
  int elem = kU8;
  int cls = -1;       // 2 * class + split; -1: beyond the kernel's instances
  int wnb[kStripForms] = {0, 0};  // strips per workgroup at most, by form (0: no instance)
  int col0 = 0, line0 = 0;
  int p_v = 1;
  int resident = 3;   // workgroups of the usual form resident on a compute unit (registers)
  size_t lds[kStripForms] = {0, 0};  // bytes of a workgroup, by form
  StripFilter host{};
  DeviceBuf d_filter;  // the filter, followed by its operands and biases
};

// AOL_OK with out.cls = -1 when no instance serves the filters.
aol_status build_strip_tables(const FilterHost& hf, const FilterHost& vf, int elem, StripTables& out);

// Descriptor of one plane or stream (segments: see strip_set_segments).
// False for planes of 4 GiB or more (the kernel's lane offsets are 32-bit) and
// for output sides above 2^30.
bool build_strip_stream(const StripTables& t, int64_t h, int64_t w, int64_t in_pitch, int64_t out_pitch,
                        StripStream& S);

uint32_t strip_magic(int d);  // floor(2^32 / d) + 1 (0 for 1)

// A line of the plane is not whole 16-byte chunks.
bool strip_edges(const StripTables& t, const StripStream& S);

// Workgroups of at most wnb strips (evened out over a row) and segments of at
// most segb vertical blocks.
void strip_set_segments(StripStream& S, int wnb, int segb);

// edges: some line of the launch is not whole 16-byte chunks.
hipError_t strip_prepare(int elem, int cls, int form, bool edges, size_t lds_bytes);

// A batch: units of streams of any filter class; edges: of streams with a line
// that is not whole 16-byte chunks.
hipError_t strip_batch_prepare(int elem, bool edges, size_t lds_bytes);
hipError_t strip_batch_launch(int elem, bool edges, const StripBatch& L, int grid, size_t lds_bytes, hipStream_t stream);

hipError_t strip_launch(int elem, int cls, int form, bool edges, const StripLaunch& L, int grid, size_t lds_bytes,
                        hipStream_t stream);

}  // namespace aol
