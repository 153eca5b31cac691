// Structures of the strip kernel (fused downscaler, workgroups of four waves
// on strips of output columns), shared by the host library and the device code.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "aol_internal.h"

namespace aol {

constexpr int kStripSlots = 3;       // 16-byte chunks a thread stages per step of 16 lines
constexpr int kStripMaxBlocks = 16;  // 16-output blocks per period (16 repetitions) and axis at most

// Chunks of a line a workgroup of so many waves stages at most, and the bytes
// of one of its two staging buffers.
constexpr int strip_chunks(int waves) { return 4 * waves * kStripSlots; }
constexpr int strip_stage(int waves) { return 16 * (strip_chunks(waves) | 1) * 16; }

// Kernel instances of a filter pair by the K-steps of its horizontal blocks
// and of its vertical windows, each with the number of adjacent 16-column
// output blocks (strips) a wave takes at most.
struct StripClass {
  int kh, kv, nb;
};
constexpr StripClass kStripU8[] = {{1, 1, 4}, {1, 2, 4}, {2, 2, 2}, {4, 4, 1}};
constexpr StripClass kStripF[] = {{2, 2, 2}, {2, 3, 2}, {4, 5, 1}};
constexpr int kStripU8Classes = 4, kStripFClasses = 3;

// Forms of a launch: four waves a workgroup, or eight (the first class with
// whole coefficients, lines of whole chunks).
enum StripForm : int32_t { kStripUsual = 0, kStripWide = 1, kStripForms = 2 };
constexpr int strip_waves(int form) { return form == kStripWide ? 8 : 4; }

// One filter pair on the device. Horizontal blocks repeat every period (16
// repetitions, q_h * 16 inputs, p_h blocks). The vertical axis is cut into
// steps of 16 input lines counted from line s_min (the least window start);
// a vertical block is computed after step v1 - 1 of its period, from the
// window of the last kv K-steps of intermediate lines.
struct alignas(16) StripFilter {
  const void* hfrag;  // horizontal coefficient operands (64 lanes x 16 B, two parts when split)
  const void* vfrag;  // vertical ones: [block][K-step][part][64][16]
  const int32_t* bias;  // integer form: kStripMaxBlocks * 16 horizontal biases, then the vertical ones
  int32_t nblk_h, per_chunks;   // blocks and 16-byte chunks per period along a line
  int32_t nblk_v, per_steps;    // blocks and steps of 16 lines per period down a column
  uint32_t mg_h, mg_v;          // floor(2^32 / n) + 1 of nblk_h and nblk_v
  int32_t vfrag_bytes;          // bytes of vfrag
  int32_t lds_x;                // LDS byte offset of the staging buffers
  int32_t zfrag;                // index of an all-zero horizontal operand
  int32_t ubias, hbias0, vbias0;  // integer form: 1 if every output of an axis has one bias, and the biases
  int32_t hblk[kStripMaxBlocks];  // chunk0 | operand index << 16 | K-steps << 24
  int32_t hend[kStripMaxBlocks];  // end (chunk) of a block's window
  int32_t v0[kStripMaxBlocks];  // first step a vertical block's window reads
  int32_t v1[kStripMaxBlocks];  // end of the window's steps
  int32_t vlo[kStripMaxBlocks], vhi[kStripMaxBlocks];  // lines of the window
};

// One plane or video stream.
struct alignas(16) StripStream {
  int64_t in_pitch, out_pitch;  // elements
  int32_t h, w, mh, mw;         // input and output sizes
  int32_t col0, line0;          // input column of chunk 0 and line of step 0 (before the wrap)
  int32_t nbh, nbv;             // 16-output blocks along a row / down a column
  int32_t wnb, wgx;             // strips per workgroup, workgroups across a row
  int32_t segb, nseg;           // vertical blocks per segment, segments
  uint32_t mg_wgx;              // floor(2^32 / wgx) + 1
  int32_t wg_base;              // first workgroup of the plane inside a frame
  int32_t tiny;                 // a line is shorter than one 16-byte chunk
  int32_t pad[3];
};

// One workgroup of a batch: strips [wb0, wb0 + wnb) and vertical blocks
// [B0, B1) of a stream.
struct alignas(16) StripUnit {
  const StripFilter* filter;
  int32_t cls;                  // 2 * class + split
  int32_t stream;               // index of the stream and of its pointers
  int32_t wb0, wnb, B0, B1;
};

// One launch of a batch: a workgroup per unit.
struct StripBatch {
  const StripStream* streams;
  const StripUnit* units;
  void* const* ptr_table;       // [in, out] per stream
};

struct StripLaunch {
  StripFilter filter;            // a plan's filters, in the launch's arguments: one dependent load less
  StripStream st[kMaxPlanes];    // a plan's planes
  const void* ptrs[2 * kMaxPlanes];  // in, out per plane
  int64_t fstride[2 * kMaxPlanes];   // elements between frames (in, out) per plane
  int32_t n_planes, wgs_per_frame;
  uint32_t mg_wgs;               // floor(2^32 / wgs_per_frame) + 1
  int32_t first;                 // the launch's first workgroup (a large launch is cut)
  int32_t by_xcd;                // items of one XCD: consecutive ones (-1, first is 0) or in runs of 2^by_xcd
};

}  // namespace aol
