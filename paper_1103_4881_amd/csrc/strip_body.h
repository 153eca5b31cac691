// Fused downscaler for gfx950 (integer and float forms): small workgroups
// that walk down a plane with the intermediate frame in registers.
//
// Both filters of the downscaler (Sec. III: horizontal filter over every
// line, then vertical filter over every column, per frame and colour plane;
// Sec. III-A: one independent elementary task per repetition) on the matrix
// cores:
//
//  * a workgroup of four waves owns up to 4 * NB adjacent 16-column output
//    blocks (strips) and a segment of vertical output blocks, and walks down
//    the plane 16 input lines per step: the step's lines are loaded once, in
//    16-byte chunks of consecutive lanes, and staged in LDS (two buffers, one
//    barrier per step); each wave takes NB strips;
//  * the product of 16 staged lines with a strip's coefficients leaves each
//    lane four intermediate lines of one output column. K is a contraction
//    index, so the vertical product may take its lines in any order that its
//    coefficients share: packed as they stand, the last steps' results are
//    its operand, and the intermediate frame never leaves the registers;
//  * after the step that completes a vertical block's window, the vertical
//    product runs on the last steps and its 16 x 16 outputs are stored, in
//    whole 16-byte pieces of rows (integer form: the strips' words change
//    places between lane groups first).
//
// Rows need not be aligned: gfx950 loads and stores 16 bytes at any address.
// A chunk that crosses the end of a line (Array-OL tilers index modulo the
// line) is joined from the line's last 16 bytes and its first 16 by a byte
// shift; only the workgroups that own such a chunk run that code.
//
// Integer: i8 MFMA on x ^ 0x80 (x - 128), 128 * sum(c) restored through the
// bias, taps beyond int8 as lo + 128 * hi, int32 accumulation (exact), uint8
// intermediate. Float: bf16/fp16 MFMA with fp32 accumulation, the
// intermediate kept as a hi/lo pair of 16-bit values, fp32 output.

#pragma once
#include "strip.h"

namespace aol {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
// memory accesses at any byte address
typedef int v4i_any __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t v2u_any __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));

// Device data is read and written through global (1) and constant (4)
// address-space pointers: pointers read from tables are generic to the
// compiler, and generic accesses compile to flat instructions.
#define STRIP_GLOBAL __attribute__((address_space(1)))
#define STRIP_CONST __attribute__((address_space(4)))
typedef const STRIP_GLOBAL uint8_t* gsrc_t;
typedef STRIP_GLOBAL uint8_t* gdst_t;
typedef const STRIP_CONST StripFilter* cfilt_t;

template <class T>
__device__ __forceinline__ T load_const(const STRIP_CONST T* p) {
  static_assert(sizeof(T) % 4 == 0, "descriptor of whole words");
  T v;
  const STRIP_CONST uint32_t* src = (const STRIP_CONST uint32_t*)p;
  uint32_t* dst = reinterpret_cast<uint32_t*>(&v);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) dst[i] = src[i];
  return v;
}

__device__ __forceinline__ int pmod(int x, int m) {
  const int r = x % m;
  return r < 0 ? r + m : r;
}

__device__ __forceinline__ v4i to_i8(v4i x) {
  const int m = (int)0x80808080u;
  return v4i{x[0] ^ m, x[1] ^ m, x[2] ^ m, x[3] ^ m};
}

// clamp(floor(acc / 256), 0, 255) x 4, packed (acc holds the bias and the
// rounding). Clamped before the shift on purpose: a clamp after it lets the
// compiler use v_ashr_pk_u8_i32 and OR the register's stale upper half into
// the neighbouring bytes.
__device__ __forceinline__ uint32_t quant4(v4i acc) {
  uint32_t x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = (uint32_t)min(max(acc[i], 0), 65535);
  return __builtin_amdgcn_perm(x[1], x[0], 0x0c0c0501u) | __builtin_amdgcn_perm(x[3], x[2], 0x05010c0cu);
}

template <int ELEM>
__device__ __forceinline__ v4f mfma16(v4i a, v4i b, v4f c) {
  if constexpr (ELEM == kBF16) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
  } else {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
  }
}

template <int ELEM>
__device__ __forceinline__ uint32_t pack2(float x, float y) {
  if constexpr (ELEM == kBF16) {
    return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)x) | ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)y) << 16);
  } else {
    return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)x) | ((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)y) << 16);
  }
}

template <int ELEM>
__device__ __forceinline__ float lo16(uint32_t v) {
  if constexpr (ELEM == kBF16) return __uint_as_float(v << 16);
  else return (float)__builtin_bit_cast(_Float16, (uint16_t)(v & 0xFFFFu));
}

template <int ELEM>
__device__ __forceinline__ float hi16(uint32_t v) {
  if constexpr (ELEM == kBF16) return __uint_as_float(v & 0xFFFF0000u);
  else return (float)__builtin_bit_cast(_Float16, (uint16_t)(v >> 16));
}

// Bytes [s, s + 16) of the 32 bytes a, b (s in 0 .. 15, per lane).
__device__ __forceinline__ v4i join_bytes(v4i a, v4i b, int s) {
  asm("" : "+v"(s));  // the masks are not worth registers of the step loop
  uint32_t d[8] = {(uint32_t)a[0], (uint32_t)a[1], (uint32_t)a[2], (uint32_t)a[3],
                   (uint32_t)b[0], (uint32_t)b[1], (uint32_t)b[2], (uint32_t)b[3]};
  const uint32_t m8 = 0u - ((uint32_t)s >> 3 & 1u), m4 = 0u - ((uint32_t)s >> 2 & 1u);
#pragma unroll
  for (int i = 0; i < 6; ++i) d[i] = (d[i + 2] & m8) | (d[i] & ~m8);  // v_bfi
#pragma unroll
  for (int i = 0; i < 5; ++i) d[i] = (d[i + 1] & m4) | (d[i] & ~m4);
  v4i r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = (int)__builtin_amdgcn_alignbyte(d[i + 1], d[i], (uint32_t)(s & 3));
  return r;
}

// One chunk of a line shorter than a chunk, element by element with the wrap.
template <int ES>
__device__ __forceinline__ v4i gather_chunk(gsrc_t row, int col, int w) {
  uint32_t r[4] = {0, 0, 0, 0};
  int c = pmod(col, w);
#pragma unroll 1
  for (int e = 0; e < 16 / ES; ++e) {
    const uint32_t v = ES == 1 ? (uint32_t)row[c] : (uint32_t)((const STRIP_GLOBAL uint16_t*)row)[c];
    c = c + 1 == w ? 0 : c + 1;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __builtin_amdgcn_alignbyte(i < 3 ? r[i + 1] : v, r[i], ES);
  }
  return v4i{(int)r[0], (int)r[1], (int)r[2], (int)r[3]};
}

// Workgroup barrier that orders LDS only: global loads and stores stay in
// flight (__syncthreads() would wait for them all).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

enum { kWhole, kJoin, kGather };  // how a workgroup's chunks lie on their lines

// floor(n / d) for 0 <= n < 2^31 from m = floor(2^32 / d) + 1 (the product's
// high word is the quotient or one more).
__device__ __forceinline__ int div_by(int n, int d, uint32_t m) {
  if (d == 1) return n;  // m would be 2^32 + 1
  const uint32_t q = __umulhi((uint32_t)n, m);
  return (int)(q * (uint32_t)d > (uint32_t)n ? q - 1 : q);
}

// W: waves of the workgroup; D: steps of input lines in flight beside the
// staged one.
template <int ELEM, bool SPLIT, int KH, int KV, int NB, int W, int D>
struct Strip {
  static constexpr int ES = ELEM == kU8 ? 1 : 2;    // input element bytes
  static constexpr int E = 16 / ES;                 // elements per chunk
  static constexpr int OES = ELEM == kU8 ? 1 : 4;   // output element bytes
  static constexpr int SK = ELEM == kU8 ? 4 : 2;    // steps per vertical K-step
  static constexpr int NZ = SK * KV;                // steps of the vertical window
  static constexpr int PARTS = SPLIT ? 2 : 1;
  // The window is a ring of registers: a step's slot is a constant where the
  // step loop is unrolled over the ring (longer windows shift instead).
  static constexpr bool RING = NZ <= 8;
  static constexpr int U = RING ? NZ : 2;           // steps per iteration of the loop
  static_assert(U % D == 0 && U % 2 == 0, "whole rounds of the loads in flight and of the staging buffers");

  gsrc_t src;
  gdst_t dst;
  int b0, nb, B0, B1;     // the wave's first strip, its strips, vertical blocks
  int tid, lane, g, n;
  int s0, s1;             // steps [s0, s1)
  int lo, hi;             // the segment's input lines, counted from line0
  bool far;               // some of them wrap more than once
  // staging: the thread's chunks of a step's 16 lines
  int srow[kStripSlots];       // line
  uint32_t soff[kStripSlots];  // byte offset from the step's first line
  int sshift[kStripSlots];     // bytes past the line's end (kJoin), or the column (kGather)
  int sdst[kStripSlots];       // LDS byte offset
  // strips
  int aoff[NB][KH];            // LDS byte offset of the lane's operand chunk
  v4i bf[NB][KH], bfh[SPLIT ? NB : 1][KH];  // horizontal coefficients
  int hb[NB];             // horizontal bias of the lane's column (integer form, biases that differ)
  int v1tab;              // lane i: v1[i]

  // wb0, wnb: the workgroup's first strip and its strips
  __device__ __forceinline__ int setup(const StripStream& S, cfilt_t F, int wb0, int wnb) {
    lane = tid & 63;
    g = lane >> 4;
    n = lane & 15;
    const int nblk = F->nblk_h;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per_wave = (wnb + W - 1) / W;
    b0 = wb0 + wave * per_wave;
    nb = min(per_wave, wb0 + wnb - b0);
    // the workgroup's chunks: from its first strip's window to its last one's
    const int fper = div_by(wb0, nblk, F->mg_h), lper = div_by(wb0 + wnb - 1, nblk, F->mg_h);
    const int cfirst = (int)((uint32_t)F->hblk[wb0 - fper * nblk] & 0xFFFFu) + fper * F->per_chunks;
    const int nch = F->hend[wb0 + wnb - 1 - lper * nblk] + lper * F->per_chunks - cfirst;
    const int colf = S.col0 + cfirst * E, pitch = (nch | 1) * 16;  // an odd number of chunks: no bank conflict
    const uint32_t magic = (uint32_t)((1 << 20) / nch) + 1;        // idx / nch for idx < 4096, nch < 256
#pragma unroll
    for (int i = 0; i < kStripSlots; ++i) {
      // a lane past the last chunk stages chunk 0 of line 15 again
      const uint32_t idx = (uint32_t)(tid + i * 64 * W);
      int row = (int)((idx * magic) >> 20), c = (int)idx - row * nch;
      if (row >= 16) {
        row = 15;
        c = 0;
      }
      srow[i] = row;
      sdst[i] = row * pitch + c * 16;
      int col = colf + c * E;
      if (S.tiny) {
        sshift[i] = col;
        soff[i] = (uint32_t)row * (uint32_t)(S.in_pitch * ES);
      } else {
        if (col < 0 || col >= S.w) col = pmod(col, S.w);
        const int past = max(col + E - S.w, 0);
        sshift[i] = past * ES;
        soff[i] = (uint32_t)((col - past) * ES) + (uint32_t)row * (uint32_t)(S.in_pitch * ES);
      }
    }
    v1tab = ((const STRIP_GLOBAL int32_t*)(uint64_t)F->v1)[lane & (kStripMaxBlocks - 1)];
    const gsrc_t hf = (gsrc_t)(uint64_t)F->hfrag + lane * 16;
    const int bs = min(b0, wb0 + wnb - 1);  // (a wave without strips repeats the last one and stores nothing)
    int per = div_by(bs, nblk, F->mg_h), lb = bs - per * nblk;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const uint32_t e = (uint32_t)F->hblk[lb];
      const int c0 = (int)(e & 0xFFFFu) + per * F->per_chunks - cfirst;
      const int cend = F->hend[lb] + per * F->per_chunks - cfirst;
      const int f0 = (int)((e >> 16) & 0xFFu), nk = (int)(e >> 24);
#pragma unroll
      for (int k = 0; k < KH; ++k) {
        // K-steps and chunks beyond the window: zero coefficients on the window's own
        // chunks (0 * x is not 0 for an infinity or NaN)
        const bool on = k < nk;
        aoff[j][k] = n * pitch + min(c0 + (on ? 4 * k : 0) + g, cend - 1) * 16;
        const int f = (on ? f0 + k : F->zfrag) * PARTS;
        bf[j][k] = *(const STRIP_GLOBAL v4i*)(hf + f * 1024);
        if constexpr (SPLIT) bfh[j][k] = *(const STRIP_GLOBAL v4i*)(hf + f * 1024 + 1024);
      }
      hb[j] = 0;
      if constexpr (ELEM == kU8)
        hb[j] = ((const STRIP_GLOBAL int32_t*)(uint64_t)F->bias)[lb * 16 + n];
      if (j + 1 < nb) {  // a missing strip repeats the last one
        if (++lb == nblk) {
          lb = 0;
          ++per;
        }
      }
    }
    const int nv = F->nblk_v;
    const int p0 = div_by(B0, nv, F->mg_v), p1 = div_by(B1 - 1, nv, F->mg_v);
    s0 = F->v0[B0 - p0 * nv] + p0 * F->per_steps;
    s1 = F->v1[(B1 - 1) - p1 * nv] + p1 * F->per_steps;
    lo = F->vlo[B0 - p0 * nv] + 16 * p0 * F->per_steps;
    hi = F->vhi[(B1 - 1) - p1 * nv] + 16 * p1 * F->per_steps;
    far = S.line0 + lo < -S.h || S.line0 + hi > 2 * S.h;
    return S.tiny ? kGather : S.w % E != 0 && (colf < 0 || colf + nch * E > S.w) ? kJoin : kWhole;
  }

  // Loads of one step. A line the segment does not need (of its first and
  // last step, or past them) is its nearest line again: a cache hit instead of
  // memory traffic (a seventh of the reads of a 432-line segment otherwise). A
  // plane is under 4 GiB in this kernel: a uniform base and a 32-bit offset
  // per lane.
  template <int EDGE>
  __device__ __forceinline__ void issue(const StripStream& S, int s, v4i (&pre)[kStripSlots],
                                        v4i (&first)[kStripSlots]) const {
    const int top = S.line0 + 16 * s;
    const uint32_t pitch = (uint32_t)(S.in_pitch * ES);
    gsrc_t base = src + (int64_t)top * (int64_t)pitch;
    uint32_t off[kStripSlots], line[kStripSlots];
#pragma unroll
    for (int i = 0; i < kStripSlots; ++i) {
      off[i] = soff[i];
      if constexpr (EDGE != kWhole) line[i] = (uint32_t)srow[i] * pitch;
    }
    if (16 * s < lo || 16 * s + 16 > hi || top < 0 || top + 16 > S.h) {  // uniform; lines wrap modulo the height
      base = src;
#pragma unroll
      for (int i = 0; i < kStripSlots; ++i) {
        int row = S.line0 + min(max(16 * s + srow[i], lo), hi - 1);
        if (far) {  // uniform: more than one wrap
          row = pmod(row, S.h);
        } else {
          row += row < 0 ? S.h : 0;
          row -= row >= S.h ? S.h : 0;
        }
        const uint32_t wrapped = (uint32_t)row * pitch;
        off[i] = soff[i] - (uint32_t)srow[i] * pitch + wrapped;
        if constexpr (EDGE != kWhole) line[i] = wrapped;
      }
    }
#pragma unroll
    for (int i = 0; i < kStripSlots; ++i) {
      if constexpr (EDGE == kGather) {
        pre[i] = gather_chunk<ES>(base + line[i], sshift[i], S.w);
      } else {
        pre[i] = *(const STRIP_GLOBAL v4i_any*)(base + off[i]);
        if constexpr (EDGE == kJoin) first[i] = *(const STRIP_GLOBAL v4i_any*)(base + line[i]);
      }
    }
  }

  // Integer form: staged as signed bytes x - 128 (the matrix-core operand).
  template <int EDGE>
  __device__ __forceinline__ void commit(const v4i (&pre)[kStripSlots], const v4i (&first)[kStripSlots],
                                         uint8_t* xs) const {
#pragma unroll
    for (int i = 0; i < kStripSlots; ++i) {
      v4i a = pre[i];
      if constexpr (EDGE == kJoin) a = join_bytes(a, first[i], sshift[i]);
      if constexpr (ELEM == kU8) a = to_i8(a);
      *reinterpret_cast<v4i*>(xs + sdst[i]) = a;
    }
  }

  // Stores the wave's blocks of vertical block B: lane (g, n) holds columns
  // 4g .. 4g + 3 of row n of every block.
  __device__ __forceinline__ void store(const StripStream& S, int B, const uint32_t (&y)[NB]) const {
    const uint32_t pitch = (uint32_t)S.out_pitch;
    const gdst_t base = dst + (int64_t)(16 * B) * S.out_pitch + 16 * b0;
    constexpr int LB = 4 * NB;  // bytes a lane stores
    uint32_t o[NB];
    int col;  // the lane's first column, from the wave's first
    if constexpr (NB == 4) {
      // 4 x 4 words between lane groups and blocks: lane group g gets block g whole
      const auto a = __builtin_amdgcn_permlane16_swap(y[0], y[1], false, false);
      const auto b = __builtin_amdgcn_permlane16_swap(y[2], y[3], false, false);
      const auto c = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false);
      const auto d = __builtin_amdgcn_permlane32_swap(a[1], b[1], false, false);
      o[0] = c[0];
      o[1] = d[0];
      o[2] = c[1];
      o[3] = d[1];
      col = 16 * g;
    } else if constexpr (NB == 2) {
      // lane groups 0 and 2 get the two halves of block 0, groups 1 and 3 of block 1
      const auto a = __builtin_amdgcn_permlane16_swap(y[0], y[1], false, false);
      o[0] = a[0];
      o[1] = a[1];
      col = 16 * (g & 1) + 8 * (g >> 1);
    } else {
      o[0] = y[0];
      col = 4 * g;
    }
    uint32_t at = (uint32_t)n * pitch + (uint32_t)col;
    // the lane's bytes inside the plane and the wave's strips
    int left = 16 * B + n < S.mh ? min(S.mw - 16 * b0, 16 * nb) - col : 0;
    if (left >= LB) {
      if constexpr (NB == 4) *(STRIP_GLOBAL v4i_any*)(base + at) = v4i{(int)o[0], (int)o[1], (int)o[2], (int)o[3]};
      else if constexpr (NB == 2) *(STRIP_GLOBAL v2u_any*)(base + at) = v2u_any{o[0], o[1]};
      else *(STRIP_GLOBAL u32_any*)(base + at) = o[0];
    } else if (left > 0) {
      asm("" : "+v"(left), "+v"(at));  // (nothing of this rare path is worth a register of the step loop)
#pragma unroll
      for (int i = 0; i < LB; ++i)
        if (i < left) base[at + i] = (uint8_t)(o[i >> 2] >> (8 * (i & 3)));
    }
  }

  __device__ __forceinline__ void store(const StripStream& S, int B, const v4f (&y)[NB]) const {
    const gdst_t base = dst + ((int64_t)(16 * B) * S.out_pitch + 16 * b0) * 4;
    uint32_t at = ((uint32_t)n * (uint32_t)S.out_pitch + 4 * g) * 4;
    int left = 16 * B + n < S.mh ? min(S.mw - 16 * b0, 16 * nb) - 4 * g : 0;  // from the lane's first column
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (left >= 16 * j + 4) {
        *(STRIP_GLOBAL v4f_any*)(base + (at + 64 * j)) = y[j];
      } else if (left > 16 * j) {
        asm("" : "+v"(left), "+v"(at));  // (nothing of this rare path is worth a register of the step loop)
#pragma unroll
        for (int i = 0; i < 3; ++i)
          if (16 * j + i < left) *(STRIP_GLOBAL float*)(base + (at + 64 * j + 4 * i)) = y[j][i];
      }
    }
  }

  // UB: every output of an axis has the same bias (else added per column).
  template <int EDGE, bool UB>
  __device__ __forceinline__ void run(const StripStream& S, cfilt_t F, uint8_t* lds, v4i vf0, int vb0t) {
    // D steps of input lines in flight beside the staged one
    v4i pre[D][kStripSlots], first[D][kStripSlots];
#pragma unroll
    for (int d = 0; d < D; ++d) issue<EDGE>(S, s0 + d, pre[d], first[d]);

    // the filter's vertical coefficients and biases (vf0, vb0t: the thread's
    // first ones, loaded before the lines so that their wait is short)
    const int vbytes = F->vfrag_bytes;
    if (tid < vbytes / 16) reinterpret_cast<v4i*>(lds)[tid] = vf0;
    if (ELEM == kU8 && tid < F->nblk_v * 16) reinterpret_cast<int*>(lds + vbytes)[tid] = vb0t;
    for (int i = tid + 64 * W; i < vbytes / 16; i += 64 * W)
      reinterpret_cast<v4i*>(lds)[i] = ((const STRIP_GLOBAL v4i*)(uint64_t)F->vfrag)[i];

    const int hb0 = ELEM == kU8 && UB ? F->hbias0 : 0, vb0 = ELEM == kU8 && UB ? F->vbias0 : 0;
    const v4i hq = v4i{hb0, hb0, hb0, hb0};
    // window of intermediate lines: per block and step, four lines of the
    // lane's column (integer: bytes; float: two words hi, two words lo)
    constexpr int ZW = ELEM == kU8 ? 1 : 4;
    uint32_t z[NB][NZ][ZW];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int i = 0; i < NZ; ++i)
#pragma unroll
        for (int q = 0; q < ZW; ++q) z[j][i][q] = 0;
    const int nv = F->nblk_v, psteps = F->per_steps;
    int B = B0;
    const int vp = div_by(B0, nv, F->mg_v);
    int vlb = B0 - vp * nv, vper = vp * psteps - s0;  // block within the period, the period's first step
    int fire = __builtin_amdgcn_readlane(v1tab, vlb) + vper;

    // Vertical block B from the window ending before step `fire` (from s0);
    // r: fire mod NZ, a constant where the step loop is unrolled over the ring.
    auto vblock = [&](int r) __attribute__((always_inline)) {
      const uint8_t* fl = lds + (vlb * KV * PARTS) * 1024 + lane * 16;
      v4i vf[KV], vfh[SPLIT ? KV : 1];
      if constexpr (RING && ELEM == kU8) {
        // the coefficients in the order of the ring's slots: slot d holds
        // window step (d - fire) mod NZ
#pragma unroll
        for (int d = 0; d < NZ; ++d) {
          const int i = d - r + (d < r ? NZ : 0);
          const uint8_t* f = fl + (i >> 2) * PARTS * 1024 + (i & 3) * 4;
          vf[d >> 2][d & 3] = *reinterpret_cast<const int*>(f);
          if constexpr (SPLIT) vfh[d >> 2][d & 3] = *reinterpret_cast<const int*>(f + 1024);
        }
      } else {
#pragma unroll
        for (int k = 0; k < KV; ++k) {
          vf[k] = *reinterpret_cast<const v4i*>(fl + (k * PARTS) * 1024);
          if constexpr (SPLIT) vfh[k] = *reinterpret_cast<const v4i*>(fl + (k * PARTS) * 1024 + 1024);
        }
      }
      if constexpr (ELEM == kU8) {
        int bias = vb0;
        if constexpr (!UB) bias = *reinterpret_cast<const int*>(lds + vbytes + (vlb * 16 + n) * 4);
        const v4i bq = v4i{bias, bias, bias, bias};
        uint32_t y[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          v4i acc = bq;
          if constexpr (SPLIT) {
            v4i hi = v4i{0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < KV; ++k) hi = __builtin_amdgcn_mfma_i32_16x16x64_i8(zop8(z[j], k), vfh[k], hi, 0, 0, 0);
            acc = hi * 128 + bq;
          }
#pragma unroll
          for (int k = 0; k < KV; ++k) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(zop8(z[j], k), vf[k], acc, 0, 0, 0);
          y[j] = quant4(acc);
        }
        store(S, B, y);
      } else {
        // The low halves first: their sums round at their own small size. The window's
        // steps in order wherever the ring starts: sums round alike in every schedule.
        // (Where it starts at an odd slot the operands cross the pairs of slots that are
        // adjacent registers; an xor with zero copies them, which the compiler would
        // otherwise do for the whole window at once, in registers it does not have.)
        v4f y[NB];
        float sum = 0.f;  // not finite if one of the results is not
        int zero = 0;
        asm("" : "+s"(zero));
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          y[j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int h = 2; h >= 0; h -= 2)
#pragma unroll
            for (int k = 0; k < KV; ++k) {
              const auto &a = z[j][slot(2 * k, r)], &b = z[j][slot(2 * k + 1, r)];
              v4i x = v4i{(int)a[h], (int)a[h + 1], (int)b[h], (int)b[h + 1]};
              if (RING && (r & 1))
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] ^= zero;
              y[j] = mfma16<ELEM>(x, vf[k], y[j]);
            }
#pragma unroll
          for (int i = 0; i < 4; ++i) sum += y[j][i];
        }
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!__builtin_isfinite(sum)) != 0, 0)) {  // uniform
          // An infinity or NaN. The window's K-steps hold lines of other blocks too, and
          // 0 * x is not 0 there: the products again with all lines but the block's own
          // ones zero, so that a result depends on its block's lines alone, whatever the
          // schedule. (One product after the other: no registers of the step loop.)
          const int w0 = 16 * (F->v1[vlb] - NZ), lo = F->vlo[vlb] - w0, n_lines = F->vhi[vlb] - w0 - lo;
          auto next = [&]() {
            int at = lane;
            asm volatile("" : "+v"(at));
            __builtin_amdgcn_sched_barrier(0);
            return at;
          };
          // mask of word q of window step i: the lines inside the block's window (at: the lane)
          auto own = [&](int at, int i, int q) {
            const int t = (at >> 4 << 2) + (16 * i + 2 * (q & 1) - lo);  // the word's first line, from the block's first
            return ((uint32_t)t < (uint32_t)n_lines ? 0xFFFFu : 0u) |
                   ((uint32_t)(t + 1) < (uint32_t)n_lines ? 0xFFFF0000u : 0u);
          };
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            // a window that shifts: masked in place, since no later block reads a line
            // before this one's first; the last step's lines past the window are put back
            uint32_t last[ZW];
            if constexpr (!RING)
#pragma unroll
              for (int i = 0; i < NZ; ++i)
#pragma unroll
                for (int q = 0; q < ZW; ++q) {
                  if (i == NZ - 1) last[q] = z[j][i][q];
                  z[j][i][q] &= own(next(), i, q);
                }
            y[j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int h = 2; h >= 0; h -= 2)
#pragma unroll
              for (int k = 0; k < KV; ++k) {
                const int at = next();
                v4i x;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  const int i = 2 * k + (e >> 1);
                  x[e] = (int)z[j][slot(i, r)][h + (e & 1)];
                  if constexpr (RING) x[e] &= (int)own(at, i, e & 1);
                }
                y[j] = mfma16<ELEM>(x, vf[k], y[j]);
              }
            if constexpr (!RING)
#pragma unroll
              for (int q = 0; q < ZW; ++q) z[j][NZ - 1][q] = last[q];
          }
        }
        store(S, B, y);
      }
      ++B;
      if (++vlb == nv) {
        vlb = 0;
        vper += psteps;
      }
      fire = __builtin_amdgcn_readlane(v1tab, vlb) + vper;
    };

    // staging buffers after the vertical coefficients and biases
    uint8_t* xs[2] = {lds + F->lds_x, lds + F->lds_x + strip_stage(W)};
    commit<EDGE>(pre[0], first[0], xs[0]);
    issue<EDGE>(S, s0 + D, pre[0], first[0]);
    lds_barrier();  // step s0 staged, the vertical coefficients in place
    const int M = s1 - s0;
    // Whole rounds of U steps, the ones past the segment without products: an
    // exit from inside a round would reach the loop head, as the compiler lays
    // it out, on a path with another load newest, and make every wait there
    // drain the loads in flight.
    for (int m = 0; m < M; m += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        constexpr int last = NZ - 1;
        const int slot = RING ? u : last;
        commit<EDGE>(pre[(u + 1) % D], first[(u + 1) % D], xs[(u + 1) & 1]);
        issue<EDGE>(S, s0 + m + u + 1 + D, pre[(u + 1) % D], first[(u + 1) % D]);
        if (m + u < M) {  // uniform
          // horizontal products of step m + u
          v4i acc[NB];
          v4f accf[NB];
          v4i a[NB][KH];
#pragma unroll
          for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int k = 0; k < KH; ++k) a[j][k] = *reinterpret_cast<const v4i*>(xs[u & 1] + aoff[j][k]);
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            if constexpr (ELEM == kU8) {
              acc[j] = hq;
              if constexpr (SPLIT) {
                v4i hi = v4i{0, 0, 0, 0};
#pragma unroll
                for (int k = 0; k < KH; ++k) hi = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[j][k], bfh[j][k], hi, 0, 0, 0);
                acc[j] = hi * 128 + hq;
              }
#pragma unroll
              for (int k = 0; k < KH; ++k) acc[j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[j][k], bf[j][k], acc[j], 0, 0, 0);
            } else {
              accf[j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int k = 0; k < KH; ++k) accf[j] = mfma16<ELEM>(a[j][k], bf[j][k], accf[j]);
            }
          }
          // into the window
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            if constexpr (!RING) {
#pragma unroll
              for (int i = 0; i < last; ++i)
#pragma unroll
                for (int q = 0; q < ZW; ++q) z[j][i][q] = z[j][i + 1][q];
            }
            if constexpr (ELEM == kU8) {
              if constexpr (!UB) acc[j] = acc[j] + hb[j];
              z[j][slot][0] = quant4(acc[j]) ^ 0x80808080u;  // signed bytes z - 128, the vertical operand
            } else {
              // hi = round(z), lo = round(z - hi)
              const v4f r = accf[j];
              const uint32_t h01 = pack2<ELEM>(r[0], r[1]), h23 = pack2<ELEM>(r[2], r[3]);
              z[j][slot][0] = h01;
              z[j][slot][1] = h23;
              z[j][slot][2] = pack2<ELEM>(r[0] - lo16<ELEM>(h01), r[1] - hi16<ELEM>(h01));
              z[j][slot][3] = pack2<ELEM>(r[2] - lo16<ELEM>(h23), r[3] - hi16<ELEM>(h23));
            }
          }
          while (B < B1 && fire == m + u + 1) vblock(RING ? (u + 1) % NZ : 0);
        }
        lds_barrier();  // every wave is done with step m + u, the next one is staged
      }
    }
  }

  // Register slot of window step i where the ring starts at r.
  static __device__ __forceinline__ int slot(int i, int r) { return RING ? (i + r) % NZ : i; }

  // The vertical operand of K-step k (integer form): four steps' words.
  static __device__ __forceinline__ v4i zop8(const uint32_t (&w)[NZ][ELEM == kU8 ? 1 : 4], int k) {
    return v4i{(int)w[4 * k][0], (int)w[4 * k + 1][0], (int)w[4 * k + 2][0], (int)w[4 * k + 3][0]};
  }
};

// One workgroup's share: wnb strips of one stream from wb0 and one segment.
// EDGES: an instance for launches with a line that is not whole chunks.
template <int ELEM, bool SPLIT, int KH, int KV, int NB, int W, int D, bool EDGES>
__device__ __forceinline__ void strip_body(const StripStream& S, cfilt_t F, gsrc_t src, gdst_t dst, int wb0, int wnb,
                                           int B0, int B1, uint8_t* lds) {
  static_assert(kStripMaxBlocks * 16 <= 64 * W, "a thread copies one bias");
  Strip<ELEM, SPLIT, KH, KV, NB, W, D> T;
  T.tid = threadIdx.x;
  T.src = src;
  T.dst = dst;
  T.B0 = B0;
  T.B1 = B1;
  const v4i vf0 = ((const STRIP_GLOBAL v4i*)(uint64_t)F->vfrag)[min(T.tid, F->vfrag_bytes / 16 - 1)];
  int vb0 = 0;
  if constexpr (ELEM == kU8)
    vb0 = ((const STRIP_GLOBAL int32_t*)(uint64_t)F->bias)[kStripMaxBlocks * 16 + min(T.tid, kStripMaxBlocks * 16 - 1)];
  const int edge = T.setup(S, F, wb0, wnb);
  // (the paths that few workgroups take add the biases per column always)
  if constexpr (EDGES) {
    if (edge == kJoin) {
      T.template run<kJoin, false>(S, F, lds, vf0, vb0);
      return;
    }
    if (edge == kGather) {
      T.template run<kGather, false>(S, F, lds, vf0, vb0);
      return;
    }
  }
  if (ELEM != kU8 || F->ubias) T.template run<kWhole, true>(S, F, lds, vf0, vb0);
  else T.template run<kWhole, false>(S, F, lds, vf0, vb0);
}

}  // namespace

}  // namespace aol
