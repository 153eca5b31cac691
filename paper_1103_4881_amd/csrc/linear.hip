// Array-OL repetition with a linear integer elementary task (uint8 arrays),
// for gfx950.
//
// Sec. III: the application reads 24-bit RGB frames, filters their colour
// components and composes the output frame from the colour-space results;
// Sec. III-A and its tiler footnote: each step is a repetitive task whose
// input tiler cuts pattern element i of repetition r out of A at
// (o + P.r + F.i) mod S and whose output tiler writes result element j to B
// at (o' + P'.r + F'.j) mod S'. Here the elementary task is linear with
// integer weights:
//
//   y[j] = clamp(floor((sum_i W[j][i] x[i] + bias[j] + 128) / 256), 0, 255)
//
// which covers interleaved-RGB <-> planar colour conversions (3 -> 3),
// non-separable 2-D filters with several outputs per repetition (a 2-D
// polyphase downscale: span x span -> p x p) and box filters.
//
// Threads run along the last repetition dimension. The pattern offsets and
// weights are the same for every thread and come through scalar loads;
// pairs of pattern elements are multiplied
// with v_dot2_i32_i16 (two exact 16-bit products per instruction into an
// int32 accumulator, exact under the host's bound on sum |W| * 255).
// Patterns that stay inside the array use constant flat offsets; a point
// whose pattern crosses a border wraps each axis. For small patterns a staged
// form reads each chunk of a row's input from LDS, loaded with 16-byte loads,
// and stores dense output ranges from LDS the same way (byte-wide global
// accesses were its limit). Colour conversions of whole frames have a packed
// form without LDS, patterns of many elements a matrix-core form.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "linear.h"

namespace aol {

namespace {

typedef short v2s __attribute__((ext_vector_type(2)));
#define LIN_CONST __attribute__((address_space(4)))
typedef const LIN_CONST int32_t* ctab_t;
typedef const __attribute__((address_space(1))) uint8_t* lin_in_t;
typedef __attribute__((address_space(1))) uint8_t* lin_out_t;

}  // namespace

// Points xb + threadIdx.x, + kLinThreads, ... below xe of the repetition
// row r (every index but the last), point by point: each thread advances its
// wrapped input and output base points by a constant per step; a point whose
// pattern stays inside the array uses constant flat offsets, one that crosses
// a border wraps each axis.
template <int NOUT>
__device__ __forceinline__ void linear_points(const LinearArgs& a, const int (&r0)[kLinRank], int xb, int xe,
                                              int rot = 0) {
  const int last = a.rr - 1;
  int r[kLinRank];
#pragma unroll
  for (int k = 0; k < kLinRank; ++k) r[k] = r0[k];
  r[last] = xb + (int)threadIdx.x + rot;  // rot: only with xb = 0 and one point per thread
  if (r[last] >= a.R[last]) r[last] -= a.R[last];
  // wrapped base points of the thread's first point, input and output
  int b[kLinRank] = {0, 0, 0, 0}, ob[kLinRank] = {0, 0, 0, 0};
#pragma unroll
  for (int d = 0; d < kLinRank; ++d) {
    if (d < a.ra) {
      int64_t v = a.o[d];
#pragma unroll
      for (int k = 0; k < kLinRank; ++k)
        if (k < a.rr) v += (int64_t)a.P[d][k] * r[k];
      b[d] = (int)(v % a.S[d]);
    }
    if (d < a.ro) {
      int64_t v = a.oo[d];
#pragma unroll
      for (int k = 0; k < kLinRank; ++k)
        if (k < a.rr) v += (int64_t)a.Po[d][k] * r[k];
      ob[d] = (int)(v % a.So[d]);
    }
  }
  const ctab_t tab = (ctab_t)a.tab;
  const ctab_t ioff = tab;
  const ctab_t ifd = tab + a.t_ifd;
  const ctab_t wpair = tab + a.t_w;
  const ctab_t ooff = tab + a.t_ooff;
  const ctab_t ofd = tab + a.t_ofd;
  const int n2 = 2 * a.n_pairs;
  const lin_in_t in = (lin_in_t)a.in;
  const lin_out_t out = (lin_out_t)a.out;

  // (coordinates and offsets are below 2^31, the sum of two below 2^32)
  auto wrap = [](int c, int step, int S) {
    uint32_t v = (uint32_t)c + (uint32_t)step;
    if (v >= (uint32_t)S) v -= (uint32_t)S;
    return (int)v;
  };

  for (uint32_t rl = (uint32_t)xb + threadIdx.x; rl < (uint32_t)xe; rl += kLinThreads) {
    bool inside = true, oinside = true;
    int flat = 0, oflat = 0;
#pragma unroll
    for (int d = 0; d < kLinRank; ++d) {
      if (d < a.ra) {
        inside = inside && b[d] >= -a.lo[d] && b[d] < a.S[d] - a.hi[d];
        flat += b[d] * a.st[d];
      }
      if (d < a.ro) {
        oinside = oinside && ob[d] >= -a.olo[d] && ob[d] < a.So[d] - a.ohi[d];
        oflat += ob[d] * a.sto[d];
      }
    }
    auto wrapped = [&](int i) -> uint32_t {
      int f = 0;
#pragma unroll
      for (int d = 0; d < kLinRank; ++d) {
        if (d < a.ra) f += wrap(b[d], ifd[d * n2 + i], a.S[d]) * a.st[d];  // both in [0, S)
      }
      return in[f];
    };
    int acc[NOUT];
#pragma unroll
    for (int j = 0; j < NOUT; ++j) acc[j] = tab[a.t_bias + j];
    auto madd = [&](int k, uint32_t x) {
      const v2s xv = __builtin_bit_cast(v2s, x);
#pragma unroll
      for (int j = 0; j < NOUT; ++j)
        acc[j] = __builtin_amdgcn_sdot2(xv, __builtin_bit_cast(v2s, wpair[k * NOUT + j]), acc[j], false);
    };
    if (inside) {  // the usual case: constant flat offsets, four pairs of loads in flight
      int k = 0;
      for (; k + 4 <= a.n_pairs; k += 4) {
        uint32_t x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = in[flat + ioff[2 * (k + u)]] | ((uint32_t)in[flat + ioff[2 * (k + u) + 1]] << 16);
#pragma unroll
        for (int u = 0; u < 4; ++u) madd(k + u, x[u]);
      }
      for (; k < a.n_pairs; ++k) madd(k, in[flat + ioff[2 * k]] | ((uint32_t)in[flat + ioff[2 * k + 1]] << 16));
    } else {
      for (int k = 0; k < a.n_pairs; ++k) madd(k, wrapped(2 * k) | (wrapped(2 * k + 1) << 16));
    }
#pragma unroll
    for (int j = 0; j < NOUT; ++j) {
      if (j >= a.n_out) continue;  // uniform
      int f = oflat + ooff[j];
      if (!oinside) {
        f = 0;
#pragma unroll
        for (int d = 0; d < kLinRank; ++d) {
          if (d < a.ro) f += wrap(ob[d], ofd[d * NOUT + j], a.So[d]) * a.sto[d];
        }
      }
      out[f] = (uint8_t)min(max(acc[j] >> 8, 0), 255);  // arithmetic shift: floor division by 256
    }
    // next point of the thread along the last repetition dimension
#pragma unroll
    for (int d = 0; d < kLinRank; ++d) {
      if (d < a.ra) b[d] = wrap(b[d], a.inc[d], a.S[d]);
      if (d < a.ro) ob[d] = wrap(ob[d], a.oinc[d], a.So[d]);
    }
  }
}

// the repetition row of workgroup-row index `row` (every index but the last)
__device__ __forceinline__ void linear_row(const LinearArgs& a, uint32_t row, int (&r)[kLinRank]) {
  const int last = a.rr - 1;
#pragma unroll
  for (int k = kLinRank - 1; k >= 0; --k) {
    r[k] = 0;
    if (k < last) {
      r[k] = (int)(row % (uint32_t)a.R[k]);
      row /= (uint32_t)a.R[k];
    }
  }
}

// floor(n / d) for n, d < 2^31 from m = floor(2^32 / d) + 1 (the product's
// high word is the quotient or one more)
__device__ __forceinline__ uint32_t lin_div(uint32_t n, uint32_t d, uint32_t m) {
  if (d == 1) return n;  // m would be 2^32 + 1
  const uint32_t q = __umulhi(n, m);
  return q * d > n ? q - 1 : q;
}

// One workgroup per row of the repetition space; thread l takes the row's
// points l, l + 256, ...
template <int NOUT>
__global__ __launch_bounds__(kLinThreads) void k_linear(LinearArgs a) {
  int r[kLinRank];
  linear_row(a, blockIdx.x, r);
  linear_points<NOUT>(a, r, 0, a.R[a.rr - 1], a.rot);  // no barrier in this kernel
}

// The staged form (one workgroup per chunk of C = kLinThreads * ppt points of
// a row; see LinearStage). A chunk whose points all keep their whole input
// and output patterns inside the arrays, with no coordinate wrapping between
// its first and last point (a uniform test of the two ends per axis), reads
// its input ranges from LDS and writes dense output ranges through LDS; any
// other chunk runs point by point. Same arithmetic either way.
template <int NOUT>
__global__ __launch_bounds__(kLinThreads) void k_linear_staged(LinearArgs a, LinearStage st) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  typedef int v4i __attribute__((ext_vector_type(4)));
  const int last = a.rr - 1;
  const int tid = threadIdx.x;
  const uint32_t rowi = lin_div(blockIdx.x, (uint32_t)st.chunks, st.mg_R[last]);
  const int chunk = (int)(blockIdx.x - rowi * (uint32_t)st.chunks);
  const int C = kLinThreads * st.ppt;
  const int x0 = chunk * C;
  const int npts = min(C, a.R[last] - x0);  // uniform, >= 1
  const ctab_t tab = (ctab_t)a.tab;
  // the chunk's flat input and output positions of its first point, or -1:
  // not clean (computed on the host)
  const int flat0 = tab[st.cq + 2 * blockIdx.x], oflat0 = tab[st.cq + 2 * blockIdx.x + 1];
  const bool clean = flat0 >= 0;
  if (!clean) {  // uniform
    int r[kLinRank] = {0, 0, 0, 0};
    uint32_t row = rowi;
#pragma unroll
    for (int k = kLinRank - 1; k >= 0; --k) {
      if (k < last) {
        const uint32_t q = lin_div(row, (uint32_t)a.R[k], st.mg_R[k]);
        r[k] = (int)(row - q * (uint32_t)a.R[k]);
        row = q;
      }
    }
    linear_points<NOUT>(a, r, x0, x0 + npts);
    return;
  }
  const lin_in_t in = (lin_in_t)a.in;
  const lin_out_t out = (lin_out_t)a.out;
  const ctab_t grp = tab + st.t_grp;
  const ctab_t wpair = tab + a.t_w;
  // ---- the chunk's input ranges into LDS, 16-byte chunks aligned as in
  // memory: the byte at flat position F of group g sits at LDS gl[g] - A_g + F,
  // A_g the group's first position rounded down to 16 (every position the
  // chunk reads lies inside the array)
#pragma unroll
  for (int g = 0; g < kLinGroups; ++g) {
    if (g < st.ng) {
      const int start = flat0 + st.gb[g];
      const int end = start + (npts - 1) * st.P + st.gs[g];
      const int A = start & ~15;
      const int nch = (end - A + 15) >> 4;
      for (int c = tid; c < nch; c += kLinThreads) {
        const int F = A + 16 * c;
        v4i v;
        if ((int64_t)F + 16 <= st.n_in) {
          v = *(const __attribute__((address_space(1))) v4i*)(in + F);
        } else {  // the array's last chunk: its bytes only
          uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
          for (int q = 0; q < 16; ++q)
            if (F + q < st.n_in) w[q >> 2] |= (uint32_t)in[F + q] << (8 * (q & 3));
          v = v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
        }
        *reinterpret_cast<v4i*>(lds + st.gl[g] + 16 * c) = v;
      }
    }
  }
  // ---- per element, its LDS position for the chunk's first point: etab[e]
  // (inputs), otab[j] (outputs staged in LDS) or the output's flat position
  int* etab = reinterpret_cast<int*>(lds);
  int* otab = etab + 2 * a.n_pairs;
  for (int e = tid; e < 2 * a.n_pairs + NOUT; e += kLinThreads) {
    if (e < 2 * a.n_pairs) {
      const int g = tab[st.t_eg + e];
      etab[e] = grp[4 * g + 1] - ((flat0 + grp[4 * g]) & ~15) + flat0 + tab[e];
    } else {
      const int j = e - 2 * a.n_pairs;
      const int g = tab[st.t_og + j];
      otab[j] = st.ngo > 0 ? grp[4 * g + 3] - ((oflat0 + grp[4 * g + 2]) & ~15) + oflat0 + tab[a.t_ooff + j]
                           : oflat0 + tab[a.t_ooff + j];
    }
  }
  __syncthreads();
  // ---- the points: point x0 + i reads etab[e] + i * P (one range: the
  // range's LDS base + ioff[e] + i * P), writes otab[j] + i * Po. A pass
  // takes PP points per thread (i, i + 256, ...), so each pair's offsets and
  // weights (scalar loads) serve PP points; a point past the chunk reads
  // position 0 and writes nothing.
  constexpr int PP = NOUT <= 2 ? 8 : NOUT <= 4 ? 4 : NOUT <= 8 ? 2 : 1;
  const int in_base1 = st.gl[0] - ((flat0 + st.gb[0]) & ~15) + flat0;
  for (int i0 = tid; i0 < npts; i0 += PP * kLinThreads) {
    int di[PP];
    bool ok[PP];
#pragma unroll
    for (int p = 0; p < PP; ++p) {
      const int i = i0 + p * kLinThreads;
      ok[p] = i < npts;
      di[p] = ok[p] ? i * st.P : 0;
    }
    int acc[PP][NOUT];
#pragma unroll
    for (int j = 0; j < NOUT; ++j) {
      const int bj = tab[a.t_bias + j];
#pragma unroll
      for (int p = 0; p < PP; ++p) acc[p][j] = bj;
    }
    auto madd = [&](int k, const uint32_t (&x)[PP]) {
#pragma unroll
      for (int j = 0; j < NOUT; ++j) {
        const v2s w = __builtin_bit_cast(v2s, wpair[k * NOUT + j]);
#pragma unroll
        for (int p = 0; p < PP; ++p) acc[p][j] = __builtin_amdgcn_sdot2(__builtin_bit_cast(v2s, x[p]), w, acc[p][j], false);
      }
    };
    for (int k = 0; k < a.n_pairs; ++k) {
      int e0, e1;
      if (st.ng == 1) {  // uniform: one range, the element offsets straight from the table
        e0 = in_base1 + tab[2 * k];
        e1 = in_base1 + tab[2 * k + 1];
      } else {
        const int2 e = reinterpret_cast<const int2*>(etab)[k];  // the same for every lane
        e0 = e.x;
        e1 = e.y;
      }
      uint32_t x[PP];
#pragma unroll
      for (int p = 0; p < PP; ++p) x[p] = (uint32_t)lds[e0 + di[p]] | ((uint32_t)lds[e1 + di[p]] << 16);
      madd(k, x);
    }
#pragma unroll
    for (int p = 0; p < PP; ++p) {
      if (!ok[p]) continue;
      const int dout = (i0 + p * kLinThreads) * st.Po;
#pragma unroll
      for (int j = 0; j < NOUT; ++j) {
        if (j >= a.n_out) continue;  // uniform
        const uint8_t y = (uint8_t)min(max(acc[p][j] >> 8, 0), 255);
        if (st.ngo > 0) lds[otab[j] + dout] = y;
        else out[otab[j] + dout] = y;
      }
    }
  }
  if (st.ngo == 0) return;  // uniform
  __syncthreads();
  // ---- the chunk's output ranges, whole aligned 16-byte chunks where they lie inside
#pragma unroll
  for (int g = 0; g < kLinGroups; ++g) {
    if (g < st.ngo) {
      const int S0 = oflat0 + st.ob[g], E0 = S0 + npts * st.Po;
      const int OA = S0 & ~15;
      const int nch = (E0 - OA + 15) >> 4;
      for (int c = tid; c < nch; c += kLinThreads) {
        const int F = OA + 16 * c;
        const uint8_t* src = lds + st.ol[g] + 16 * c;
        if (F >= S0 && F + 16 <= E0) {
          *(__attribute__((address_space(1))) v4i*)(out + F) = *reinterpret_cast<const v4i*>(src);
        } else {
          for (int q = max(F, S0); q < min(F + 16, E0); ++q) out[q] = src[q - F];
        }
      }
    }
  }
}

// Packed form (see LinearPack): a thread takes 16 consecutive points, whole
// 16-byte loads and stores at any address, the points' bytes taken from and
// put into registers by byte permutes at constant selectors. What bounds it:
// memory; a point costs about 14 vector instructions. The staged form spent
// seven byte-wide LDS accesses per point. 30 frames of 1920x1080 RGB to planar:
// 0.171 -> 0.067 ms, 5.6 TB/s, the rate of a large copy.
template <int SI, int NI, int SO, int NO>
__global__ __launch_bounds__(kLinThreads) void k_linear_pack(LinearArgs a, LinearPack pk) {
  typedef int v4i __attribute__((ext_vector_type(4)));
  typedef int v4i_any __attribute__((ext_vector_type(4), aligned(1)));
  constexpr int QI = SI * NI, QO = SO * NO, PT = kLinPackPoints;
  static_assert(QI == 3 && QO == 3, "two pairs of input bytes per point");
  uint32_t run = lin_div(blockIdx.x, (uint32_t)pk.groups, pk.mg_groups);
  const int x = ((int)(blockIdx.x - run * (uint32_t)pk.groups) * kLinThreads + (int)threadIdx.x) * PT;
  if (x >= pk.len) return;
  int64_t in0 = 0, out0 = 0;  // uniform: the run's positions
#pragma unroll
  for (int k = kLinRank - 1; k >= 0; --k) {
    if (k < pk.n_outer) {
      const uint32_t q = lin_div(run, (uint32_t)pk.R[k], pk.mg_R[k]);
      const int64_t r = (int64_t)(run - q * (uint32_t)pk.R[k]);
      in0 += r * pk.fi[k];
      out0 += r * pk.fo[k];
      run = q;
    }
  }
  const lin_in_t in = (lin_in_t)a.in + in0;
  const lin_out_t out = (lin_out_t)a.out + out0;
  const int left = pk.len - x;  // points of the thread inside the run
  // byte b of stream s: d[s][b / 4], b = SI * point + byte
  uint32_t d[NI][4 * SI];
  if (left >= PT) {
#pragma unroll
    for (int s = 0; s < NI; ++s)
#pragma unroll
      for (int c = 0; c < SI; ++c) {
        const v4i v = *(const __attribute__((address_space(1))) v4i_any*)(in + pk.bi[s] + (int64_t)x * SI + 16 * c);
#pragma unroll
        for (int e = 0; e < 4; ++e) d[s][4 * c + e] = (uint32_t)v[e];
      }
  } else {  // the run's last points, byte by byte
#pragma unroll
    for (int s = 0; s < NI; ++s)
#pragma unroll
      for (int c = 0; c < 4 * SI; ++c) {
        d[s][c] = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (4 * c + e < left * SI) d[s][c] |= (uint32_t)in[pk.bi[s] + (int64_t)x * SI + 4 * c + e] << (8 * e);
      }
  }
  v2s w01[QO];
#pragma unroll
  for (int j = 0; j < QO; ++j)
    w01[j] = __builtin_bit_cast(v2s, (uint32_t)(pk.w[j][0] & 0xFFFF) | (uint32_t)pk.w[j][1] << 16);
  // results, output slot q of point t: byte SO * t + q % SO of stream q / SO
  uint32_t o[NO][4 * SO];
#pragma unroll
  for (int t4 = 0; t4 < PT; t4 += 4) {  // four points: one word per output slot
    uint32_t y[4][QO];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      auto byte_at = [&](int q) { return (t4 + t) * SI + q % SI; };  // slot q's byte in its stream
      const int b0 = byte_at(0), b1 = byte_at(1), b2 = byte_at(2);
      // the pair (slot 0, slot 1) as two 16-bit values, and slot 2
      const uint32_t x01 = __builtin_amdgcn_perm(d[1 / SI][b1 / 4], d[0][b0 / 4],
                                                 0x0c000c00u | (uint32_t)(b0 & 3) | (uint32_t)(4 + (b1 & 3)) << 16);
      const int x2 = (int)(d[2 / SI][b2 / 4] >> (8 * (b2 & 3)) & 0xFFu);
#pragma unroll
      for (int j = 0; j < QO; ++j) {
        int v = __builtin_amdgcn_sdot2(__builtin_bit_cast(v2s, x01), w01[j], pk.bias[j], false);
        v += __mul24(x2, pk.w[j][2]);
        y[t][j] = (uint32_t)min(max(v, 0), 65535);  // the result is byte 1
      }
    }
    if constexpr (SO == 1) {
#pragma unroll
      for (int j = 0; j < NO; ++j)
        o[j][t4 / 4] = __builtin_amdgcn_perm(y[1][j], y[0][j], 0x0c0c0501u) |
                       __builtin_amdgcn_perm(y[3][j], y[2][j], 0x05010c0cu);
    } else {
#pragma unroll
      for (int c = 0; c < SO; ++c) {  // bytes 4c .. 4c + 3 of the four points
        const uint32_t &p0 = y[4 * c / SO][4 * c % SO], &p1 = y[(4 * c + 1) / SO][(4 * c + 1) % SO],
                       &p2 = y[(4 * c + 2) / SO][(4 * c + 2) % SO], &p3 = y[(4 * c + 3) / SO][(4 * c + 3) % SO];
        o[0][t4 / 4 * SO + c] = __builtin_amdgcn_perm(p1, p0, 0x0c0c0501u) | __builtin_amdgcn_perm(p3, p2, 0x05010c0cu);
      }
    }
  }
  if (left >= PT) {
#pragma unroll
    for (int s = 0; s < NO; ++s)
#pragma unroll
      for (int c = 0; c < SO; ++c)
        *(__attribute__((address_space(1))) v4i_any*)(out + pk.bo[s] + (int64_t)x * SO + 16 * c) =
            v4i{(int)o[s][4 * c], (int)o[s][4 * c + 1], (int)o[s][4 * c + 2], (int)o[s][4 * c + 3]};
  } else {
#pragma unroll
    for (int s = 0; s < NO; ++s)
#pragma unroll
      for (int c = 0; c < 16 * SO; ++c)
        if (c < left * SO) out[pk.bo[s] + (int64_t)x * SO + c] = (uint8_t)(o[s][c / 4] >> (8 * (c & 3)));
  }
}

hipError_t linear_pack_launch(const LinearArgs& a, const LinearPack& p, hipStream_t stream) {
  int64_t blocks = p.groups;
  for (int k = 0; k < p.n_outer; ++k) blocks *= p.R[k];
  const dim3 grid((unsigned)blocks), block(kLinThreads);
  if (p.inst == 1) hipLaunchKernelGGL((k_linear_pack<3, 1, 1, 3>), grid, block, 0, stream, a, p);
  else hipLaunchKernelGGL((k_linear_pack<1, 3, 3, 1>), grid, block, 0, stream, a, p);
  return hipGetLastError();
}

// 16 bytes of LDS at a position that is a multiple of AL: aligned reads, since
// one 16-byte read across them takes several times as long.
template <int AL>
__device__ __forceinline__ int __attribute__((ext_vector_type(4))) lds_read16(const uint8_t* p) {
  typedef int v4i __attribute__((ext_vector_type(4)));
  typedef int v4i_any __attribute__((ext_vector_type(4), aligned(1)));
  if constexpr (AL >= 16) {
    return *reinterpret_cast<const v4i*>(p);
  } else if constexpr (AL == 8) {
    const int2 a = *reinterpret_cast<const int2*>(p), b = *reinterpret_cast<const int2*>(p + 8);
    return v4i{a.x, a.y, b.x, b.y};
  } else {
    return *reinterpret_cast<const v4i_any*>(p);
  }
}

// Bytes [s, s + 16) of the 32 bytes a, b (s in 0 .. 15, per lane).
__device__ __forceinline__ int __attribute__((ext_vector_type(4))) join16(
    int __attribute__((ext_vector_type(4))) a, int __attribute__((ext_vector_type(4))) b, int s) {
  typedef int v4i __attribute__((ext_vector_type(4)));
  uint32_t d[8] = {(uint32_t)a[0], (uint32_t)a[1], (uint32_t)a[2], (uint32_t)a[3],
                   (uint32_t)b[0], (uint32_t)b[1], (uint32_t)b[2], (uint32_t)b[3]};
  const uint32_t m8 = 0u - ((uint32_t)s >> 3 & 1u), m4 = 0u - ((uint32_t)s >> 2 & 1u);
#pragma unroll
  for (int i = 0; i < 6; ++i) d[i] = (d[i + 2] & m8) | (d[i] & ~m8);
#pragma unroll
  for (int i = 0; i < 5; ++i) d[i] = (d[i + 1] & m4) | (d[i] & ~m4);
  v4i r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = (int)__builtin_amdgcn_alignbyte(d[i + 1], d[i], (uint32_t)(s & 3));
  return r;
}

// Matrix-core form (see LinearBox). What bounds it: waits on memory, 58 % of the
// waves' cycles (the box, and each K-step's weights, which feed two products a
// part); vector instructions take 17 %, LDS 1 %, without bank conflicts. The
// point-by-point form spent two byte loads, a pack and n_out dot products per
// pair of elements and point on the vector units.
// 30 frames of 1920x1080, 17 x 17 elements to 3 x 3 outputs: 0.239 -> 0.059 ms
// (blocks of 64 x 4 points 0.062, 64 x 8 0.080, 32 x 16 0.089: small boxes keep
// more workgroups resident, and their set-up and loads overlap others' products).
template <bool SPLIT, int AL>
__global__ __launch_bounds__(kLinThreads) void k_linear_box(LinearArgs a, LinearBox bx) {
  typedef int v4i __attribute__((ext_vector_type(4)));
  typedef int v4i_any __attribute__((ext_vector_type(4), aligned(1)));
  typedef const __attribute__((address_space(1))) int32_t* gtab_t;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, n = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int last = a.rr - 1;
  const ctab_t tab = (ctab_t)a.tab;
  const gtab_t gtab = (gtab_t)a.tab;
  const lin_in_t in = (lin_in_t)a.in;
  const lin_out_t out = (lin_out_t)a.out;
  constexpr int PARTS = SPLIT ? 2 : 1;
  // the block's corner point, its box origin and its output base, wrapped
  int rl0 = 0, rj0 = 0, lo[kLinRank], ob0[kLinRank];
#pragma unroll
  for (int d = 0; d < kLinRank; ++d) {
    lo[d] = d < a.ra ? bx.org0[d] : 0;
    ob0[d] = d < a.ro ? bx.oorg0[d] : 0;
  }
  uint32_t blk = blockIdx.x;
#pragma unroll
  for (int k = kLinRank - 1; k >= 0; --k) {
    if (k < a.rr) {
      const uint32_t q = lin_div(blk, (uint32_t)bx.nb[k], bx.mg_nb[k]);
      const int i = (int)(blk - q * (uint32_t)bx.nb[k]);
      blk = q;
      if (k == last) rl0 = i * kLinBoxX;
      if (k == bx.k_loop) rj0 = i * kLinBoxY;
      const ctab_t t = tab + bx.t_org[k] + i * (a.ra + a.ro);
#pragma unroll
      for (int d = 0; d < kLinRank; ++d) {
        if (d < a.ra) {
          lo[d] += t[d];
          if (lo[d] >= a.S[d]) lo[d] -= a.S[d];
        }
        if (d < a.ro) {
          ob0[d] += t[a.ra + d];
          if (ob0[d] >= a.So[d]) ob0[d] -= a.So[d];
        }
      }
    }
  }
  // chunk offsets; the box rows' wrapped offsets (the weights are read from memory, the same for every workgroup)
  const __attribute__((address_space(1))) v4i* gw = (const __attribute__((address_space(1))) v4i*)(a.tab + bx.t_w);
  int* choff = reinterpret_cast<int*>(lds);
  int* roff = reinterpret_cast<int*>(lds + bx.lds_roff);
  uint8_t* box = lds + bx.lds_box;
  for (int q = tid; q < bx.rows; q += kLinThreads) {
    uint32_t rem = (uint32_t)q;
    int off = 0;
#pragma unroll
    for (int d = kLinRank - 2; d >= 0; --d) {
      if (d >= a.ra - 1) continue;
      const uint32_t up = lin_div(rem, (uint32_t)bx.bn[d], bx.mg_bn[d]);
      int c = lo[d] + (int)(rem - up * (uint32_t)bx.bn[d]);  // lo < S, extent <= 2 S: two subtractions wrap it
      rem = up;
      if (c >= a.S[d]) c -= a.S[d];
      if (c >= a.S[d]) c -= a.S[d];
      off += c * a.st[d];
    }
    roff[q] = off;
  }
  for (int i = tid; i < 4 * bx.steps; i += kLinThreads) choff[i] = gtab[bx.t_choff + i];
  __syncthreads();
  // The box, a 16-byte chunk of a row at a time, several loads in flight per
  // thread. A chunk that crosses the end of the axis is joined from the axis'
  // last 16 elements and its first 16; an axis shorter than that is gathered.
  const int S1 = a.S[a.ra - 1], lo1 = lo[a.ra - 1];
  const int total = bx.rows * bx.nch;
  constexpr int QB = 5;
  typedef const __attribute__((address_space(1))) v4i_any* chunk_t;
  for (int i0 = tid; i0 < total; i0 += QB * kLinThreads) {
    v4i v[QB], f[QB];
    int dst[QB], past[QB];
#pragma unroll
    for (int u = 0; u < QB; ++u) {
      const int i = min(i0 + u * kLinThreads, total - 1);  // past the end: the last chunk again
      const int row = (int)lin_div((uint32_t)i, (uint32_t)bx.nch, bx.mg_nch), c = i - row * bx.nch;
      int col = lo1 + 16 * c;
      if (col >= S1) col -= S1;
      if (col >= S1) col %= S1;
      dst[u] = row * bx.pitch + 16 * c;
      past[u] = max(col + 16 - S1, 0);
      const lin_in_t line = in + roff[row];
      if (S1 >= 16) {  // uniform
        v[u] = *(chunk_t)(line + (col - past[u]));
        f[u] = v[u];
        if (past[u]) f[u] = *(chunk_t)line;
      } else {
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll 1
        for (int q = 0; q < 16; ++q) {
#pragma unroll
          for (int e = 0; e < 3; ++e) w[e] = __builtin_amdgcn_alignbyte(w[e + 1], w[e], 1);
          w[3] = w[3] >> 8 | (uint32_t)line[col] << 24;
          col = col + 1 == S1 ? 0 : col + 1;
        }
        v[u] = f[u] = v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
        past[u] = 0;
      }
    }
#pragma unroll
    for (int u = 0; u < QB; ++u) {
      const v4i y = join16(v[u], f[u], past[u]);
      const int x = (int)0x80808080u;
      *reinterpret_cast<v4i*>(box + dst[u]) = v4i{y[0] ^ x, y[1] ^ x, y[2] ^ x, y[3] ^ x};
    }
  }
  __syncthreads();

  // wave w: the block's points with indices w, w + 4, ... along k_loop, in groups of 16 along the last dim
  constexpr int NG = kLinBoxX / 16, NW = kLinThreads / 64;
  v4i bias;
  int j0[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    bias[i] = gtab[bx.t_bias + 4 * g + i];
    j0[i] = gtab[a.t_ooff + min(4 * g + i, a.n_out - 1)];
  }
  for (int ly = wave; ly < kLinBoxY; ly += NW) {  // no barrier below
    if (bx.k_loop < 0 ? ly > 0 : rj0 + ly >= a.R[bx.k_loop]) return;
    const uint8_t* pb = box + ly * bx.jstep + n * bx.lstep;
    v4i acc[NG], hi[SPLIT ? NG : 1];
#pragma unroll
    for (int p = 0; p < NG; ++p) {
      acc[p] = bias;
      if constexpr (SPLIT) hi[p] = v4i{0, 0, 0, 0};
    }
    for (int k = 0; k < bx.steps; ++k) {
      const v4i w = gw[k * PARTS * 64 + lane];
      v4i wh;
      if constexpr (SPLIT) wh = gw[(k * PARTS + 1) * 64 + lane];
      const uint8_t* src = pb + choff[4 * k + g];
#pragma unroll
      for (int p = 0; p < NG; ++p) {
        const v4i x = lds_read16<AL>(src + 16 * p * bx.lstep);
        acc[p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w, x, acc[p], 0, 0, 0);
        if constexpr (SPLIT) hi[p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wh, x, hi[p], 0, 0, 0);
      }
    }
    // lane (g, n): outputs 4g .. 4g + 3 of point n of each group
#pragma unroll
    for (int p = 0; p < NG; ++p) {
      const int pl = 16 * p + n;
      if (rl0 + pl >= a.R[last]) continue;
      int ob[kLinRank], flat = 0;
      bool inside = true;
#pragma unroll
      for (int d = 0; d < kLinRank; ++d) {
        ob[d] = 0;
        if (d < a.ro) {
          int v = ob0[d] + bx.Pl[d] * pl + bx.Pj[d] * ly;
          if (v < 0) v += a.So[d];
          if (v >= a.So[d]) v -= a.So[d];
          ob[d] = v;
          inside = inside && v + a.olo[d] >= 0 && v + a.ohi[d] < a.So[d];
          flat += v * a.sto[d];
        }
      }
      v4i y = acc[p];
      if constexpr (SPLIT) y = y + hi[p] * 128;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (4 * g + i >= a.n_out) continue;
        int f = flat + j0[i];
        if (!inside) {
          f = 0;
#pragma unroll
          for (int d = 0; d < kLinRank; ++d) {
            if (d < a.ro) {
              int c = ob[d] + gtab[a.t_ofd + d * a.nout_pad + 4 * g + i];
              if (c >= a.So[d]) c -= a.So[d];
              f += c * a.sto[d];
            }
          }
        }
        out[f] = (uint8_t)(min(max(y[i], 0), 65535) >> 8);
      }
    }
  }
}

using LinearBoxFn = void (*)(LinearArgs, LinearBox);

static LinearBoxFn linear_box_pick(bool split, int align) {
  if (align >= 16) return split ? k_linear_box<true, 16> : k_linear_box<false, 16>;
  if (align == 8) return split ? k_linear_box<true, 8> : k_linear_box<false, 8>;
  return split ? k_linear_box<true, 1> : k_linear_box<false, 1>;
}

hipError_t linear_box_prepare(const LinearBox& b) {
  return hipFuncSetAttribute((const void*)linear_box_pick(b.split != 0, b.align),
                             hipFuncAttributeMaxDynamicSharedMemorySize, b.lds_bytes);
}

hipError_t linear_box_launch(const LinearArgs& a, const LinearBox& b, hipStream_t stream) {
  int64_t blocks = 1;
  for (int k = 0; k < a.rr; ++k) blocks *= b.nb[k];
  hipLaunchKernelGGL(linear_box_pick(b.split != 0, b.align), dim3((unsigned)blocks), dim3(kLinThreads),
                     (size_t)b.lds_bytes, stream, a, b);
  return hipGetLastError();
}

hipError_t linear_launch(int nout, const LinearArgs& a, hipStream_t stream) {
  const int64_t blocks = a.nrep / a.R[a.rr - 1];  // rows of the repetition space
  const dim3 grid((unsigned)blocks), block(kLinThreads);
  switch (nout) {
    case 1: hipLaunchKernelGGL(k_linear<1>, grid, block, 0, stream, a); break;
    case 2: hipLaunchKernelGGL(k_linear<2>, grid, block, 0, stream, a); break;
    case 3: hipLaunchKernelGGL(k_linear<3>, grid, block, 0, stream, a); break;
    case 4: hipLaunchKernelGGL(k_linear<4>, grid, block, 0, stream, a); break;
    case 6: hipLaunchKernelGGL(k_linear<6>, grid, block, 0, stream, a); break;
    case 8: hipLaunchKernelGGL(k_linear<8>, grid, block, 0, stream, a); break;
    case 9: hipLaunchKernelGGL(k_linear<9>, grid, block, 0, stream, a); break;
    case 12: hipLaunchKernelGGL(k_linear<12>, grid, block, 0, stream, a); break;
    default: hipLaunchKernelGGL(k_linear<16>, grid, block, 0, stream, a); break;
  }
  return hipGetLastError();
}

template <int NOUT>
static void staged_launch(const LinearArgs& a, const LinearStage& st, dim3 grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_linear_staged<NOUT>, grid, dim3(kLinThreads), (size_t)st.lds_bytes, stream, a, st);
}

hipError_t linear_staged_launch(int nout, const LinearArgs& a, const LinearStage& st, hipStream_t stream) {
  const int64_t rows = a.nrep / a.R[a.rr - 1];
  const dim3 grid((unsigned)(rows * st.chunks));
  switch (nout) {
    case 1: staged_launch<1>(a, st, grid, stream); break;
    case 2: staged_launch<2>(a, st, grid, stream); break;
    case 3: staged_launch<3>(a, st, grid, stream); break;
    case 4: staged_launch<4>(a, st, grid, stream); break;
    case 6: staged_launch<6>(a, st, grid, stream); break;
    case 8: staged_launch<8>(a, st, grid, stream); break;
    case 9: staged_launch<9>(a, st, grid, stream); break;
    case 12: staged_launch<12>(a, st, grid, stream); break;
    default: staged_launch<16>(a, st, grid, stream); break;
  }
  return hipGetLastError();
}

}  // namespace aol
