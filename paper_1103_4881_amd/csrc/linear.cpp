// Host side of the Array-OL repetition with a linear integer elementary task:
// tiler validation, the output tiler's exact-coverage check, pattern tables.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "aolmi.h"
#include "common.h"
#include "linear.h"

using namespace aol;

struct aol_linear_plan {
  LinearArgs args{};
  LinearStage stage{};  // staged form (stage.ppt == 0: not available)
  LinearBox box{};      // matrix-core form (box.use == 0: not available)
  LinearPack pack{};    // packed form (pack.inst == 0: not available)
  int nout = 1;  // kernel instance: output pattern elements rounded up to 1, 2, 3, 4, 6, 8, 9, 12 or 16
  DeviceBuf d_tab;
};

namespace {

// floor(2^32 / d) + 1 (the kernel's division by d; d == 1 is special-cased there)
uint32_t magic(uint32_t d) { return d <= 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) / d) + 1); }

int64_t pmod64(int64_t a, int64_t m) {
  const int64_t r = a % m;
  return r < 0 ? r + m : r;
}

int64_t count(const int64_t* shape, int rank) {
  int64_t n = 1;
  for (int k = 0; k < rank; ++k) n *= shape[k];
  return n;
}

aol_status check_tiler(const aol_tiler* t, const char* name, int max_pat) {
  if (!t) return fail(AOL_ERR_INVALID, "%s: NULL tiler", name);
  if (t->array_rank < 1 || t->rep_rank < 1 || t->pat_rank < 0)
    return fail(AOL_ERR_INVALID, "%s: ranks must be >= 1 (pattern >= 0)", name);
  if (t->array_rank > AOL_MAX_RANK || t->rep_rank > AOL_MAX_RANK || t->pat_rank > AOL_MAX_RANK)
    return fail(AOL_ERR_UNSUPPORTED, "%s: ranks above %d", name, AOL_MAX_RANK);
  int64_t n = 1;
  for (int d = 0; d < t->array_rank; ++d) {
    if (t->array_shape[d] < 1) return fail(AOL_ERR_INVALID, "%s: array_shape[%d] < 1", name, d);
    n *= t->array_shape[d];
    if (n >= (1LL << 31)) return fail(AOL_ERR_UNSUPPORTED, "%s: arrays of 2^31 elements or more", name);
  }
  int64_t nr = 1;
  for (int k = 0; k < t->rep_rank; ++k) {
    if (t->rep_shape[k] < 1) return fail(AOL_ERR_INVALID, "%s: rep_shape[%d] < 1", name, k);
    nr *= t->rep_shape[k];
    if (nr >= (1LL << 31)) return fail(AOL_ERR_UNSUPPORTED, "%s: repetition spaces of 2^31 points or more", name);
  }
  int64_t np = 1;
  for (int b = 0; b < t->pat_rank; ++b) {
    if (t->pat_shape[b] < 1) return fail(AOL_ERR_INVALID, "%s: pat_shape[%d] < 1", name, b);
    np *= t->pat_shape[b];
    if (np > max_pat) return fail(AOL_ERR_UNSUPPORTED, "%s: patterns of more than %d elements", name, max_pat);
  }
  return AOL_OK;
}

// Pattern element i of tiler t: its fitting offset along each array dim.
void fitting_offsets(const aol_tiler* t, int i, int64_t* f) {
  int64_t idx[AOL_MAX_RANK] = {0, 0, 0, 0};
  int rem = i;
  for (int b = t->pat_rank - 1; b >= 0; --b) {
    idx[b] = rem % t->pat_shape[b];
    rem /= (int)t->pat_shape[b];
  }
  for (int d = 0; d < t->array_rank; ++d) {
    f[d] = 0;
    for (int b = 0; b < t->pat_rank; ++b) f[d] += t->fitting[d][b] * idx[b];
  }
}

// One side (input or output) of the launch arguments: shape, strides,
// origin and paving reduced mod the shape, the extents of the pattern's
// offsets (patterns inside the array use flat offsets: a pattern longer than
// an axis always takes the wrapping path), the per-thread step along the last
// repetition dim; fills the flat and per-dim offset tables.
void side(const aol_tiler* t, int n_pat, int n_pad, int32_t* S, int32_t* st, int32_t* o, int32_t (*P)[kLinRank],
          int32_t* lo, int32_t* hi, int32_t* inc, std::vector<int32_t>& off, std::vector<int32_t>& fd) {
  const int ra = t->array_rank, rr = t->rep_rank;
  int64_t s = 1;
  for (int d = ra - 1; d >= 0; --d) {
    S[d] = (int32_t)t->array_shape[d];
    st[d] = (int32_t)s;
    s *= t->array_shape[d];
  }
  for (int d = 0; d < ra; ++d) {
    o[d] = (int32_t)pmod64(t->origin[d], S[d]);
    for (int k = 0; k < rr; ++k) P[d][k] = (int32_t)pmod64(t->paving[d][k], S[d]);
    inc[d] = (int32_t)pmod64((int64_t)kLinThreads * t->paving[d][rr - 1], S[d]);
    lo[d] = 0;
    hi[d] = 0;
  }
  off.assign((size_t)n_pad, 0);
  fd.assign((size_t)ra * n_pad, 0);
  for (int i = 0; i < n_pad; ++i) {
    int64_t f[AOL_MAX_RANK];
    fitting_offsets(t, i < n_pat ? i : 0, f);  // padding repeats element 0 (its weights are zero)
    int64_t flat = 0;
    for (int d = 0; d < ra; ++d) {
      if (f[d] <= -S[d] || f[d] >= S[d]) {  // longer than the axis: no point counts as inside
        lo[d] = -S[d];
        hi[d] = S[d];
      } else {
        lo[d] = (int32_t)std::min<int64_t>(lo[d], f[d]);
        hi[d] = (int32_t)std::max<int64_t>(hi[d], f[d]);
      }
      fd[(size_t)d * n_pad + i] = (int32_t)pmod64(f[d], S[d]);
      flat += std::max<int64_t>(std::min<int64_t>(f[d], S[d]), -S[d]) * st[d];
    }
    off[(size_t)i] = (int32_t)flat;
  }
}

// Groups of pattern offsets for the staged form: sorted distinct offsets,
// neighbours closer than `gap` share a group (their ranges over a chunk
// overlap or touch), then the closest groups merge until at most kLinGroups
// remain. Returns the groups as (least offset, extent).
std::vector<std::pair<int64_t, int64_t>> offset_groups(std::vector<int64_t> offs, int64_t gap) {
  std::sort(offs.begin(), offs.end());
  offs.erase(std::unique(offs.begin(), offs.end()), offs.end());
  std::vector<std::pair<int64_t, int64_t>> g;  // (first, last)
  for (int64_t o : offs) {
    if (!g.empty() && o - g.back().second <= gap) g.back().second = o;
    else g.push_back({o, o});
  }
  while (g.size() > (size_t)kLinGroups) {
    size_t best = 0;
    for (size_t k = 1; k + 1 < g.size(); ++k)
      if (g[k + 1].first - g[k].second < g[best + 1].first - g[best].second) best = k;
    g[best].second = g[best + 1].second;
    g.erase(g.begin() + (long)best + 1);
  }
  for (auto& x : g) x.second = x.second - x.first + 1;
  return g;
}

// Flat stride between consecutive points along the last repetition dim (the
// pavings reduced mod the shape, as the kernel walks them).
int64_t flat_stride(const int32_t* st, const int32_t (*P)[kLinRank], int rank, int last) {
  int64_t s = 0;
  for (int d = 0; d < rank; ++d) s += (int64_t)P[d][last] * st[d];
  return s;
}

// The staged form's layout for a plan, or ppt = 0 when it does not apply:
// at most kLinStageMaxIn input pattern elements, positive strides of at most
// 64 elements per point, arrays below 2^30 elements, the groups' LDS within
// kLinStageLds.
void plan_stage(const LinearArgs& a, int nout, const std::vector<int32_t>& ioff, const std::vector<int32_t>& ooff,
                int n_in, int n_out, LinearStage& st, std::vector<int32_t>& eg, std::vector<int32_t>& og) {
  memset(&st, 0, sizeof st);
  const int last = a.rr - 1;
  int64_t nin = 1, nout_el = 1;
  for (int d = 0; d < a.ra; ++d) nin *= a.S[d];
  for (int d = 0; d < a.ro; ++d) nout_el *= a.So[d];
  const int64_t P = flat_stride(a.st, a.P, a.ra, last), Po = flat_stride(a.sto, a.Po, a.ro, last);
  // Small patterns only: with many elements per point (a 17 x 17 window, nine
  // outputs) the point's own arithmetic and weight reads set the time, and
  // the point-by-point form measured faster (0.31 against 0.46 ms on 30
  // frames of 1920 x 1080); with a handful (colour conversions) the staged
  // form is 1.6x faster.
  if (n_in > kLinStageMaxIn) return;
  if (P <= 0 || P > 64 || Po <= 0 || Po > 64 || nin >= (1LL << 30) || nout_el >= (1LL << 30)) return;
  // dense output groups: the sorted offsets in runs of Po consecutive ones
  std::vector<int64_t> os(ooff.begin(), ooff.begin() + n_out);
  std::sort(os.begin(), os.end());
  bool dense = n_out % Po == 0 && n_out / Po <= kLinGroups;
  for (int k = 0; dense && k < n_out; ++k) dense = os[k] == os[(k / Po) * Po] + k % Po;
  const int R = a.R[last];
  for (int ppt : {8, 4, 2, 1}) {
    if (ppt > 1 && kLinThreads * (ppt / 2) >= R) continue;  // no more points per thread than the row needs
    const int C = kLinThreads * ppt;
    std::vector<int64_t> is(ioff.begin(), ioff.begin() + n_in);
    auto groups = offset_groups(is, (int64_t)C * P);
    int lds = (4 * (2 * a.n_pairs + nout) + 15) / 16 * 16;  // the element tables
    LinearStage t;
    memset(&t, 0, sizeof t);
    t.ng = (int)groups.size();
    for (int g = 0; g < t.ng; ++g) {
      t.gb[g] = (int32_t)groups[g].first;
      t.gs[g] = (int32_t)groups[g].second;
      t.gl[g] = lds;
      lds += (int)((((int64_t)(C - 1) * P + groups[g].second + 30) / 16) * 16);
    }
    if (dense) {
      t.ngo = n_out / (int)Po;
      for (int g = 0; g < t.ngo; ++g) {
        t.ob[g] = (int32_t)os[(size_t)g * Po];
        t.ol[g] = lds;
        lds += (int)((((int64_t)C * Po + 30) / 16) * 16);
      }
    }
    if (lds > kLinStageLds) continue;
    t.ppt = ppt;
    t.chunks = (R + C - 1) / C;
    t.P = (int32_t)P;
    t.Po = (int32_t)Po;
    t.lds_bytes = lds;
    t.n_in = nin;
    t.n_out = nout_el;
    st = t;
    break;
  }
  if (!st.ppt) return;
  eg.assign((size_t)2 * a.n_pairs, 0);
  for (int i = 0; i < 2 * a.n_pairs; ++i) {
    const int64_t o = ioff[(size_t)i];
    for (int g = 0; g < st.ng; ++g)
      if (o >= st.gb[g] && o < (int64_t)st.gb[g] + st.gs[g]) eg[(size_t)i] = g;
  }
  og.assign((size_t)nout, 0);
  for (int j = 0; j < n_out && st.ngo; ++j)
    for (int g = 0; g < st.ngo; ++g)
      if (ooff[(size_t)j] >= st.ob[g] && ooff[(size_t)j] < (int64_t)st.ob[g] + Po) og[(size_t)j] = g;
}

// The packed form, or inst = 0 when it does not apply: no point's pattern
// leaves its array before the modulo, the last dim's flat strides and the
// pattern's bytes per point make one of kLinPacks' shapes, each stream's bytes
// in one order.
void plan_pack(const LinearArgs& a, const aol_tiler* in, const aol_tiler* out, const int16_t* weights,
               const int32_t* bias, int n_in, int n_out, LinearPack& p) {
  memset(&p, 0, sizeof p);
  if (n_in > kLinPackSlots || n_out > kLinPackSlots) return;
  const int last = a.rr - 1;
  // flat strides per repetition dim and flat origin, from the tilers' own (signed) numbers
  int64_t fs[2][kLinRank], base[2], off[2][kLinPackSlots];
  for (int side = 0; side < 2; ++side) {
    const aol_tiler* t = side ? out : in;
    const int np = side ? n_out : n_in;
    for (int k = 0; k < a.rr; ++k) fs[side][k] = 0;
    base[side] = 0;
    for (int i = 0; i < np; ++i) off[side][i] = 0;
    int64_t st = 1;
    for (int d = t->array_rank - 1; d >= 0; --d) {
      const int64_t S = t->array_shape[d], o = pmod64(t->origin[d], S);
      int64_t lo = o, hi = o, flo = 0, fhi = 0;
      for (int k = 0; k < a.rr; ++k) {
        if (t->paving[d][k] > S || t->paving[d][k] < -S) return;  // (the spans below stay far inside int64)
        const int64_t span = t->paving[d][k] * (t->rep_shape[k] - 1);
        (span < 0 ? lo : hi) += span;
        fs[side][k] += t->paving[d][k] * st;
      }
      for (int i = 0; i < np; ++i) {
        int64_t f[AOL_MAX_RANK];
        fitting_offsets(t, i, f);
        flo = std::min(flo, f[d]);
        fhi = std::max(fhi, f[d]);
        if (f[d] > S || f[d] < -S) return;
        off[side][i] += f[d] * st;
      }
      if (lo + flo < 0 || hi + fhi >= S) return;
      base[side] += o * st;
      st *= S;
    }
  }
  int slot[2][kLinPackSlots];
  for (int v = 0; v < 2 && !p.inst; ++v) {
    const LinearPackShape sh = kLinPacks[v];
    bool ok = fs[0][last] == sh.si && fs[1][last] == sh.so && n_in == sh.si * sh.ni && n_out == sh.so * sh.no;
    for (int side = 0; side < 2 && ok; ++side) {
      const int S = side ? sh.so : sh.si, np = side ? n_out : n_in;
      std::vector<std::pair<int64_t, int>> el;
      for (int i = 0; i < np; ++i) el.push_back({off[side][i], i});
      std::sort(el.begin(), el.end());
      for (int q = 0; q < np; ++q) {
        ok = ok && el[(size_t)q].first == el[(size_t)(q / S * S)].first + q % S;
        slot[side][el[(size_t)q].second] = q;
        if (q % S == 0) (side ? p.bo : p.bi)[q / S] = base[side] + el[(size_t)q].first;
      }
    }
    if (ok) p.inst = v + 1;
  }
  if (!p.inst) return;
  for (int j = 0; j < n_out; ++j) {
    for (int i = 0; i < n_in; ++i) p.w[slot[1][j]][slot[0][i]] = weights[(size_t)j * n_in + i];
    p.bias[slot[1][j]] = (bias ? bias[j] : 0) + 128;
  }
  // the run: the last dim, and those before it that continue it in both arrays
  int64_t len = a.R[last];
  int k = last - 1;
  while (k >= 0 && fs[0][k] == fs[0][last] * len && fs[1][k] == fs[1][last] * len && len * a.R[k] < (1LL << 30)) {
    len *= a.R[k];
    --k;
  }
  p.len = (int32_t)len;
  const int per = kLinThreads * kLinPackPoints;
  p.groups = (int32_t)((len + per - 1) / per);
  p.mg_groups = magic((uint32_t)p.groups);
  p.n_outer = k + 1;
  int64_t blocks = p.groups;
  for (int d = 0; d <= k; ++d) {
    p.R[d] = a.R[d];
    p.mg_R[d] = magic((uint32_t)a.R[d]);
    p.fi[d] = fs[0][d];
    p.fo[d] = fs[1][d];
    blocks *= a.R[d];
  }
  if (blocks >= (1LL << 24)) p.inst = 0;
}

// Whether the matrix-core form is the faster one: times in us estimated for it
// and for the point-by-point form, each the longer of what all its workgroups
// take on the whole device and of one workgroup's chain. Fitted to 2,753
// plans of 3,840 to 1,000,000 points (8 % off in the median): a product's K-step
// on chunks at any byte costs about as much as five pairs of elements point by
// point, so patterns with few elements per chunk and few outputs are slower as
// products (1000 x 1000 points, 33 x 1 elements, one output: nine K-steps 71 us,
// point by point 33; 6 x 6 elements, four outputs: 29 and 38; 17 x 17, nine
// outputs at 1/8: 59 and 239). Chosen with a tenth to spare: of those plans 19 are
// slower than the other form (9 % at most), 63 miss a gain (1.4 times at most).
bool box_pays(const LinearArgs& a, const LinearBox& b, const int32_t (&Ps)[kLinRank][kLinRank], int64_t blocks,
              int chunks) {
  const int last = a.rr - 1;
  const double kb = b.lds_bytes / 1024.0, mb = blocks * 256 / 1e6;
  const double step = (b.align < 8 ? 6.2 : 0.0) + (b.split ? 1.0 : 0.0);
  const double box = std::max({mb * (12.3 + 1.7 * kb + b.steps * step + 0.2 * a.n_out), mb * 29.0,
                               7.3 + 0.45 * b.steps + 0.1 * std::max(0.0, kb - 16)});
  // point by point: a workgroup per row, 256 points of it at a time; lanes `stride` bytes apart
  const int64_t rows = a.nrep / a.R[last], turns = (a.R[last] + kLinThreads - 1) / kLinThreads;
  if (rows >= (1LL << 24)) return true;  // (more rows than a grid holds)
  const double mp = (double)rows * turns * kLinThreads / 1e6;
  int64_t stride = 0;
  bool wraps = false;  // some point's pattern leaves the array: its wave computes every address
  for (int d = 0; d < a.ra; ++d) {
    stride += std::abs((int64_t)Ps[d][last]) * a.st[d];
    int64_t lo = (int64_t)a.o[d] + a.lo[d], hi = (int64_t)a.o[d] + a.hi[d];
    for (int k = 0; k < a.rr; ++k) (Ps[d][k] < 0 ? lo : hi) += (int64_t)Ps[d][k] * (a.R[k] - 1);
    wraps = wraps || lo < 0 || hi >= a.S[d];
  }
  const double far = (double)std::min<int64_t>(std::max<int64_t>(stride - 1, 0), 15);
  const double inner = 0.05 + 0.0022 * a.nout_pad, edge = 0.335 + 0.011 * a.nout_pad;
  const double points =
      std::max(mp * (a.n_pairs * (1.24 + 0.073 * a.nout_pad) + chunks * (0.09 + 0.24 * far) + 0.28 * a.nout_pad),
               6.0 + a.n_pairs * ((turns - 1) * inner + (wraps ? edge : inner)));
  return box < 0.9 * points;
}

// The matrix-core form's layout and tables (appended to tab), or use = 0 when
// it does not apply: more than kLinStageMaxIn pattern elements (smaller
// patterns have the staged form, or keep too little of a product busy), no two
// on one position and none reaching as far as an axis is long, axes of at most
// 2^30 (the kernel adds two coordinates in 32 bits), a box that fits
// kLinBoxLds and is no longer than twice an axis, at most
// kLinBoxSteps K-steps, weights within two int8 parts, and faster than point by
// point.
void plan_box(const LinearArgs& a, const aol_tiler* in, const int16_t* weights, const int32_t* bias, int n_in,
              int n_out, LinearBox& b, std::vector<int32_t>& tab) {
  memset(&b, 0, sizeof b);
  const int last = a.rr - 1, last_d = a.ra - 1;
  if (n_in <= kLinStageMaxIn) return;
  for (int j = 0; j < n_out; ++j) {  // the sums over x - 128 stay in int32 too
    int64_t m = 128 + (bias ? std::abs((int64_t)bias[j]) : 0);
    for (int i = 0; i < n_in; ++i) m += 512 * std::abs((int64_t)weights[(size_t)j * n_in + i]);
    if (m >= (1LL << 31)) return;
  }
  for (int d = 0; d < a.ra; ++d)
    if (a.lo[d] <= -a.S[d] || a.hi[d] >= a.S[d] || a.S[d] > (1 << 30)) return;
  for (int d = 0; d < a.ro; ++d)
    if (a.So[d] > (1 << 30)) return;
  int32_t Ps[kLinRank][kLinRank];  // pavings, signed, nearest zero
  for (int d = 0; d < a.ra; ++d)
    for (int k = 0; k < a.rr; ++k) Ps[d][k] = (int64_t)a.P[d][k] * 2 > a.S[d] ? a.P[d][k] - a.S[d] : a.P[d][k];
  bool split = false;
  for (int64_t i = 0; i < (int64_t)n_in * n_out; ++i) {
    if (weights[i] < -128 || weights[i] > 127) split = true;
    if (weights[i] < -64 - 128 * 128 || weights[i] > 63 + 127 * 128) return;  // lo + 128 * hi, both int8
  }
  const int parts = split ? 2 : 1;
  // the other dim of a block: the one with the smallest box
  int64_t best = -1;
  for (int kj = -1; kj < last; ++kj) {
    if (kj < 0 && last > 0) continue;
    int64_t ext[kLinRank], lo[kLinRank], bytes = 1;
    bool fit = true;
    for (int d = 0; d < a.ra; ++d) {
      ext[d] = a.hi[d] - a.lo[d] + 1;
      lo[d] = a.lo[d];
      for (int k : {last, kj}) {
        if (k < 0) continue;
        const int64_t span = (int64_t)Ps[d][k] * (k == last ? kLinBoxX - 1 : kLinBoxY - 1);
        ext[d] += span < 0 ? -span : span;
        lo[d] += span < 0 ? span : 0;
      }
      fit = fit && ext[d] <= 2 * (int64_t)a.S[d];
      if (d == last_d) ext[d] = (ext[d] + 15) / 16 * 16;
      if (bytes * ext[d] > kLinBoxLds) fit = false;
      if (fit) bytes *= ext[d];
    }
    if (!fit || (best >= 0 && bytes >= best)) continue;
    best = bytes;
    b.k_loop = kj;
    for (int d = 0; d < a.ra; ++d) {
      b.bn[d] = (int32_t)ext[d];
      b.dlo[d] = (int32_t)pmod64(lo[d], a.S[d]);
    }
  }
  if (best < 0) return;
  const int kj = b.k_loop;
  b.pitch = b.bn[last_d];
  b.nch = b.pitch / 16;
  b.rows = (int32_t)(best / b.pitch);
  if ((int64_t)b.rows * b.nch >= 65536) return;
  int64_t bst[kLinRank], s1 = 1;
  for (int d = last_d; d >= 0; --d) {
    bst[d] = s1;
    s1 *= b.bn[d];
  }
  int64_t ls = 0, js = 0, corner = 0;  // corner: box position of the corner point's base
  for (int d = 0; d < a.ra; ++d) {
    ls += Ps[d][last] * bst[d];
    if (kj >= 0) js += Ps[d][kj] * bst[d];
    int64_t lo = a.lo[d];
    for (int k : {last, kj}) {
      if (k < 0) continue;
      const int64_t span = (int64_t)Ps[d][k] * (k == last ? kLinBoxX - 1 : kLinBoxY - 1);
      lo += span < 0 ? span : 0;
    }
    corner -= lo * bst[d];
  }
  b.lstep = (int32_t)ls;
  b.jstep = (int32_t)js;
  // chunks of 16 bytes that cover the pattern's elements, in order of position
  std::vector<std::pair<int64_t, int>> el((size_t)n_in);
  for (int i = 0; i < n_in; ++i) {
    int64_t f[AOL_MAX_RANK], o = corner;
    fitting_offsets(in, i, f);
    for (int d = 0; d < a.ra; ++d) o += f[d] * bst[d];
    el[(size_t)i] = {o, i};
  }
  std::sort(el.begin(), el.end());
  for (int i = 1; i < n_in; ++i)
    if (el[(size_t)i].first == el[(size_t)i - 1].first) return;
  std::vector<int64_t> chunks;
  std::vector<std::vector<std::pair<int, int>>> member;  // (byte of the chunk, element)
  for (const auto& e : el) {
    if (chunks.empty() || e.first >= chunks.back() + 16) {
      chunks.push_back(e.first);
      member.emplace_back();
    }
    member.back().push_back({(int)(e.first - chunks.back()), e.second});
  }
  b.steps = (int32_t)((chunks.size() + 3) / 4);
  if (b.steps > kLinBoxSteps) return;
  b.lds_roff = 4 * b.steps * 4;
  b.lds_box = (b.lds_roff + b.rows * 4 + 15) / 16 * 16;
  // (a chunk may reach 15 bytes past the box: weight zero there)
  b.lds_bytes = (int32_t)((b.lds_box + best + 16 + 15) / 16 * 16);
  if (b.lds_bytes > kLinBoxLds) return;
  int64_t blocks = 1, terms = 0;
  for (int k = 0; k < a.rr; ++k) {
    const int e = k == last ? kLinBoxX : k == kj ? kLinBoxY : 1;
    b.nb[k] = (a.R[k] + e - 1) / e;
    b.mg_nb[k] = magic((uint32_t)b.nb[k]);
    blocks *= b.nb[k];
    terms += (int64_t)b.nb[k] * (a.ra + a.ro);
  }
  if (blocks >= (1LL << 24) || terms > kLinCoordTable) return;
  b.align = 16;
  for (int64_t v : chunks)
    while (v % b.align) b.align /= 2;
  while (b.lstep % b.align || b.jstep % b.align) b.align /= 2;
  b.split = split ? 1 : 0;
  if (!box_pays(a, b, Ps, blocks, (int)chunks.size())) return;
  // weights in lane order: lane (g, m): output m, bytes of chunk 4 k + g
  while (tab.size() % 4) tab.push_back(0);
  b.t_w = (int32_t)tab.size();
  std::vector<int8_t> w((size_t)b.steps * parts * 1024, 0);
  for (size_t c = 0; c < chunks.size(); ++c)
    for (const auto& m : member[c])
      for (int j = 0; j < n_out; ++j) {
        const int v = weights[(size_t)j * n_in + m.second];
        const int lo7 = split ? (int)pmod64(v + 64, 128) - 64 : v;
        const size_t at = (c / 4) * parts * 1024 + ((c % 4) * 16 + (size_t)j) * 16 + (size_t)m.first;
        w[at] = (int8_t)lo7;
        if (split) w[at + 1024] = (int8_t)((v - lo7) / 128);
      }
  const size_t at = tab.size();
  tab.resize(at + w.size() / 4);
  memcpy(&tab[at], w.data(), w.size());
  b.t_choff = (int32_t)tab.size();
  for (int c = 0; c < 4 * b.steps; ++c) tab.push_back(c < (int)chunks.size() ? (int32_t)chunks[(size_t)c] : (int32_t)chunks[0]);
  b.t_bias = (int32_t)tab.size();
  for (int j = 0; j < 16; ++j) {
    int64_t sum = 0;
    for (int i = 0; j < n_out && i < n_in; ++i) sum += weights[(size_t)j * n_in + i];
    tab.push_back((int32_t)((j < n_out && bias ? bias[j] : 0) + 128 + 128 * sum));
  }
  for (int k = 0; k < a.rr; ++k) {
    const int64_t e = k == last ? kLinBoxX : k == kj ? kLinBoxY : 1;
    b.t_org[k] = (int32_t)tab.size();
    for (int64_t i = 0; i < b.nb[k]; ++i) {
      for (int d = 0; d < a.ra; ++d) tab.push_back((int32_t)pmod64((int64_t)Ps[d][k] * (i * e), a.S[d]));
      for (int d = 0; d < a.ro; ++d) tab.push_back((int32_t)((int64_t)a.Po[d][k] * (i * e) % a.So[d]));
    }
  }
  for (int d = 0; d < a.ra; ++d) {
    b.org0[d] = (int32_t)pmod64((int64_t)a.o[d] + b.dlo[d], a.S[d]);
    b.mg_bn[d] = magic((uint32_t)b.bn[d]);
  }
  for (int d = 0; d < a.ro; ++d) {
    b.oorg0[d] = a.oo[d];
    auto near = [&](int k) { return (int64_t)a.Po[d][k] * 2 > a.So[d] ? a.Po[d][k] - a.So[d] : a.Po[d][k]; };
    b.Pl[d] = near(last);
    b.Pj[d] = kj >= 0 ? near(kj) : 0;
    // a point's base from its block's corner: one addition or subtraction wraps it
    if (std::abs((int64_t)b.Pl[d]) * (kLinBoxX - 1) + std::abs((int64_t)b.Pj[d]) * (kLinBoxY - 1) > a.So[d]) return;
  }
  b.mg_nch = magic((uint32_t)b.nch);
  b.use = 1;
}

}  // namespace

extern "C" {

aol_status aol_linear_plan_create(const aol_tiler* in, const aol_tiler* out, const int16_t* weights,
                                  const int32_t* bias, aol_linear_plan** plan) {
  if (!plan) return fail(AOL_ERR_INVALID, "NULL plan output");
  *plan = nullptr;
  aol_status st = check_tiler(in, "in", kLinMaxIn);
  if (!st) st = check_tiler(out, "out", kLinMaxOut);
  if (st) return st;
  if (!weights) return fail(AOL_ERR_INVALID, "NULL weights");
  if (out->rep_rank != in->rep_rank) return fail(AOL_ERR_INVALID, "input and output repetition ranks differ");
  for (int k = 0; k < in->rep_rank; ++k)
    if (out->rep_shape[k] != in->rep_shape[k]) return fail(AOL_ERR_INVALID, "repetition spaces differ");
  const int n_in = (int)count(in->pat_shape, in->pat_rank);
  const int n_out = (int)count(out->pat_shape, out->pat_rank);
  const int64_t nrep = count(in->rep_shape, in->rep_rank);
  // int32 accumulation must be exact: |sum_i W x + bias + 128| < 2^31 for any x in 0..255
  for (int j = 0; j < n_out; ++j) {
    int64_t m = 128 + (bias ? std::abs((int64_t)bias[j]) : 0);
    for (int i = 0; i < n_in; ++i) m += 255 * std::abs((int64_t)weights[(size_t)j * n_in + i]);
    if (m >= (1LL << 31)) return fail(AOL_ERR_UNSUPPORTED, "output %d: weights too large for exact int32 sums", j);
  }
  // exact coverage: the output tiler writes every element of its array once
  const int64_t out_elems = count(out->array_shape, out->array_rank);
  if (out_elems != nrep * n_out)
    return fail(AOL_ERR_INVALID, "output array has %lld elements for %lld repetitions x %d pattern elements",
                (long long)out_elems, (long long)nrep, n_out);
  {
    std::vector<uint8_t> seen((size_t)out_elems, 0);
    std::vector<int64_t> ofs((size_t)n_out * out->array_rank);
    for (int j = 0; j < n_out; ++j) fitting_offsets(out, j, &ofs[(size_t)j * out->array_rank]);
    int64_t r[AOL_MAX_RANK] = {0, 0, 0, 0};
    for (int64_t n = 0; n < nrep; ++n) {
      for (int j = 0; j < n_out; ++j) {
        int64_t flat = 0;
        for (int d = 0; d < out->array_rank; ++d) {
          int64_t v = out->origin[d] + ofs[(size_t)j * out->array_rank + d];
          for (int k = 0; k < out->rep_rank; ++k) v += out->paving[d][k] * r[k];
          flat = flat * out->array_shape[d] + pmod64(v, out->array_shape[d]);
        }
        if (seen[(size_t)flat]) return fail(AOL_ERR_INVALID, "output tiler writes an element twice (not a bijection)");
        seen[(size_t)flat] = 1;
      }
      for (int k = out->rep_rank - 1; k >= 0; --k) {
        if (++r[k] < out->rep_shape[k]) break;
        r[k] = 0;
      }
    }
  }

  aol_linear_plan* p = new (std::nothrow) aol_linear_plan();
  if (!p) return fail(AOL_ERR_NOMEM, "plan allocation");
  LinearArgs& a = p->args;
  for (int v : {1, 2, 3, 4, 6, 8, 9, 12, 16})
    if (n_out <= v) {
      p->nout = v;
      break;
    }
  const int NOUT = p->nout;
  const int n_pairs = (n_in + 1) / 2, n_pad = 2 * n_pairs;
  a.nrep = nrep;
  a.rr = in->rep_rank;
  for (int k = 0; k < a.rr; ++k) a.R[k] = (int32_t)in->rep_shape[k];
  a.ra = in->array_rank;
  a.ro = out->array_rank;
  a.n_pairs = n_pairs;
  a.n_out = n_out;
  a.nout_pad = NOUT;
  std::vector<int32_t> ioff, ifd, ooff, ofd;
  side(in, n_in, n_pad, a.S, a.st, a.o, a.P, a.lo, a.hi, a.inc, ioff, ifd);
  side(out, n_out, NOUT, a.So, a.sto, a.oo, a.Po, a.olo, a.ohi, a.oinc, ooff, ofd);
  // Rotation of a row's points over its threads (a schedule choice; results
  // do not depend on it): start the threads at the first point of a cyclic
  // run of points whose input pattern leaves the array along an axis that
  // moves with the row (axes fixed along a row wrap every point of it or none).
  a.rot = 0;
  if (a.R[a.rr - 1] <= kLinThreads) {
    const int R = a.R[a.rr - 1];
    std::vector<char> wraps((size_t)R, 0);
    for (int x = 0; x < R; ++x)
      for (int d = 0; d < a.ra; ++d) {
        if (a.P[d][a.rr - 1] == 0) continue;
        const int64_t b = pmod64((int64_t)a.o[d] + (int64_t)a.P[d][a.rr - 1] * x, a.S[d]);
        if (b + a.lo[d] < 0 || b + a.hi[d] >= a.S[d]) wraps[(size_t)x] = 1;
      }
    for (int x = 0; x < R; ++x)
      if (wraps[(size_t)x] && !wraps[(size_t)((x + R - 1) % R)]) {
        a.rot = x;
        break;
      }
  }
  // the table: ioff, ifd, packed weight pairs, bias + 128, ooff, ofd
  std::vector<int32_t> tab(ioff);
  a.t_ifd = (int32_t)tab.size();
  tab.insert(tab.end(), ifd.begin(), ifd.end());
  a.t_w = (int32_t)tab.size();
  for (int k = 0; k < n_pairs; ++k)
    for (int j = 0; j < NOUT; ++j) {
      auto w = [&](int i) -> uint32_t {
        return (j < n_out && i < n_in) ? (uint16_t)weights[(size_t)j * n_in + i] : 0u;
      };
      tab.push_back((int32_t)(w(2 * k) | (w(2 * k + 1) << 16)));
    }
  a.t_bias = (int32_t)tab.size();
  for (int j = 0; j < NOUT; ++j) tab.push_back((j < n_out && bias ? bias[j] : 0) + 128);
  a.t_ooff = (int32_t)tab.size();
  tab.insert(tab.end(), ooff.begin(), ooff.end());
  a.t_ofd = (int32_t)tab.size();
  tab.insert(tab.end(), ofd.begin(), ofd.end());
  plan_pack(a, in, out, weights, bias, n_in, n_out, p->pack);
  if (!p->pack.inst) {
    std::vector<int32_t> eg, og;
    plan_stage(a, NOUT, ioff, ooff, n_in, n_out, p->stage, eg, og);
    if (p->stage.ppt) {
      LinearStage& st = p->stage;
      st.t_eg = (int32_t)tab.size();
      tab.insert(tab.end(), eg.begin(), eg.end());
      st.t_og = (int32_t)tab.size();
      tab.insert(tab.end(), og.begin(), og.end());
      st.t_grp = (int32_t)tab.size();
      for (int g = 0; g < kLinGroups; ++g) {
        tab.push_back(g < st.ng ? st.gb[g] : 0);
        tab.push_back(g < st.ng ? st.gl[g] : 0);
        tab.push_back(g < st.ngo ? st.ob[g] : 0);
        tab.push_back(g < st.ngo ? st.ol[g] : 0);
      }
      // per-chunk clean test and first positions (see LinearStage)
      const int last = a.rr - 1;
      const int64_t rows = a.nrep / a.R[last];
      const int64_t nchunks = rows * st.chunks;
      if (2 * nchunks + (int64_t)tab.size() > kLinCoordTable) {
        st.ppt = 0;  // too large: point by point
      } else {
        st.cq = (int32_t)tab.size();
        const int C = kLinThreads * st.ppt;
        int64_t r[kLinRank] = {0, 0, 0, 0};
        for (int64_t row = 0; row < rows; ++row) {
          for (int c = 0; c < st.chunks; ++c) {
            const int64_t x0 = (int64_t)c * C, npts = std::min<int64_t>(C, a.R[last] - x0);
            r[last] = x0;
            bool clean = true;
            int64_t flat0 = 0, oflat0 = 0;
            for (int d = 0; d < a.ra; ++d) {
              int64_t v = a.o[d];
              for (int k = 0; k < a.rr; ++k) v += (int64_t)a.P[d][k] * r[k];
              const int64_t b = v % a.S[d];
              clean = clean && b + a.lo[d] >= 0 && b + (npts - 1) * a.P[d][last] + a.hi[d] < a.S[d];
              flat0 += b * a.st[d];
            }
            for (int d = 0; d < a.ro; ++d) {
              int64_t v = a.oo[d];
              for (int k = 0; k < a.rr; ++k) v += (int64_t)a.Po[d][k] * r[k];
              const int64_t b = v % a.So[d];
              clean = clean && b + a.olo[d] >= 0 && b + (npts - 1) * a.Po[d][last] + a.ohi[d] < a.So[d];
              oflat0 += b * a.sto[d];
            }
            tab.push_back(clean ? (int32_t)flat0 : -1);
            tab.push_back(clean ? (int32_t)oflat0 : -1);
          }
          for (int k = last - 1; k >= 0; --k) {  // next row, row-major
            if (++r[k] < a.R[k]) break;
            r[k] = 0;
          }
        }
        for (int k = 0; k < last; ++k) st.mg_R[k] = magic((uint32_t)a.R[k]);
        st.mg_R[last] = magic((uint32_t)st.chunks);
      }
    }
  }
  if (!p->pack.inst && !p->stage.ppt) {
    plan_box(a, in, weights, bias, n_in, n_out, p->box, tab);
    if (p->box.use) {
      const hipError_t e = linear_box_prepare(p->box);
      if (e != hipSuccess) {
        delete p;
        return hip_fail(e, "linear kernel attributes");
      }
    }
  }
  if ((st = p->d_tab.upload(tab.data(), tab.size() * sizeof(int32_t)))) {
    delete p;
    return st;
  }
  a.tab = (const int32_t*)p->d_tab.ptr;
  *plan = p;
  return ok();
}

aol_status aol_linear_run(aol_linear_plan* plan, const uint8_t* d_in, uint8_t* d_out, hipStream_t stream) {
  if (!plan) return fail(AOL_ERR_INVALID, "NULL plan");
  if (!d_in || !d_out) return fail(AOL_ERR_INVALID, "NULL buffer");
  LinearArgs a = plan->args;
  a.in = d_in;
  a.out = d_out;
  // the staged form loads and stores whole 16-byte chunks: both arrays 16-byte aligned
  const bool staged = plan->stage.ppt > 0 && (((uintptr_t)d_in | (uintptr_t)d_out) & 15) == 0;
  hipError_t e = plan->pack.inst ? linear_pack_launch(a, plan->pack, stream)
                 : staged        ? linear_staged_launch(plan->nout, a, plan->stage, stream)
                 : plan->box.use ? linear_box_launch(a, plan->box, stream)
                                 : linear_launch(plan->nout, a, stream);
  if (e != hipSuccess) return hip_fail(e, "linear task launch");
  return ok();
}

aol_status aol_linear_plan_destroy(aol_linear_plan* plan) {
  delete plan;
  return ok();
}

}  // extern "C"
