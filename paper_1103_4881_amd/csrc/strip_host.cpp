// Host-side construction of the strip kernel's descriptors: per-filter
// operand tables, per-plane geometry and segments.
#include "strip_host.h"

#include <algorithm>
#include <climits>
#include <cstring>

#include "band_host.h"

namespace aol {

namespace {

int64_t pmod64(int64_t a, int64_t m) {
  const int64_t r = a % m;
  return r < 0 ? r + m : r;
}

uint16_t coeff_bits(int elem, int c) {
  const float x = (float)c / 256.0f;  // exact in the format (checked by build_band)
  uint16_t r;
  if (elem == kBF16) {
    uint32_t u;
    memcpy(&u, &x, 4);
    r = (uint16_t)(u >> 16);
  } else {
    const _Float16 h = (_Float16)x;
    memcpy(&r, &h, 2);
  }
  return r;
}

}  // namespace

aol_status build_strip_tables(const FilterHost& hf, const FilterHost& vf, int elem, StripTables& out) {
  out.cls = -1;
  std::vector<uint8_t> hfr, vfr;
  AxisBand hb, vb;
  aol_status st = build_band(hf, 16, elem, true, false, hb, hfr, "hf");
  if (st) return st == AOL_ERR_UNSUPPORTED ? AOL_OK : st;
  st = build_band(vf, 16, elem, false, hb.split != 0, vb, vfr, "vf");
  if (st) return st == AOL_ERR_UNSUPPORTED ? AOL_OK : st;
  if (vb.split && !hb.split) {  // one kernel instance carries both axes: same operand layout
    st = build_band(hf, 16, elem, true, true, hb, hfr, "hf");
    if (st) return st;
  }
  const bool split = hb.split != 0;
  if (hb.nblk > kStripMaxBlocks || vb.nblk > kStripMaxBlocks) return AOL_OK;

  StripFilter& F = out.host;
  memset(&F, 0, sizeof F);
  const int E = elem == kU8 ? 16 : 8;
  F.nblk_h = hb.nblk;
  F.per_chunks = hb.q * 16 / E;
  F.zfrag = hb.zfrag;
  F.ubias = hb.ubias && vb.ubias;
  for (int b = 0; b < hb.nblk; ++b) F.hblk[b] = hb.chunk0[b] | hb.frag[b] << 16 | hb.nk[b] << 24;
  for (int b = 0; b < hb.nblk; ++b) F.hend[b] = (hb.wend[b] + E - 1) / E;
  // vertical windows in steps of 16 lines from line s_min
  F.nblk_v = vb.nblk;
  F.per_steps = vb.q;
  F.hbias0 = hb.bias[0];
  F.vbias0 = vb.bias[0];
  F.mg_h = strip_magic(hb.nblk);
  F.mg_v = strip_magic(vb.nblk);
  std::vector<int32_t> bias(2 * kStripMaxBlocks * 16, 0);
  memcpy(&bias[0], hb.bias, sizeof(int32_t) * hb.nblk * 16);
  memcpy(&bias[kStripMaxBlocks * 16], vb.bias, sizeof(int32_t) * vb.nblk * 16);
  const int p = vf.p, q = vf.q, T = vf.taps;
  int steps = 1;
  for (int b = 0; b < vb.nblk; ++b) {
    int lo = INT_MAX, hi = INT_MIN;
    for (int o = 16 * b; o < 16 * b + 16; ++o) {
      const int t0 = q * (o / p) + vf.s[o % p] - vb.s_min;
      lo = std::min(lo, t0);
      hi = std::max(hi, t0 + T);
    }
    F.vlo[b] = lo;
    F.vhi[b] = hi;
    F.v0[b] = lo / 16;
    F.v1[b] = (hi + 15) / 16;
    steps = std::max(steps, F.v1[b] - F.v0[b]);
  }
  const int sk = elem == kU8 ? 4 : 2;  // steps per vertical K-step
  const int kv = (steps + sk - 1) / sk;
  const StripClass* tab = elem == kU8 ? kStripU8 : kStripF;
  const int n_cls = elem == kU8 ? kStripU8Classes : kStripFClasses;
  int c = 0;
  while (c < n_cls && (tab[c].kh < hb.kmax || tab[c].kv < kv)) ++c;
  if (c == n_cls) return AOL_OK;
  const int KV = tab[c].kv, parts = split ? 2 : 1;
  // Vertical operands: K-step k of block b covers steps v1 - sk*KV + sk*k ...;
  // lane (g, n) element sk-step i, line j of the step's four: line 16*step +
  // 4g + j (the order the horizontal products leave the lines in)
  vfr.assign((size_t)vb.nblk * KV * parts * kLanes * 16, 0);
  for (int b = 0; b < vb.nblk; ++b)
    for (int k = 0; k < KV; ++k)
      for (int lane = 0; lane < kLanes; ++lane)
        for (int e = 0; e < 4 * sk; ++e) {
          const int g = lane >> 4, o = 16 * b + (lane & 15);
          const int line = 16 * (F.v1[b] - sk * KV + sk * k + e / 4) + 4 * g + e % 4;
          const int t = line - (q * (o / p) + vf.s[o % p] - vb.s_min);
          const int cf = t >= 0 && t < T ? vf.c[(size_t)(o % p) * T + t] : 0;
          uint8_t* f = &vfr[((size_t)(b * KV + k) * parts * kLanes + lane) * 16];
          if (elem == kU8) {
            const int lo7 = (int)pmod64(cf + 64, 128) - 64;  // c = lo7 + 128 * hi
            f[e] = (uint8_t)(int8_t)(split ? lo7 : cf);
            if (split) f[(size_t)kLanes * 16 + e] = (uint8_t)(int8_t)((cf - lo7) / 128);
          } else {
            const uint16_t bits = coeff_bits(elem, cf);
            memcpy(f + 2 * e, &bits, 2);
          }
        }
  F.vfrag_bytes = (int32_t)vfr.size();
  F.lds_x = (int32_t)((vfr.size() + (size_t)vb.nblk * 16 * 4 + 15) / 16 * 16);
  // strips per workgroup: as many as its waves take, within the staged chunks
  // wherever in the period the first one lies
  for (int f = 0; f < kStripForms; ++f) {
    out.wnb[f] = 0;
    out.lds[f] = (size_t)F.lds_x + 2 * strip_stage(strip_waves(f));
    if ((f == kStripWide && (c > 0 || split)) || out.lds[f] > 160 * 1024) continue;
    for (int m = 1; m <= strip_waves(f) * tab[c].nb; ++m) {
      int most = 0;
      for (int b = 0; b < hb.nblk; ++b) {
        const int e = b + m - 1;
        most = std::max(most, F.hend[e % hb.nblk] + e / hb.nblk * F.per_chunks - hb.chunk0[b]);
      }
      if (most > strip_chunks(strip_waves(f))) break;
      out.wnb[f] = m;
    }
  }
  if (out.wnb[kStripUsual] < 1) return AOL_OK;
  // one allocation and one copy: the filter, then its operands and biases
  const size_t bias_bytes = bias.size() * sizeof(int32_t);
  std::vector<uint8_t> mem(sizeof F + hfr.size() + vfr.size() + bias_bytes);
  if ((st = out.d_filter.alloc(mem.size()))) return st;
  const uint8_t* dev = (const uint8_t*)out.d_filter.ptr;
  size_t at = sizeof F;
  auto place = [&](const void* src, size_t n) {
    memcpy(&mem[at], src, n);
    const uint8_t* p = dev + at;
    at += n;
    return p;
  };
  static_assert(sizeof F % 16 == 0, "operands of whole 16-byte chunks follow");
  F.hfrag = place(hfr.data(), hfr.size());
  F.vfrag = place(vfr.data(), vfr.size());
  F.bias = (const int32_t*)place(bias.data(), bias_bytes);
  memcpy(&mem[0], &F, sizeof F);
  hipError_t e = hipMemcpy(out.d_filter.ptr, mem.data(), mem.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpy");
  out.elem = elem;
  out.col0 = hb.s_min - hb.delta;
  out.line0 = vb.s_min;
  out.p_v = p;
  out.resident = c == 0 && !split ? 4 : 3;
  out.cls = 2 * c + (split ? 1 : 0);
  return AOL_OK;
}

bool build_strip_stream(const StripTables& t, int64_t h, int64_t w, int64_t in_pitch, int64_t out_pitch,
                        StripStream& S) {
  memset(&S, 0, sizeof S);
  const int64_t es = t.elem == kU8 ? 1 : 2, oes = t.elem == kU8 ? 1 : 4;
  const StripFilter& F = t.host;
  if (((h - 1) * in_pitch + w) * es > 0xFFFFFFFFLL || 16 * out_pitch * oes > 0xFFFFFFFFLL) return false;
  const int E = (int)(16 / es);
  S.in_pitch = in_pitch;
  S.out_pitch = out_pitch;
  S.h = (int32_t)h;
  S.w = (int32_t)w;
  // p outputs per q inputs: per period of 16 repetitions, nblk blocks of 16
  const int64_t qh = (int64_t)F.per_chunks * E / 16, qv = F.per_steps;
  const int64_t mh = F.nblk_v * ((h + qv - 1) / qv), mw = F.nblk_h * ((w + qh - 1) / qh);
  if (mh > (1 << 30) || mw > (1 << 30)) return false;  // (a plan's sides are checked, a batch's are not)
  S.mh = (int32_t)mh;
  S.mw = (int32_t)mw;
  S.col0 = t.col0;
  S.line0 = t.line0;
  S.nbh = (S.mw + 15) / 16;
  S.nbv = (S.mh + 15) / 16;
  S.tiny = w * es < 16 ? 1 : 0;
  return true;
}

uint32_t strip_magic(int d) { return d <= 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) / (uint32_t)d) + 1); }

bool strip_edges(const StripTables& t, const StripStream& S) { return S.w % (t.elem == kU8 ? 16 : 8) != 0; }

void strip_set_segments(StripStream& S, int wnb, int segb) {
  segb = std::min(segb, S.nbv);  // (a caller's segment may be any length)
  S.wgx = (S.nbh + wnb - 1) / wnb;
  S.wnb = (S.nbh + S.wgx - 1) / S.wgx;
  S.mg_wgx = strip_magic(S.wgx);
  S.nseg = (S.nbv + segb - 1) / segb;
  S.segb = (S.nbv + S.nseg - 1) / S.nseg;
  S.nseg = (S.nbv + S.segb - 1) / S.segb;
}

}  // namespace aol
