// Vertical scan of the two-pass family for few planes: the columns of a plane
// spread over several workgroups.
//
// gspn_vpass_impl.hpp gives a plane's direction to one workgroup; with one
// plane two of the 256 compute units then work, each on a whole row at a time
// (2048 columns with Eq. 6 logits: 0.9 us a row, the compute unit's arithmetic).
// Here a launch advances 128 (or 64) rows.  A workgroup keeps a band of columns
// and scans as many more on each side that has a neighbouring band: wrong
// values creep in from the ends of its span by one column a row, so after the
// launch's rows the band itself is exact.  The state between launches is the
// previous launch's last row of h, read back from the output array (fp32, so
// nothing is rounded).  Inside the workgroup the waves exchange 8-column halos
// every 8 rows, as in the one-workgroup pass; the sums are formed in the same
// order, and the result is the same bit for bit.
//
// What bounds it: a wave's serial chain and the launches' gaps.  Two columns a
// lane and one wave per SIMD give the shortest row step.
#pragma once

#include <algorithm>

#include "gspn_vpass_impl.hpp"

namespace gspn {

struct VBandParams {
  VScanParams v;
  int sb, se;  // rows of this launch in scan order: [sb, se), se - sb a multiple of E but for rows before 0
  int nb, mid, hb;  // VBandGeom
};

template <typename T, int R, bool LG>
__global__ void __launch_bounds__(64 * VBandCfg::NW) vband_kernel(VBandParams bp) {
  using C = VBandCfg;
  constexpr int G = C::G, E = VPassCfg::E, ES = (int)sizeof(T), NW = C::NW;
  static_assert(E % R == 0, "ring slots repeat with the exchange");
  typedef Pack<T, G> PK;
  const VScanParams& p = bp.v;
  __shared__ float xbuf[2 * VPassCfg::MAX_WAVES * 2 * E];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroup -> (direction, plane, band)
  const int band = blockIdx.x % bp.nb;
  const int64_t id = blockIdx.x / bp.nb;
  const bool two = p.slot[0] >= 0 && p.slot[1] >= 0;
  const int dir = two ? (id >= p.planes ? 1 : 0) : (p.slot[0] >= 0 ? 0 : 1);
  const int64_t plane = two && dir ? id - p.planes : id;
  const int H = p.H, W = p.W, LT = W / G;
  // kept lanes of the row [kb, ke), scanned ones [b0, b1)
  const bool last = band == bp.nb - 1;
  const int kb = band == 0 ? 0 : bp.hb + band * bp.mid;
  const int ke = last ? LT : bp.hb + (band + 1) * bp.mid;
  const int b0 = band == 0 ? 0 : kb - bp.hb;
  const int b1 = last ? LT : min(LT, ke + bp.hb);
  const int kw = (b1 - b0 + NW - 1) / NW;  // lanes kept per wave
  VSpan<G> sp((b1 - b0) * G, kw, wave, lane);
  sp.gl += b0;
  sp.ks += b0;
  sp.ke += b0;
  const bool kept = sp.kept && sp.gl >= kb && sp.gl < ke;
  const int voff = sp.valid ? sp.gl * (G * ES) : kWideOob;
  const int voff_h = sp.valid ? sp.gl * (G * 4) : kWideOob;
  const int voff_o = kept ? sp.gl * (G * 4) : kWideOob;
  const int64_t pb = plane * (int64_t)H * W;
  const int PB = H * W * ES, rowb = W * ES;
  const int slot = dir ? p.slot[1] : p.slot[0];
  const T* w0 = (const T*)p.w + (int64_t)slot * 3 * p.npc + pb;
  const wide_rsrc_t rb[5] = {wide_rsrc((const T*)p.x + pb, PB), wide_rsrc((const T*)p.lam + pb, PB), wide_rsrc(w0, PB),
                             wide_rsrc(w0 + p.npc, PB), wide_rsrc(w0 + 2 * p.npc, PB)};
  const wide_rsrc_t ro = wide_rsrc((dir ? p.out[1] : p.out[0]) + pb, H * W * 4);
  // rows in scan order; steps outside this launch's touch nothing
  const int first = max(bp.sb, 0), count = bp.se - first;
  auto row = [&](int s, int bytes) {
    return (unsigned)(s - first) < (unsigned)count ? (dir ? H - 1 - s : s) * bytes : kWideOob;
  };
  // state: h of the row before
  float hp[G];
  {
    const int so = bp.sb > 0 ? (dir ? H - bp.sb : bp.sb - 1) * (W * 4) : kWideOob;
    const auto t = __builtin_amdgcn_raw_buffer_load_b64(ro, voff_h, so, 0);
    hp[0] = __uint_as_float(t[0]);
    hp[1] = __uint_as_float(t[1]);
  }
  PK ring[R][5];
  auto load = [&](int k, int s) __attribute__((always_inline)) {
    const int so = row(s, rowb);
#pragma unroll
    for (int m = 0; m < 5; ++m) wide_load<T, G>(ring[k][m], rb[m], voff, so);
  };
  // local GSPN: the step whose row starts the next group
  const int grp = p.grp;
  int nxt = dir ? (H % grp ? H % grp : grp) : grp;
  if (nxt < bp.sb) nxt += (bp.sb - nxt + grp - 1) / grp * grp;
  const int pos0 = sp.gl * G;

  auto step = [&](auto kc, int s) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value % R;
    if (s == nxt) {
      hp[0] = hp[1] = 0.f;
      nxt += grp;
    }
    float xv[G], lv[G], a[G], b[G], c[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      xv[q] = ring[k][0].get(q);
      lv[q] = ring[k][1].get(q);
      a[q] = ring[k][2].get(q);
      b[q] = ring[k][3].get(q);
      c[q] = ring[k][4].get(q);
    }
    norm_weights<LG, G>(a, b, c, pos0, W, p.renorm != 0);
    const float left = from_prev_lane(hp[G - 1]), right = from_next_lane(hp[0]);
    float h[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const float hl = q == 0 ? left : hp[q - 1];
      const float hr = q == G - 1 ? right : hp[q + 1];
      float v = lv[q] * xv[q];
      v = fmaf(a[q], hl, v);
      v = fmaf(b[q], hp[q], v);
      v = fmaf(c[q], hr, v);
      h[q] = sp.valid ? v : 0.f;
    }
#pragma unroll
    for (int q = 0; q < G; ++q) hp[q] = h[q];
    load(k, s + R);
    const vp_u32x2 t = {__float_as_uint(h[0]), __float_as_uint(h[1])};
    __builtin_amdgcn_raw_buffer_store_b64(t, ro, voff_o, row(s, W * 4), 0);
  };

#pragma unroll
  for (int k = 0; k < R; ++k) {
    load(k, bp.sb + k);
    __builtin_amdgcn_sched_barrier(0);
  }
  int par = 0;
  for (int s = bp.sb; s < bp.se; s += E) {
    static_for<0, E>([&](auto kc) __attribute__((always_inline)) { step(kc, s + decltype(kc)::value); });
    if (s + E < bp.se) {
      vp_exchange<G>(hp, sp, xbuf, par, wave, NW);
      par ^= 1;
    }
  }
}

template <typename T>
hipError_t launch_vband(const VScanParams& p, const VBandGeom& g, bool lg, hipStream_t st) {
  constexpr int E = VPassCfg::E, R = 8;
  VBandParams bp{p, 0, 0, g.nb, g.mid, g.hb};
  const int64_t grid = p.planes * (p.slot[0] >= 0 && p.slot[1] >= 0 ? 2 : 1) * g.nb;
  if (grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  auto kern = lg ? vband_kernel<T, R, true> : vband_kernel<T, R, false>;
  // idle steps before row 0 make the step count a multiple of E
  int s = -((E - p.H % E) % E);
  while (s < p.H) {
    bp.sb = s;
    bp.se = std::min(p.H, s + g.rows);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * VBandCfg::NW), 0, st, bp);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    s = bp.se;
  }
  return hipSuccess;
}

}  // namespace gspn
