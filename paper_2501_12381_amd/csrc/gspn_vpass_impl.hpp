// Vertical passes of the two-pass family: the scan of T2B / B2T over planes
// too large to keep on chip (forward and the backward's recompute), and its
// adjoint.
//
// One workgroup owns one direction of one plane.  A row is spread over its
// waves, a lane holding G consecutive columns of one 8- or 16-byte vector, so
// every load instruction of a wave covers consecutive addresses.  The
// recurrence moves information by one column a row, so a wave also carries
// HL lanes (E = HL * G columns) of each neighbouring wave's span and scans E
// rows without talking to anyone: the columns it keeps stay exact while the
// wrong values creep in from the ends of the span.  Every E rows the waves
// exchange their edges through LDS (one barrier, two buffers).  A row step is
// then two DPP shifts and its multiply-adds, with no barrier and no LDS.
//
// What bounds it: the bytes a compute unit keeps in flight.  Rows stream
// through a register ring of R rows (5 maps a row), requested R rows ahead
// with buffer loads whose row offset is one scalar; reads outside the plane
// (idle steps before the first row, refills past the last one, lanes past the
// row) carry an out-of-range offset: they return zero and cost no traffic.
#pragma once

#include "gspn_device.hpp"
#include "gspn_launch.hpp"
#include "gspn_resident_impl.hpp"
#include "gspn_wide_impl.hpp"

namespace gspn {

struct VPassCfg {
  static constexpr int E = 8;           // rows between edge exchanges (columns of a halo)
  static constexpr int MAX_WAVES = 16;
};

// G fp32 values of a lane, loaded and stored as 16-byte vectors
template <int G>
__device__ __forceinline__ void vp_load_f(float (&v)[G], wide_rsrc_t r, int voff, int soff) {
#pragma unroll
  for (int i = 0; i < G; i += 4) {
    const auto t = __builtin_amdgcn_raw_buffer_load_b128(r, voff + i * 4, soff, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[i + j] = __uint_as_float(t[j]);
  }
}
typedef unsigned int vp_u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int vp_u32x4 __attribute__((ext_vector_type(4)));
// A 16-byte buffer store whose row offset is in the vector offset, never in
// the scalar one: a store of more than 8 bytes reads its data registers after
// it has issued, and with a scalar offset the compiler lets the next
// instruction overwrite them (measured on gfx950: a quarter of the lanes then
// store the new value); without one it keeps the wait state.
__device__ __forceinline__ void vp_store16(vp_u32x4 t, wide_rsrc_t r, int voff, int soff) {
  __builtin_amdgcn_raw_buffer_store_b128(t, r, (int)((unsigned)voff + (unsigned)soff), 0, 0);
}
template <int G>
__device__ __forceinline__ void vp_store_f(const float (&v)[G], wide_rsrc_t r, int voff, int soff) {
#pragma unroll
  for (int i = 0; i < G; i += 4) {
    const vp_u32x4 t = {__float_as_uint(v[i]), __float_as_uint(v[i + 1]), __float_as_uint(v[i + 2]),
                        __float_as_uint(v[i + 3])};
    vp_store16(t, r, voff + i * 4, soff);
  }
}
template <typename T, int G>
__device__ __forceinline__ void vp_store(const float (&v)[G], wide_rsrc_t r, int voff, int soff) {
  if constexpr (sizeof(T) == 4) {
    vp_store_f<G>(v, r, voff, soff);
  } else if constexpr (G == 4) {
    const vp_u32x2 t = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
    __builtin_amdgcn_raw_buffer_store_b64(t, r, voff, soff, 0);
  } else {
    static_assert(G == 8, "8- or 16-byte bf16 vectors");
    const vp_u32x4 t = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
    vp_store16(t, r, voff, soff);
  }
}

template <int N>
__device__ __forceinline__ void vp_store_words(const uint32_t (&v)[N], wide_rsrc_t r, int voff, int soff) {
  if constexpr (N == 2) {
    const vp_u32x2 t = {v[0], v[1]};
    __builtin_amdgcn_raw_buffer_store_b64(t, r, voff, soff, 0);
  } else {
    static_assert(N == 4, "8 or 16 bytes");
    const vp_u32x4 t = {v[0], v[1], v[2], v[3]};
    vp_store16(t, r, voff, soff);
  }
}

// A wave's span of a row: `k` lanes of columns kept per wave, HL halo lanes on
// each side that has a neighbouring wave.
template <int G>
struct VSpan {
  static constexpr int HL = VPassCfg::E / G;  // halo lanes
  int ks, ke;     // kept lanes of the row [ks, ke)
  int gl;         // the lane's place in the row (in lanes)
  bool kept, valid;
  __device__ __forceinline__ VSpan(int W, int k, int wave, int lane) {
    const int LT = W / G;  // W is a multiple of G
    ks = wave * k;
    ke = min(LT, ks + k);
    gl = ks - (wave > 0 ? HL : 0) + lane;
    kept = gl >= ks && gl < ke;
    valid = gl < min(LT, ke + HL);
  }
};

// Edge exchange of one value row: the kept edges of every wave into LDS, the
// halo lanes' values from the neighbouring waves.  buf: [2 parities][waves][2
// sides][E] floats.
template <int G>
__device__ __forceinline__ void vp_exchange(float (&v)[G], const VSpan<G>& sp, float* __restrict__ buf, int par,
                                            int wave, int nw) {
  constexpr int E = VPassCfg::E, HL = VSpan<G>::HL;
  float* b = buf + par * (VPassCfg::MAX_WAVES * 2 * E);
  if (sp.kept && sp.gl - sp.ks < HL) {
    float* d = b + (wave * 2 + 0) * E + (sp.gl - sp.ks) * G;
#pragma unroll
    for (int j = 0; j < G; ++j) d[j] = v[j];
  }
  if (sp.kept && sp.ke - sp.gl <= HL) {
    float* d = b + (wave * 2 + 1) * E + (HL - (sp.ke - sp.gl)) * G;
#pragma unroll
    for (int j = 0; j < G; ++j) d[j] = v[j];
  }
  lds_barrier();
  if (sp.gl < sp.ks) {  // left halo (waves after the first)
    const float* s = b + ((wave - 1) * 2 + 1) * E + (sp.gl - (sp.ks - HL)) * G;
#pragma unroll
    for (int j = 0; j < G; ++j) v[j] = s[j];
  }
  if (sp.valid && sp.gl >= sp.ke) {  // right halo
    const float* s = b + ((wave + 1) * 2 + 0) * E + (sp.gl - sp.ke) * G;
#pragma unroll
    for (int j = 0; j < G; ++j) v[j] = s[j];
  }
}

// ---------------------------------------------------------------------------
// forward scan (also the backward's recompute)
//   OUT 0: h (fp32) to out[dir]
//   OUT 1: y = u * h
//   OUT 2: y = u * (acc + h)   (the other vertical direction's h in acc)
// ---------------------------------------------------------------------------
struct VScanParams {
  const void* x;
  const void* lam;
  const void* w;      // packed [n][3][planes][H][W]
  const void* u;
  void* y;
  const float* acc;   // OUT 2
  float* out[2];      // OUT 0: h of top-to-bottom, bottom-to-top
  int64_t planes, npc;
  int H, W;
  int slot[2];        // weight slots of top-to-bottom, bottom-to-top (-1: absent)
  int k;              // lanes kept per wave
  int grp;            // rows per local-GSPN group (H: the global scan)
  int renorm;
  int y_pd;           // y is (n, B, C, H, W): this direction's map at slot * npc
};

template <typename T, int G, int R, int OUT, bool LG, int MAXT>
__global__ void __launch_bounds__(MAXT) vscan_kernel(VScanParams p) {
  constexpr int E = VPassCfg::E, ES = (int)sizeof(T);
  static_assert(E % R == 0 && E % G == 0, "ring slots and halo lanes repeat with the exchange");
  typedef Pack<T, G> PK;
  __shared__ float xbuf[2 * VPassCfg::MAX_WAVES * 2 * E];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const bool two = p.slot[0] >= 0 && p.slot[1] >= 0;
  const int dir = two ? (blockIdx.x >= p.planes ? 1 : 0) : (p.slot[0] >= 0 ? 0 : 1);
  const int64_t plane = two && dir ? blockIdx.x - p.planes : blockIdx.x;
  const int H = p.H, W = p.W;
  const VSpan<G> sp(W, p.k, wave, lane);
  const int voff = sp.valid ? sp.gl * (G * ES) : kWideOob;
  const int voff_o = sp.kept ? sp.gl * (G * (OUT == 0 ? 4 : ES)) : kWideOob;
  const int voff_f = sp.kept ? sp.gl * (G * 4) : kWideOob;
  const int64_t pb = plane * (int64_t)H * W;
  const int PB = H * W * ES, rowb = W * ES;
  const int slot = dir ? p.slot[1] : p.slot[0];
  const T* w0 = (const T*)p.w + (int64_t)slot * 3 * p.npc + pb;
  const wide_rsrc_t rb[5] = {wide_rsrc((const T*)p.x + pb, PB), wide_rsrc((const T*)p.lam + pb, PB), wide_rsrc(w0, PB),
                             wide_rsrc(w0 + p.npc, PB), wide_rsrc(w0 + 2 * p.npc, PB)};
  wide_rsrc_t ro, ru, ra;
  if constexpr (OUT == 0) {
    ro = wide_rsrc((dir ? p.out[1] : p.out[0]) + pb, H * W * 4);
  } else {
    ro = wide_rsrc((T*)p.y + (p.y_pd ? (int64_t)slot * p.npc : 0) + pb, PB);
    ru = wide_rsrc((const T*)p.u + pb, PB);
    if constexpr (OUT == 2) ra = wide_rsrc(p.acc + pb, H * W * 4);
  }
  // rows in scan order; steps outside [0, H) touch nothing
  auto line_of = [&](int s) { return dir ? H - 1 - s : s; };
  auto row = [&](int s, int bytes) { return (unsigned)s < (unsigned)H ? line_of(s) * bytes : kWideOob; };
  PK ring[R][5];
  PK uring[R];
  float aring[R][G];
  auto load = [&](int k, int s) __attribute__((always_inline)) {
    const int so = row(s, rowb);
#pragma unroll
    for (int m = 0; m < 5; ++m) wide_load<T, G>(ring[k][m], rb[m], voff, so);
    if constexpr (OUT >= 1) wide_load<T, G>(uring[k], ru, voff, so);
    if constexpr (OUT == 2) vp_load_f<G>(aring[k], ra, voff_f, row(s, W * 4));
  };
  float hp[G];
#pragma unroll
  for (int q = 0; q < G; ++q) hp[q] = 0.f;
  // local GSPN: the step whose row starts the next group
  const int grp = p.grp;
  int nxt = dir ? (H % grp ? H % grp : grp) : grp;
  const int pos0 = sp.gl * G;

  auto step = [&](auto kc, int s) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value % R;
    if (s == nxt) {
#pragma unroll
      for (int q = 0; q < G; ++q) hp[q] = 0.f;
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
    float o[G];
    if constexpr (OUT >= 1) {
#pragma unroll
      for (int q = 0; q < G; ++q) o[q] = uring[k].get(q) * (OUT == 2 ? aring[k][q] + h[q] : h[q]);
    }
    load(k, s + R);
    if constexpr (OUT == 0) vp_store_f<G>(h, ro, voff_o, row(s, W * 4));
    else vp_store<T, G>(o, ro, voff_o, row(s, rowb));
  };

  // idle steps before row 0 make the step count a multiple of E
  const int s0 = -((E - H % E) % E);
#pragma unroll
  for (int k = 0; k < R; ++k) load(k, s0 + k);
  int par = 0;
  for (int s = s0; s < H; s += E) {
    static_for<0, E>([&](auto kc) __attribute__((always_inline)) { step(kc, s + decltype(kc)::value); });
    if (nw > 1 && s + E < H) {
      vp_exchange<G>(hp, sp, xbuf, par, wave, nw);
      par ^= 1;
    }
  }
}

// ---------------------------------------------------------------------------
// adjoint: rows against the scan order,
//   g = u dy + a1 + a0(p+1) + a2(p-1)      (a_k = w_k g of the row done before)
//   dw_k = g h[previous row](p + k - 1)
// gsum += g for the direction that comes first (top-to-bottom when present).
// The other one runs in the same launch, so its g goes to a place of its own:
// the dx and dlam maps, which hold nothing until the finish overwrites them
// (fp32 storage: g in dx; bf16: the upper halves of g's bits in dx, the lower
// ones in dlam).  The finish adds it to gsum.
// ---------------------------------------------------------------------------
struct VAdjParams {
  const void* dy;
  const void* u;
  const void* w;        // all directions, packed
  void* dw;             // all directions, packed
  const float* h[2];    // h of top-to-bottom, bottom-to-top
  float* gsum;
  void* g_hi;           // dx and dlam, the second direction's g
  void* g_lo;
  int64_t planes, npc;
  int H, W;
  int slot[2];
  int k;
  int grp;
  int renorm;
  int y_pd;             // dy is (n, B, C, H, W): the direction's map at slot * npc
};

template <typename T, int G, int R, bool LG, int MAXT>
__global__ void __launch_bounds__(MAXT) vadj_kernel(VAdjParams p) {
  constexpr int E = VPassCfg::E, ES = (int)sizeof(T);
  static_assert(E % R == 0 && E % G == 0, "ring slots and halo lanes repeat with the exchange");
  typedef Pack<T, G> PK;
  __shared__ float xbuf[2 * VPassCfg::MAX_WAVES * 2 * E];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const bool two = p.slot[0] >= 0 && p.slot[1] >= 0;
  const int dir = two ? (blockIdx.x >= p.planes ? 1 : 0) : (p.slot[0] >= 0 ? 0 : 1);
  const int64_t plane = two && dir ? blockIdx.x - p.planes : blockIdx.x;
  const int H = p.H, W = p.W;
  const VSpan<G> sp(W, p.k, wave, lane);
  const int voff = sp.valid ? sp.gl * (G * ES) : kWideOob;
  const int voff_h = sp.valid ? sp.gl * (G * 4) : kWideOob;
  const int voff_o = sp.kept ? sp.gl * (G * ES) : kWideOob;
  const int voff_f = sp.kept ? sp.gl * (G * 4) : kWideOob;
  const int64_t pb = plane * (int64_t)H * W;
  const int PB = H * W * ES, PF = H * W * 4, rowb = W * ES, rowf = W * 4;
  const int slot = dir ? p.slot[1] : p.slot[0];
  const T* w0 = (const T*)p.w + (int64_t)slot * 3 * p.npc + pb;
  const wide_rsrc_t rb[5] = {wide_rsrc((const T*)p.dy + (p.y_pd ? (int64_t)slot * p.npc : 0) + pb, PB),
                             wide_rsrc((const T*)p.u + pb, PB), wide_rsrc(w0, PB), wide_rsrc(w0 + p.npc, PB),
                             wide_rsrc(w0 + 2 * p.npc, PB)};
  T* d0 = (T*)p.dw + (int64_t)slot * 3 * p.npc + pb;
  const wide_rsrc_t rd[3] = {wide_rsrc(d0, PB), wide_rsrc(d0 + p.npc, PB), wide_rsrc(d0 + 2 * p.npc, PB)};
  const wide_rsrc_t rh = wide_rsrc((dir ? p.h[1] : p.h[0]) + pb, PF);
  const bool add = !(two && dir);
  const wide_rsrc_t rg = wide_rsrc(p.gsum + pb, PF);
  const int voff_g = add ? voff_f : kWideOob;  // not added to: nothing is read
  const wide_rsrc_t rhi = wide_rsrc((T*)p.g_hi + pb, PB), rlo = wide_rsrc((T*)p.g_lo + pb, PB);
  auto line_of = [&](int s) { return dir ? s : H - 1 - s; };
  auto row = [&](int s, int bytes) { return (unsigned)s < (unsigned)H ? line_of(s) * bytes : kWideOob; };
  PK ring[R][5];
  float hring[R][G], gring[R][G];
  auto load = [&](int k, int s) __attribute__((always_inline)) {
    const int so = row(s, rowb);
#pragma unroll
    for (int m = 0; m < 5; ++m) wide_load<T, G>(ring[k][m], rb[m], voff, so);
    // the previous row in scan order is the next step's row (none after the last step)
    vp_load_f<G>(hring[k], rh, voff_h, row(s + 1, rowf));
    vp_load_f<G>(gring[k], rg, voff_g, row(s, rowf));
  };
  float a0[G], a1[G], a2[G];
#pragma unroll
  for (int q = 0; q < G; ++q) a0[q] = a1[q] = a2[q] = 0.f;
  // the step whose row starts a group: it read a zero state, and the row after
  // it in this order (the row before it in scan order) gets nothing from it
  const int grp = p.grp;
  int nxt = dir ? grp - 1 : (H - 1) % grp;
  const int pos0 = sp.gl * G;
  int par = 0;

  auto step = [&](auto kc, int s) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value % R;
    const bool rst = s == nxt;
    if (rst) {
#pragma unroll
      for (int q = 0; q < G; ++q) hring[k][q] = 0.f;
      nxt += grp;
    }
    const float ar = from_next_lane(a0[0]), al = from_prev_lane(a2[G - 1]);
    float g[G], hv[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const float an = q == G - 1 ? ar : a0[q + 1];
      const float ap = q == 0 ? al : a2[q - 1];
      const float in = a1[q] + an + ap;
      const float gv = fmaf(ring[k][1].get(q), ring[k][0].get(q), in);
      g[q] = sp.valid ? gv : 0.f;
      hv[q] = hring[k][q];
    }
    float ga[G];
#pragma unroll
    for (int q = 0; q < G; ++q) ga[q] = gring[k][q] + g[q];
    const float hn = from_next_lane(hv[0]), hl = from_prev_lane(hv[G - 1]);
    // the last step of a block: the halo lanes take the neighbours' exact g
    // before the products are formed
    if constexpr (decltype(kc)::value == E - 1) {
      if (nw > 1 && s + 1 < H) {
        vp_exchange<G>(g, sp, xbuf, par, wave, nw);
        par ^= 1;
      }
    }
    float dv[3][G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      float wa = ring[k][2].get(q), wb = ring[k][3].get(q), wc = ring[k][4].get(q);
      Norm3 nr;
      if constexpr (LG) {
        nr = normalize3(wa, wb, wc, pos0 + q == 0, pos0 + q == W - 1, p.renorm != 0);
        wa = nr.w[0];
        wb = nr.w[1];
        wc = nr.w[2];
      }
      a0[q] = rst ? 0.f : wa * g[q];
      a1[q] = rst ? 0.f : wb * g[q];
      a2[q] = rst ? 0.f : wc * g[q];
      dv[0][q] = g[q] * (q == 0 ? hl : hv[q - 1]);
      dv[1][q] = g[q] * hv[q];
      dv[2][q] = g[q] * (q == G - 1 ? hn : hv[q + 1]);
      if constexpr (LG) norm3_vjp(nr, dv[0][q], dv[1][q], dv[2][q]);
    }
    load(k, s + R);
    const int so = row(s, rowb);
#pragma unroll
    for (int m = 0; m < 3; ++m) vp_store<T, G>(dv[m], rd[m], voff_o, so);
    if (add) {
      vp_store_f<G>(ga, rg, voff_f, row(s, rowf));
    } else if constexpr (ES == 4) {
      vp_store_f<G>(ga, rhi, voff_o, so);
    } else {
      uint32_t hi[G / 2], lo[G / 2];
#pragma unroll
      for (int q = 0; q < G / 2; ++q) split_f2(ga[2 * q], ga[2 * q + 1], hi[q], lo[q]);
      vp_store_words<G / 2>(hi, rhi, voff_o, so);
      vp_store_words<G / 2>(lo, rlo, voff_o, so);
    }
  };

  const int s0 = -((E - H % E) % E);
#pragma unroll
  for (int k = 0; k < R; ++k) load(k, s0 + k);
  for (int s = s0; s < H; s += E)
    static_for<0, E>([&](auto kc) __attribute__((always_inline)) { step(kc, s + decltype(kc)::value); });
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct VGeom {
  int g;      // columns per lane
  int waves;  // waves per row
  int k;      // lanes kept per wave
};
// 4 columns a lane as long as 16 waves hold the row (3840 columns): narrower
// lanes mean more waves, each with its own loads in flight; the widest bf16
// rows take 8 (a 16-byte vector).
inline VGeom vpass_geom(int W) {
  for (int g : {4, 8}) {
    const int lt = W / g, hl = VPassCfg::E / g;
    const int n = lt <= 64 ? 1 : (lt + 64 - 2 * hl - 1) / (64 - 2 * hl);
    if (n <= VPassCfg::MAX_WAVES) return {g, n, (lt + n - 1) / n};
  }
  return {0, 0, 0};
}

// Ring depth R and register budget (MAXT threads a workgroup): as many rows in
// flight as the registers of the workgroup's waves allow.
template <typename T, int G, int R, int MAXT>
hipError_t launch_vscan_r(const VScanParams& p, int out, bool lg, int waves, hipStream_t st) {
  const int64_t grid = p.planes * (p.slot[0] >= 0 && p.slot[1] >= 0 ? 2 : 1);
  if (grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  // the fused outputs hold rows of u (and acc) as well; 16-byte inputs with the
  // logits' temporaries leave room for two rows
  constexpr int RL = G * sizeof(T) == 16 ? R / 2 : R, RU = R / 2, R2 = 2;
  auto kern = out == 0 ? (lg ? vscan_kernel<T, G, RL, 0, true, MAXT> : vscan_kernel<T, G, R, 0, false, MAXT>)
            : out == 1 ? (lg ? vscan_kernel<T, G, RU, 1, true, MAXT> : vscan_kernel<T, G, RU, 1, false, MAXT>)
                       : (lg ? vscan_kernel<T, G, R2, 2, true, MAXT> : vscan_kernel<T, G, R2, 2, false, MAXT>);
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * waves), 0, st, p);
  return hipGetLastError();
}
// Column bands (gspn_vband_impl.hpp) for few planes.
struct VBandCfg {
  static constexpr int G = 2;   // columns per lane
  static constexpr int NW = 4;  // waves per workgroup, one per SIMD
  static constexpr int SPAN = NW * (64 - 2 * VSpan<G>::HL);  // lanes of a workgroup's span
};

struct VBandGeom {
  int rows;  // rows per launch
  int hb;    // halo lanes of a band: one column a row
  int nb;    // bands
  int mid;   // lanes kept by an inner band; the first and last keep hb more (they have one halo)
};
inline VBandGeom vband_geom(int W, int rows) {  // rows wider than one band (vband_choose)
  using C = VBandCfg;
  const int lt = W / C::G, hb = rows / C::G;
  const int nb = (lt - 2 * hb + C::SPAN - 2 * hb - 1) / (C::SPAN - 2 * hb);
  return {rows, hb, nb, (lt - 2 * hb + nb - 1) / nb};
}

// The bands of a launch, none (nb == 0) where the one-workgroup pass is the
// better one.  Bands are taken where a plane's row needs more than one wave per
// SIMD and every band still gets a compute unit of its own: 128 rows a launch,
// or 64 when their wider bands are what fits.  The whole forward, one workgroup
// a plane and direction -> bands of 64 -> of 128 rows, bf16: 1 plane 2048 x 2048
// with logits 2622 -> 1450 -> 1416 us, 16 planes 1024 x 1024 829 -> 722 -> 687,
// 20 planes 1024 x 2048 (128 rows: 400 bands) 1769 -> 1375 us.  Left as they
// were: 64 planes 1024 x 1024 1900 -> 1879 us (384 bands), 24 planes 512 x 512
// fp32 410 -> 447 us (3 waves a row).
inline VBandGeom vband_choose(const VScanParams& p) {
  const int64_t groups = p.planes * (p.slot[0] >= 0 && p.slot[1] >= 0 ? 2 : 1);
  if (vpass_geom(p.W).waves > 4)
    for (int rows : {128, 64}) {
      const VBandGeom g = vband_geom(p.W, rows);
      if (groups * g.nb <= 256) return g;
    }
  return {0, 0, 0, 0};
}
template <typename T>
hipError_t launch_vband(const VScanParams& p, const VBandGeom& g, bool lg, hipStream_t st);

template <typename T>
hipError_t launch_vscan(VScanParams p, int out, bool lg, hipStream_t st) {
  if (out == 0) {
    const VBandGeom b = vband_choose(p);
    if (b.nb > 0) return launch_vband<T>(p, b, lg, st);
  }
  const VGeom v = vpass_geom(p.W);
  p.k = v.k;
  if constexpr (sizeof(T) == 4) {  // rows of at most 2048 columns: 9 waves
    if (v.g != 4 || v.waves > 10) return hipErrorInvalidValue;
    return launch_vscan_r<T, 4, 4, 640>(p, out, lg, v.waves, st);
  } else {
    if (v.g == 4) return launch_vscan_r<T, 4, 8, 1024>(p, out, lg, v.waves, st);
    if (v.g == 8 && v.waves <= 10) return launch_vscan_r<T, 8, 4, 640>(p, out, lg, v.waves, st);
    return hipErrorInvalidValue;
  }
}

template <typename T, int G, int R, int MAXT>
hipError_t launch_vadj_r(const VAdjParams& p, bool lg, int waves, hipStream_t st) {
  const int64_t grid = p.planes * (p.slot[0] >= 0 && p.slot[1] >= 0 ? 2 : 1);
  if (grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  auto kern = lg ? vadj_kernel<T, G, R, true, MAXT> : vadj_kernel<T, G, R, false, MAXT>;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * waves), 0, st, p);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_vadj(VAdjParams p, bool lg, hipStream_t st) {
  const VGeom v = vpass_geom(p.W);
  p.k = v.k;
  if constexpr (sizeof(T) == 4) {
    if (v.g != 4 || v.waves > 10) return hipErrorInvalidValue;
    return v.waves <= 5 ? launch_vadj_r<T, 4, 4, 320>(p, lg, v.waves, st)
                        : launch_vadj_r<T, 4, 2, 640>(p, lg, v.waves, st);
  } else {
    if (v.g == 4 && v.waves <= 5) return launch_vadj_r<T, 4, 8, 320>(p, lg, v.waves, st);
    if (v.g == 4 && v.waves <= 10) return launch_vadj_r<T, 4, 4, 640>(p, lg, v.waves, st);
    if (v.g == 4) return launch_vadj_r<T, 4, 2, 1024>(p, lg, v.waves, st);
    if (v.g == 8 && v.waves <= 10) return launch_vadj_r<T, 8, 2, 640>(p, lg, v.waves, st);
    return hipErrorInvalidValue;
  }
}

}  // namespace gspn
