// Generic resident forwards: planes of any size and alignment.
//
// Quad kernel (lines of at most 64, merged; any plane, unmerged outputs): a
// workgroup owns one plane (or a wave's worth of small ones); its four waves
// run the four directions at the same time.  The vertical pair adds its h into
// one LDS array and the horizontal pair into another (QMerge), so the waves meet
// only in the middle; y = u * (vertical sum + horizontal sum).  Unmerged outputs (y_d = u_d h_d) need no array at all: each wave
// multiplies its h by u and stores it.
//
// Duo kernel (larger planes of which one sum fits LDS): the vertical pair scans,
// then the horizontal one, each direction on two waves (half of a line each,
// see QHalf), adding into one array (QMerge).  What bounds it is how few waves a
// compute unit holds, so LDS is spent on a second workgroup rather than on
// sharing lam * x: x and lam are read once per axis.  Only where two arrays a
// plane leave room for two workgroups (the registers' limit) is lam * x formed
// once into the second one (LX).  One array against two: 1280 planes of 96 x
// 168 bf16 344 -> 251 us, 640 of 104 x 152 202 -> 152, 640 of 112 x 112 145 ->
// 110; planes of which two arrays do not fit ran on two waves before: 300 planes of
// 160 x 160 328 -> 194 us, 200 x 192 with logits 589 -> 330 us.
#pragma once

#include "gspn_quad_impl.hpp"

namespace gspn {

struct QFwdParams {
  const void* x;
  const void* lam;
  const void* w;
  const void* u;
  void* y;
  int64_t npc, planes;
  int H, W, P, segsh;
  int slot[4];
  int gh, gw;        // group lengths (the line count: global)
  int renorm;
  int lam_pd, u_pd;  // per-direction maps (u_pd: unmerged outputs only)
  int split;         // duo: lines of at least 32 positions go to two waves
  // the maps from `n` elements on (npc stays the stride between them)
  template <typename T>
  void skip(int64_t n) {
    x = (const T*)x + n; lam = (const T*)lam + n; w = (const T*)w + n; u = (const T*)u + n;
    y = (T*)y + n;
  }
};

// TV: vectors of a row in the registers of a horizontal wave (fewer let more
// workgroups share a compute unit)
template <typename T, int NPV, int NPH, int VL, int TV, bool LG, bool PD>
__global__ void __launch_bounds__(256, NPH > 1 ? 1 : (TV <= 4 ? 4 : 2)) quad_fwd_kernel(QFwdParams p) {
  constexpr int ES = (int)sizeof(T), VE = VL;
  constexpr int RV = TV <= 2 ? kHalo : QRing<T, NPV>::RV;  // small planes have few rows
  extern __shared__ float lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ppw = 64 >> p.segsh;
  const int64_t g0 = (int64_t)blockIdx.x * ppw;
  const int HW = p.H * p.W;
  const int64_t left = p.planes - g0;
  const QPlanes g{p.H, p.W, p.P, (int)(left < ppw ? left : ppw), p.segsh};
  const int bytes = g.np * HW * ES;
  const int64_t gof = g0 * HW;
  const int ARR = (p.H + 1) * p.P;
  const bool rev = wave & 1, hz = wave >= 2;
  const int slot = hz ? (rev ? p.slot[3] : p.slot[2]) : (rev ? p.slot[1] : p.slot[0]);
  float* arr = lds + (lane >> p.segsh) * 2 * ARR + (hz ? ARR : 0);
  const bool other = (hz ? (rev ? p.slot[2] : p.slot[3]) : (rev ? p.slot[0] : p.slot[1])) >= 0;
  if (slot >= 0) {
    const T* w0 = (const T*)p.w + (int64_t)slot * 3 * p.npc + gof;
    const wide_rsrc_t rb[6] = {q_rsrc((const T*)p.x + gof, bytes),
                               q_rsrc((const T*)p.lam + (p.lam_pd ? slot * p.npc : 0) + gof, bytes),
                               q_rsrc(w0, bytes),
                               q_rsrc(w0 + p.npc, bytes),
                               q_rsrc(w0 + 2 * p.npc, bytes),
                               q_rsrc((const T*)p.u + (p.u_pd ? slot * p.npc : 0) + gof, bytes)};
    const wide_rsrc_t ry = q_rsrc((T*)p.y + (PD ? slot * p.npc : 0) + gof, bytes);
    if (!hz) {
      const QV<T, NPV> ln(g, lane);
      QMerge<NPV> m{arr, {}, rev, other, false};
#pragma unroll
      for (int q = 0; q < NPV; ++q) m.off[q] = ln.aoff[q];
      qv_forward<T, NPV, RV, LG, PD, false>(
          rb, ln, g, rev, p.gh, p.renorm != 0, QLamX<NPV>{},
          [&](int b, int n, int line) __attribute__((always_inline)) {
            if constexpr (!PD) m.begin(b, n, line * g.P);
          },
          [&](int line, int next, int so, const float (&h)[NPV], const QPack<T, NPV>& u)
              __attribute__((always_inline)) {
            if constexpr (PD) {
              float o[NPV];
#pragma unroll
              for (int q = 0; q < NPV; ++q) o[q] = u.get(q) * h[q];
              qv_store<T, NPV>(o, ry, ln, so);
            } else {
              m.put(line * g.P, next * g.P, h);
            }
          },
          [&](int b, int n) __attribute__((always_inline)) {
            if constexpr (!PD) m.end(b, n);
          });
    } else {
      const QH<T, NPH> ln(g, lane);
      float yb[NPH][VL];
      QMerge<NPH> m{arr, {}, rev, other, false};
#pragma unroll
      for (int q = 0; q < NPH; ++q) m.off[q] = ln.aoff[q];
      qh_forward<T, NPH, VL, TV, 1, LG, PD, false>(
          rb, ln, g, rev, p.gw, p.renorm != 0, QLamX<NPH>{},
          [&](int ti, int n, int col) __attribute__((always_inline)) {
            if constexpr (!PD) m.begin(ti, n, col);
          },
          [&](int col, int e, bool cut, const float (&h)[NPH], const QPack<T, VL> (&u)[NPH])
              __attribute__((always_inline)) {
            if constexpr (PD) {
#pragma unroll
              for (int q = 0; q < NPH; ++q) {
                yb[q][e] = u[q].get(e) * h[q];
                if (cut) q_store_elem<T>(yb[q][e], ry, ln.voff[q], col * ES);
              }
            } else {
              m.put(col, col + (rev ? -1 : 1), h);
            }
          },
          [&](int ti, int n, bool cut, int c0) __attribute__((always_inline)) {
            if constexpr (!PD) m.end(ti, n);
            if constexpr (PD) {
              if (!cut) {
#pragma unroll
                for (int q = 0; q < NPH; ++q) {
                  if (VL > 1 && rev) q_reverse<VL>(yb[q]);
                  q_store<T, VL>(yb[q], ry, ln.voff[q], c0 * ES);
                }
              }
            }
          });
    }
  } else if constexpr (!PD) {
    lds_barrier();
    lds_barrier();
  }
  if constexpr (!PD) {
    __syncthreads();
    const wide_rsrc_t ru = q_rsrc((const T*)p.u + gof, bytes), ry = q_rsrc((T*)p.y + gof, bytes);
    const bool hv = p.slot[0] >= 0 || p.slot[1] >= 0, hh = p.slot[2] >= 0 || p.slot[3] >= 0;
    constexpr int U = 4;
    QPack<T, VE> uv[U];
    q_flat<VE, U>(
        g, threadIdx.x, 256,
        [&](int k, int e) __attribute__((always_inline)) { q_load<T, VE>(uv[k], ru, e * ES, 0); },
        [&](int k, int e, const int (&li)[VE], int pl) __attribute__((always_inline)) {
          const float* a = lds + pl * 2 * ARR;
          float o[VE];
#pragma unroll
          for (int q = 0; q < VE; ++q)
            o[q] = uv[k].get(q) * ((hv ? a[li[q]] : 0.f) + (hh ? a[ARR + li[q]] : 0.f));
          q_store<T, VE>(o, ry, e * ES, 0);
        });
  }
}

// Waves of an axis: split lines (at least 32 positions) go to two waves per
// direction, shorter ones to one (the second keeps the barriers in step).
template <typename T, int NPV, int NPH, int VL, bool LG, bool LX>
__global__ void __launch_bounds__(256, 2) duo_fwd_kernel(QFwdParams p) {
  constexpr int ES = (int)sizeof(T), VE = VL;
  extern __shared__ float lds[];  // the sum, lam * x (LX), the exchange buffers of split lines
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int HW = p.H * p.W;
  const int64_t gof = (int64_t)blockIdx.x * HW;
  const QPlanes g{p.H, p.W, p.P, 1, 6};
  const int bytes = HW * ES;
  const int ARR = (p.H + 1) * p.P;
  float *const acc = lds, *const lxa = lds + ARR;
  const int dir = wave >> 1, hf = wave & 1;
  float* const xbuf = lds + (LX ? 2 : 1) * ARR + dir * (2 * 2 * kHalo);
  const bool rev = dir != 0, rn = p.renorm != 0;
  auto barrier = []() __attribute__((always_inline)) { lds_barrier(); };

  const wide_rsrc_t rx = q_rsrc((const T*)p.x + gof, bytes);
  if constexpr (LX) {
    for (int i = threadIdx.x; i < p.P; i += 256) lxa[p.H * p.P + i] = 0.f;  // idle rows read the padding row
    const wide_rsrc_t rl = q_rsrc((const T*)p.lam + gof, bytes);
    constexpr int U = 4;
    QPack<T, VE> vx[U], vl[U];
    q_flat<VE, U>(
        g, threadIdx.x, 256,
        [&](int k, int e) __attribute__((always_inline)) {
          q_load<T, VE>(vx[k], rx, e * ES, 0);
          q_load<T, VE>(vl[k], rl, e * ES, 0);
        },
        [&](int k, int, const int (&li)[VE], int) __attribute__((always_inline)) {
#pragma unroll
          for (int q = 0; q < VE; ++q) lxa[li[q]] = vl[k].get(q) * vx[k].get(q);
        });
    __syncthreads();
  }

  const bool hv = p.slot[0] >= 0 || p.slot[1] >= 0;
  // one axis: the pair's scans with exchanges and middle-line barriers
  auto axis = [&](auto hzt) __attribute__((always_inline)) {
    constexpr bool HZ = decltype(hzt)::value;
    constexpr int NP = HZ ? NPH : NPV;
    const int Pn = HZ ? p.H : p.W, grp = HZ ? p.gw : p.gh;
    const bool split = Pn >= 32 && p.split;
    const int slot = p.slot[(HZ ? 2 : 0) + dir];
    const int nt = (p.W + VL - 1) / VL;  // vectors of a horizontal scan
    if (slot < 0 || (!split && hf)) {
      // the barriers of the waves that scan: exchanges, and the two in the middle
      const int nb = QRows::make<QRing<T, NPV>::RV>(p.H, 0, false).nb;
      const int nx = !split ? 0 : (HZ ? (nt - 1) / (kHalo / VL) : nb - 1);
      for (int i = 0; i < nx + 2; ++i) lds_barrier();
      return;
    }
    const T* w0 = (const T*)p.w + (int64_t)slot * 3 * p.npc + gof;
    const wide_rsrc_t rw0 = q_rsrc(w0, bytes);
    const wide_rsrc_t rb[6] = {LX ? rw0 : rx,
                               LX ? rw0 : q_rsrc((const T*)p.lam + (p.lam_pd ? slot * p.npc : 0) + gof, bytes),
                               rw0,
                               q_rsrc(w0 + p.npc, bytes),
                               q_rsrc(w0 + 2 * p.npc, bytes),
                               rw0};
    const QHalf half{hf, ((Pn + 1) / 2 + NP - 1) / NP * NP, xbuf};
    auto exchange = [&](int par, auto& v, int pos0) __attribute__((always_inline)) {
      if (split) q_exchange<NP>(v, half, pos0, par, barrier);
    };
    QLamX<NP> lx;
    lx.lx = lxa;
    // the sum at the lane's positions (padding where the value is not this wave's)
    QMerge<NP> m{acc, {}, rev, p.slot[(HZ ? 2 : 0) + (dir ^ 1)] >= 0, HZ && hv};
    if constexpr (HZ) {
      const QH<T, NP> ln = split ? QH<T, NP>(g, lane, half) : QH<T, NP>(g, lane);
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        lx.off[q] = (ln.valid[q] ? ln.pos0 + q : 0) * g.P;
        m.off[q] = (ln.voffs[q] != kWideOob ? ln.pos0 + q : g.H) * g.P;
      }
      // vectors in a group of loads: 5 maps (LX: 3) in under 200 registers
      constexpr int TV = LX ? (NP == 4 ? 3 : 8) : (NP == 1 ? 8 : (NP == 2 ? 4 : 1));
      qh_forward<T, NP, VL, TV, LX && NP == 1 ? 2 : 1, LG, false, LX>(
          rb, ln, g, rev, grp, rn, lx,
          [&](int ti, int n, int col) __attribute__((always_inline)) { m.begin(ti, n, col); },
          [&](int col, int, bool, const float (&h)[NP], const QPack<T, VL> (&)[NP]) __attribute__((always_inline)) {
            m.put(col, col + (rev ? -1 : 1), h);
          },
          [&](int ti, int n, bool, int) __attribute__((always_inline)) { m.end(ti, n); },
          [&](int par, auto& v) __attribute__((always_inline)) { exchange(par, v, ln.pos0); });
    } else {
      const QV<T, NP> ln = split ? QV<T, NP>(g, lane, half) : QV<T, NP>(g, lane);
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        lx.off[q] = ln.valid[q] ? ln.pos0 + q : 0;
        m.off[q] = ln.valid[q] && ln.kept ? ln.pos0 + q : g.W;
      }
      qv_forward<T, NP, QRing<T, NP>::RV, LG, false, LX>(
          rb, ln, g, rev, grp, rn, lx,
          [&](int b, int n, int line) __attribute__((always_inline)) { m.begin(b, n, line * g.P); },
          [&](int line, int next, int, const float (&h)[NP], const QPack<T, NP>&) __attribute__((always_inline)) {
            m.put(line * g.P, next * g.P, h);
          },
          [&](int b, int n) __attribute__((always_inline)) { m.end(b, n); },
          [&](int par, auto& v) __attribute__((always_inline)) { exchange(par, v, ln.pos0); });
    }
  };
  if (hv) {
    axis(std::false_type{});
    __syncthreads();
  }
  if (p.slot[2] >= 0 || p.slot[3] >= 0) {
    axis(std::true_type{});
    __syncthreads();
  }

  const wide_rsrc_t ru = q_rsrc((const T*)p.u + gof, bytes), ry = q_rsrc((T*)p.y + gof, bytes);
  constexpr int U = 4;
  QPack<T, VE> uv[U];
  q_flat<VE, U>(
      g, threadIdx.x, 256,
      [&](int k, int e) __attribute__((always_inline)) { q_load<T, VE>(uv[k], ru, e * ES, 0); },
      [&](int k, int e, const int (&li)[VE], int) __attribute__((always_inline)) {
        float o[VE];
#pragma unroll
        for (int q = 0; q < VE; ++q) o[q] = uv[k].get(q) * acc[li[q]];
        q_store<T, VE>(o, ry, e * ES, 0);
      });
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct QConfig {
  int npv, nph, segsh, P;
};
inline bool quad_config(int H, int W, QConfig* c) {
  if (H > 256 || W > 256 || H < 1 || W < 1) return false;
  auto np = [](int n) { return n <= 64 ? 1 : (n <= 128 ? 2 : 4); };
  c->npv = np(W);
  c->nph = np(H);
  const int mx = H > W ? H : W;
  // a segment keeps at least one lane past the line: the zero between planes
  c->segsh = mx <= 15 ? 4 : (mx <= 31 ? 5 : 6);
  c->P = W + 1 + (W & 1);  // odd pitch: a horizontal wave's rows fall in distinct banks
  return true;
}
// LDS of `arrays` fp32 arrays for each plane of a workgroup
inline int64_t quad_lds(const QConfig& c, int H, int arrays) {
  return (int64_t)(64 >> c.segsh) * arrays * (H + 1) * c.P * 4;
}
constexpr int kQuadMaxLds = 160 * 1024;

// Launches `kern` (256 threads, `ppw` planes a workgroup) over every plane.  A
// launch's threads are counted in 32 bits, which four waves a plane reach at
// 16.8 million planes: more go in several launches.
template <typename T, typename Q>
hipError_t quad_launch(void (*kern)(Q), Q p, int ppw, int lds, hipStream_t st) {
  constexpr int64_t most = 0xffffffffll / 256;  // workgroups
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  for (int64_t left = p.planes;;) {
    p.planes = left < most * ppw ? left : most * ppw;
    hipLaunchKernelGGL(kern, dim3((unsigned)((p.planes + ppw - 1) / ppw)), dim3(256), lds, st, p);
    const hipError_t e = hipGetLastError();
    left -= p.planes;
    if (e != hipSuccess || left == 0) return e;
    p.template skip<T>(p.planes * p.H * p.W);
  }
}
constexpr int kDuoXbuf = 2 * 2 * 2 * kHalo * 4;  // exchange buffers of the duo kernel

inline bool quad_fwd_size_fits(int H, int W, bool unmerged) {
  QConfig c;
  return quad_config(H, W, &c) && (unmerged || quad_lds(c, H, 1) <= kQuadMaxLds);
}

template <typename T, int NPV, int NPH, int VL, bool LG, bool PD, int TV = QVecs<NPH>::TV>
hipError_t launch_quad_fwd_k(const QFwdParams& p, int lds, hipStream_t st) {
  return quad_launch<T>(quad_fwd_kernel<T, NPV, NPH, VL, TV, LG, PD>, p, 64 >> p.segsh, lds, st);
}
template <typename T, int NPV, int NPH, bool LG, bool LX>
hipError_t launch_duo_fwd_k(const QFwdParams& p, int lds, hipStream_t st) {
  return quad_launch<T>(duo_fwd_kernel<T, NPV, NPH, 16 / (int)sizeof(T), LG, LX>, p, 1, lds, st);
}

// positions a lane of a wave that holds half a line and the halo of the other half
inline int duo_np(int n) { return n < 32 || (n + 1) / 2 + kHalo <= 64 ? 1 : ((n + 1) / 2 + 1 + kHalo <= 128 ? 2 : 4); }

template <typename T, bool LG, bool LX>
hipError_t launch_duo_fwd(const QFwdParams& p, int lds, hipStream_t st) {
  const int v = p.split ? duo_np(p.W) : 4, h = p.split ? duo_np(p.H) : 4;
  if (v == 1)
    return h == 1 ? launch_duo_fwd_k<T, 1, 1, LG, LX>(p, lds, st)
         : h == 2 ? launch_duo_fwd_k<T, 1, 2, LG, LX>(p, lds, st) : launch_duo_fwd_k<T, 1, 4, LG, LX>(p, lds, st);
  if (v == 2 && h == 1) return launch_duo_fwd_k<T, 2, 1, LG, LX>(p, lds, st);
  if (v == 4 && h == 1) return launch_duo_fwd_k<T, 4, 1, LG, LX>(p, lds, st);
  if (v == 2 && h == 2) return launch_duo_fwd_k<T, 2, 2, LG, LX>(p, lds, st);
  // a side over 240 beside one over 112, or lines kept whole
  if constexpr (LX) return hipErrorInvalidValue;  // (two arrays of such planes exceed LDS)
  else return launch_duo_fwd_k<T, 4, 4, LG, LX>(p, lds, st);
}

// merged outputs: lines of at most 64 positions on the quad kernel (and rows
// narrower than a vector), longer ones on the duo kernel
template <typename T, bool LG>
hipError_t launch_quad_fwd(QFwdParams p, hipStream_t st) {
  QConfig c;
  constexpr int VL = 16 / (int)sizeof(T);
  if (!quad_config(p.H, p.W, &c)) return hipErrorInvalidValue;
  p.P = c.P;
  p.segsh = c.segsh;
  const int64_t one = quad_lds(c, p.H, 1);
  if (one > kQuadMaxLds) return hipErrorInvalidValue;
  if (p.W < VL || (c.npv == 1 && c.nph == 1)) {
    const int lds = (int)(2 * one);  // (at most 34 KB)
    if constexpr (VL > 4) {  // bf16 rows of 4 to 7: 8-byte vectors
      if (p.W < VL && p.W >= 4 && c.nph == 1) return launch_quad_fwd_k<T, 1, 1, 4, LG, false, 2>(p, lds, st);
    }
    if (p.W < VL)  // the horizontal scans go column by column
      return c.nph == 1 ? launch_quad_fwd_k<T, 1, 1, 1, LG, false>(p, lds, st)
           : c.nph == 2 ? launch_quad_fwd_k<T, 1, 2, 1, LG, false>(p, lds, st)
                        : launch_quad_fwd_k<T, 1, 4, 1, LG, false>(p, lds, st);
    // Rows longer than two vectors: four in a group, which lets four workgroups share
    // a compute unit, not eight, which holds two (2048 planes, eight -> four: 8 x 64
    // fp32 59 -> 37 us, bf16 48 -> 29; 48 x 48 fp32 77 -> 72, bf16 55 -> 44), but for fp32
    // planes over 10 KB, whose rows' cache lines do not last until their second half
    // is read (45 x 60 92 -> 99, 60 x 64 113 -> 126).
    if constexpr (sizeof(T) == 4) {
      if (p.H * p.W > 2560) return launch_quad_fwd_k<T, 1, 1, VL, LG, false, 8>(p, lds, st);
    }
    return p.W <= 2 * VL ? launch_quad_fwd_k<T, 1, 1, VL, LG, false, 2>(p, lds, st)
                         : launch_quad_fwd_k<T, 1, 1, VL, LG, false, 4>(p, lds, st);
  }
  p.split = one + kDuoXbuf <= kQuadMaxLds;  // else the lines stay whole: the sum fills LDS to the last bytes
  // the second array costs no workgroup: two of them share a compute unit all
  // the same, or the planes are at most one each (160 planes 136 x 144 fp32: one
  // array 101 us, two 95; 600 planes bf16: 193 against 246)
  if (!p.lam_pd && 2 * one + kDuoXbuf <= (p.planes <= 256 ? kQuadMaxLds : kQuadMaxLds / 2))
    return launch_duo_fwd<T, LG, true>(p, (int)(2 * one) + kDuoXbuf, st);
  return launch_duo_fwd<T, LG, false>(p, (int)one + (p.split ? kDuoXbuf : 0), st);
}

// unmerged outputs
template <typename T, bool LG>
hipError_t launch_quad_fwd_pd(QFwdParams p, hipStream_t st) {
  QConfig c;
  constexpr int VL = 16 / (int)sizeof(T);
  if (!quad_config(p.H, p.W, &c)) return hipErrorInvalidValue;
  p.P = c.P;
  p.segsh = c.segsh;
  // planes of few rows leave most lanes of the horizontal waves idle, and more
  // workgroups a compute unit count more than long loads (2048 planes fp32, eight
  // vectors -> two: 8 x 64 53 -> 30 us, 16 x 32 34 -> 26; 32 x 40 50 -> 62)
  if (c.npv == 1 && c.nph == 1 && p.W >= VL && (p.W <= 4 * VL || p.H <= 16))
    return p.W <= 2 * VL || p.H <= 16 ? launch_quad_fwd_k<T, 1, 1, VL, LG, true, 2>(p, 0, st)
                                      : launch_quad_fwd_k<T, 1, 1, VL, LG, true, 4>(p, 0, st);
  auto h = [&](auto npv) -> hipError_t {
    constexpr int V = decltype(npv)::value;
    switch (c.nph) {
      case 1: return launch_quad_fwd_k<T, V, 1, VL, LG, true>(p, 0, st);
      case 2: return launch_quad_fwd_k<T, V, 2, VL, LG, true>(p, 0, st);
      default: return launch_quad_fwd_k<T, V, 4, VL, LG, true>(p, 0, st);
    }
  };
  if constexpr (VL > 4) {
    if (p.W < VL && p.W >= 4 && c.nph == 1) return launch_quad_fwd_k<T, 1, 1, 4, LG, true, 2>(p, 0, st);
  }
  if (p.W < VL)
    return c.nph == 1 ? launch_quad_fwd_k<T, 1, 1, 1, LG, true>(p, 0, st)
         : c.nph == 2 ? launch_quad_fwd_k<T, 1, 2, 1, LG, true>(p, 0, st)
                      : launch_quad_fwd_k<T, 1, 4, 1, LG, true>(p, 0, st);
  switch (c.npv) {
    case 1: return h(std::integral_constant<int, 1>{});
    case 2: return h(std::integral_constant<int, 2>{});
    default: return h(std::integral_constant<int, 4>{});
  }
}

inline QFwdParams quad_fwd_params(const ResidentFwdArgs& a) {
  QFwdParams p{};
  p.x = a.x; p.lam = a.lam; p.w = a.w; p.u = a.u; p.y = a.y;
  p.npc = a.planes * (int64_t)a.H * a.W;
  p.planes = a.planes;
  p.H = a.H; p.W = a.W;
  int n = 0;
  for (int d = 0; d < 4; ++d) p.slot[d] = (a.mask >> d) & 1 ? n++ : -1;
  p.gh = (a.group_h > 0 && a.group_h < a.H) ? a.group_h : a.H;
  p.gw = (a.group_w > 0 && a.group_w < a.W) ? a.group_w : a.W;
  p.renorm = a.renorm;
  p.lam_pd = a.lam_pd; p.u_pd = a.u_pd;
  return p;
}

}  // namespace gspn
