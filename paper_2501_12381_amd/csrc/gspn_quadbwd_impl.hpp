// Generic resident backward: the exact adjoint for planes of any size and
// alignment whose fp32 states fit LDS.
//
// Quad kernel (four arrays a plane fit): a workgroup owns one plane, or a
// wave's worth of small ones, and runs everything in one launch, one wave per
// direction side by side:
//   scan     each wave recomputes its direction's h into its own LDS array;
//   du       dy * (sum of h, fixed order), elementwise over all waves;
//   adjoint  each wave walks its direction backwards, g replaces h in its
//            array, dw leaves as it is formed;
//   dx, dlam lam and x times the sum of g (fixed order).
//
// Pair kernel (two arrays fit): the same for the two directions of one axis.
// The vertical launch leaves its sums of h and g in the workspace, the
// horizontal one adds its own and finishes (16 bytes a pixel through the
// workspace, instead of the 100 and more of the two-pass family).  Only one
// workgroup fits a compute unit, so two waves share a direction (each half of
// a line and 8 positions of the other's, exchanged every 8 lines) and all four
// SIMDs scan.
#pragma once

#include "gspn_quad_impl.hpp"
#include "gspn_quadfwd_impl.hpp"

namespace gspn {

struct QBwdParams {
  const void* dy;
  const void* x;
  const void* lam;
  const void* w;
  const void* u;
  void* dx;
  void* dw;
  void* dlam;
  void* du;
  int64_t npc, planes;
  int H, W, P, segsh;
  int n;  // directions present
  int slot[4];
  int gh, gw;
  int renorm;
  int lam_pd, u_pd, y_pd;  // per-direction maps (quad kernel only)
  // pair kernel: sums of h and g of the other axis, read by the launch that
  // finishes, written by the one before it (null: this axis alone)
  float* hsum;
  float* gsum;
  // the maps from `n` elements on (npc stays the stride between them)
  template <typename T>
  void skip(int64_t n) {
    dy = (const T*)dy + n; x = (const T*)x + n; lam = (const T*)lam + n; w = (const T*)w + n; u = (const T*)u + n;
    dx = (T*)dx + n; dw = (T*)dw + n; dlam = (T*)dlam + n; du = (T*)du + n;
  }
};

// TV: vectors of a row in the registers of a horizontal wave (fewer let more
// workgroups share a compute unit)
template <typename T, int NPV, int NPH, int VL, int TV, bool LG>
__global__ void __launch_bounds__(256, NPH > 1 ? (TV == 4 ? 2 : 1) : (TV <= 2 && NPV < 4 ? 4 : (TV <= 4 ? 3 : 2)))
quad_bwd_kernel(QBwdParams p) {
  constexpr int ES = (int)sizeof(T), VE = VL;
  constexpr int RQ = QRing<T, NPV>::RV, RV = TV <= 2 && RQ > kHalo ? kHalo : RQ;  // small planes have few rows
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
  const bool rev = wave & 1, hz = wave >= 2, rn = p.renorm != 0;
  const int slot = hz ? (rev ? p.slot[3] : p.slot[2]) : (rev ? p.slot[1] : p.slot[0]);
  float* arr = lds + ((lane >> p.segsh) * p.n + (slot < 0 ? 0 : slot)) * ARR;
  const T* w0 = (const T*)p.w + (int64_t)(slot < 0 ? 0 : slot) * 3 * p.npc + gof;
  T* d0 = (T*)p.dw + (int64_t)(slot < 0 ? 0 : slot) * 3 * p.npc + gof;
  const wide_rsrc_t rw0 = q_rsrc(w0, bytes), rw1 = q_rsrc(w0 + p.npc, bytes), rw2 = q_rsrc(w0 + 2 * p.npc, bytes);

  if (slot >= 0) {
    const wide_rsrc_t rb[6] = {q_rsrc((const T*)p.x + gof, bytes),
                               q_rsrc((const T*)p.lam + (p.lam_pd ? slot * p.npc : 0) + gof, bytes),
                               rw0, rw1, rw2, rw2};
    if (!hz) {
      const QV<T, NPV> ln(g, lane);
      qv_forward<T, NPV, RV, LG, false, false>(
          rb, ln, g, rev, p.gh, rn, QLamX<NPV>{}, [](int, int, int) {},
          [&](int line, int, int, const float (&h)[NPV], const QPack<T, NPV>&) __attribute__((always_inline)) {
            float* d = arr + line * g.P;
#pragma unroll
            for (int q = 0; q < NPV; ++q) d[ln.aoff[q]] = h[q];
          },
          [](int, int) {});
    } else {
      const QH<T, NPH> ln(g, lane);
      qh_forward<T, NPH, VL, TV, 1, LG, false, false>(
          rb, ln, g, rev, p.gw, rn, QLamX<NPH>{}, [](int, int, int) {},
          [&](int col, int, bool, const float (&h)[NPH], const QPack<T, VL> (&)[NPH]) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < NPH; ++q) arr[ln.aoff[q] + col] = h[q];
          },
          [](int, int, bool, int) {});
    }
  }
  __syncthreads();

  constexpr int U = VE > 1 ? 2 : 4;
  const int64_t npc = p.npc;
  // a direction's value at an LDS offset of plane pl
  auto at = [&](int pl, int d, int o) { return lds[(pl * p.n + p.slot[d]) * ARR + o]; };
  if (p.u_pd || p.y_pd) {
    q_flat<VE, 1>(
        g, threadIdx.x, 256, [](int, int) {},
        [&](int, int e, const int (&li)[VE], int pl) __attribute__((always_inline)) {
          float acc[VE];
#pragma unroll
          for (int q = 0; q < VE; ++q) acc[q] = 0.f;
          for (int d = 0; d < 4; ++d) {
            const int sd = p.slot[d];
            if (sd < 0) continue;
            QPack<T, VE> v;
            q_load<T, VE>(v, wide_rsrc((const T*)p.dy + (p.y_pd ? sd * npc : 0) + gof, bytes), e * ES, 0);
            float t[VE];
#pragma unroll
            for (int q = 0; q < VE; ++q) t[q] = v.get(q) * at(pl, d, li[q]);
            if (p.u_pd) {
              q_store<T, VE>(t, wide_rsrc((T*)p.du + sd * npc + gof, bytes), e * ES, 0);
            } else {
#pragma unroll
              for (int q = 0; q < VE; ++q) acc[q] += t[q];
            }
          }
          if (!p.u_pd) q_store<T, VE>(acc, wide_rsrc((T*)p.du + gof, bytes), e * ES, 0);
        });
  } else {
    const wide_rsrc_t rdy = q_rsrc((const T*)p.dy + gof, bytes), rdu = q_rsrc((T*)p.du + gof, bytes);
    QPack<T, VE> v[U];
    q_flat<VE, U>(
        g, threadIdx.x, 256, [&](int k, int e) __attribute__((always_inline)) { q_load<T, VE>(v[k], rdy, e * ES, 0); },
        [&](int k, int e, const int (&li)[VE], int pl) __attribute__((always_inline)) {
          float o[VE];
#pragma unroll
          for (int q = 0; q < VE; ++q) o[q] = 0.f;
#pragma unroll
          for (int d = 0; d < 4; ++d)
            if (p.slot[d] >= 0) {
#pragma unroll
              for (int q = 0; q < VE; ++q) o[q] += at(pl, d, li[q]);
            }
#pragma unroll
          for (int q = 0; q < VE; ++q) o[q] *= v[k].get(q);
          q_store<T, VE>(o, rdu, e * ES, 0);
        });
  }
  __syncthreads();

  if (slot >= 0) {
    const wide_rsrc_t rb[5] = {q_rsrc((const T*)p.u + (p.u_pd ? slot * npc : 0) + gof, bytes),
                               q_rsrc((const T*)p.dy + (p.y_pd ? slot * npc : 0) + gof, bytes), rw0, rw1, rw2};
    const wide_rsrc_t rd[3] = {q_rsrc(d0, bytes), q_rsrc(d0 + npc, bytes), q_rsrc(d0 + 2 * npc, bytes)};
    if (!hz) {
      const QV<T, NPV> ln(g, lane);
      qv_adjoint<T, NPV, RV, LG>(rb, rd, ln, g, arr, rev, p.gh, rn);
    } else {
      const QH<T, NPH> ln(g, lane);
      qh_adjoint<T, NPH, VL, TV, 1, LG>(rb, rd, ln, g, arr, rev, p.gw, rn);
    }
  }
  __syncthreads();

  const wide_rsrc_t rx = q_rsrc((const T*)p.x + gof, bytes), rdx = q_rsrc((T*)p.dx + gof, bytes);
  if (p.lam_pd) {
    q_flat<VE, 1>(
        g, threadIdx.x, 256, [](int, int) {},
        [&](int, int e, const int (&li)[VE], int pl) __attribute__((always_inline)) {
          QPack<T, VE> vx;
          q_load<T, VE>(vx, rx, e * ES, 0);
          float acc[VE];
#pragma unroll
          for (int q = 0; q < VE; ++q) acc[q] = 0.f;
          for (int d = 0; d < 4; ++d) {
            const int sd = p.slot[d];
            if (sd < 0) continue;
            QPack<T, VE> vl;
            q_load<T, VE>(vl, wide_rsrc((const T*)p.lam + sd * npc + gof, bytes), e * ES, 0);
            float t[VE];
#pragma unroll
            for (int q = 0; q < VE; ++q) {
              const float gv = at(pl, d, li[q]);
              acc[q] += vl.get(q) * gv;
              t[q] = vx.get(q) * gv;
            }
            q_store<T, VE>(t, wide_rsrc((T*)p.dlam + sd * npc + gof, bytes), e * ES, 0);
          }
          q_store<T, VE>(acc, rdx, e * ES, 0);
        });
    return;
  }
  const wide_rsrc_t rl = q_rsrc((const T*)p.lam + gof, bytes), rdl = q_rsrc((T*)p.dlam + gof, bytes);
  QPack<T, VE> vx[U], vl[U];
  q_flat<VE, U>(
      g, threadIdx.x, 256,
      [&](int k, int e) __attribute__((always_inline)) {
        q_load<T, VE>(vx[k], rx, e * ES, 0);
        q_load<T, VE>(vl[k], rl, e * ES, 0);
      },
      [&](int k, int e, const int (&li)[VE], int pl) __attribute__((always_inline)) {
        float s[VE], a[VE], b[VE];
#pragma unroll
        for (int q = 0; q < VE; ++q) s[q] = 0.f;
#pragma unroll
        for (int d = 0; d < 4; ++d)
          if (p.slot[d] >= 0) {
#pragma unroll
            for (int q = 0; q < VE; ++q) s[q] += at(pl, d, li[q]);
          }
#pragma unroll
        for (int q = 0; q < VE; ++q) {
          a[q] = vl[k].get(q) * s[q];
          b[q] = vx[k].get(q) * s[q];
        }
        q_store<T, VE>(a, rdx, e * ES, 0);
        q_store<T, VE>(b, rdl, e * ES, 0);
      });
}

// The pair kernel: both directions of one axis (HZ: the horizontal one), two
// waves each.  NP positions a lane of half a line.
template <typename T, bool HZ, int NP, int VL, bool LG>
__global__ void __launch_bounds__(256, 1) pair_bwd_kernel(QBwdParams p, int finish) {
  constexpr int ES = (int)sizeof(T), VE = 16 / ES;
  extern __shared__ float lds[];
  __shared__ float xbuf[2][2 * 2 * kHalo];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int HW = p.H * p.W;
  const int64_t gof = (int64_t)blockIdx.x * HW;
  const QPlanes g{p.H, p.W, p.P, 1, 6};
  const int bytes = HW * ES, fbytes = HW * 4;
  const int ARR = (p.H + (HZ ? 2 * kHalo : 0) + 1) * p.P;
  const int Pn = HZ ? p.H : p.W, grp = HZ ? p.gw : p.gh;
  const int K = ((Pn + 1) / 2 + NP - 1) / NP * NP;
  const int dir = wave >> 1;  // 0: top-to-bottom / left-to-right
  const bool rev = dir != 0, rn = p.renorm != 0;
  const int slot = p.slot[(HZ ? 2 : 0) + dir];
  const QHalf half{wave & 1, K, xbuf[dir]};
  float* arr = lds + dir * ARR;
  const T* w0 = (const T*)p.w + (int64_t)(slot < 0 ? 0 : slot) * 3 * p.npc + gof;
  T* d0 = (T*)p.dw + (int64_t)(slot < 0 ? 0 : slot) * 3 * p.npc + gof;
  const wide_rsrc_t rw0 = q_rsrc(w0, bytes), rw1 = q_rsrc(w0 + p.npc, bytes), rw2 = q_rsrc(w0 + 2 * p.npc, bytes);
  const wide_rsrc_t rx = q_rsrc((const T*)p.x + gof, bytes), rl = q_rsrc((const T*)p.lam + gof, bytes);
  const wide_rsrc_t ru = q_rsrc((const T*)p.u + gof, bytes), rdy = q_rsrc((const T*)p.dy + gof, bytes);

  using LN = std::conditional_t<HZ, QH<T, NP>, QV<T, NP>>;
  const LN ln(g, lane, half);
  auto exchange = [&](int par, auto& v) __attribute__((always_inline)) {
    q_exchange<NP>(v, half, ln.pos0, par, []() __attribute__((always_inline)) { lds_barrier(); });
  };
  auto idle = [&]() __attribute__((always_inline)) {  // a direction that is absent keeps the barriers in step
    const int n = HZ ? ((p.W + VL - 1) / VL - 1) / (kHalo / VL) : QRows::make<QRing<T, NP>::RV>(p.H, 0, false).nb - 1;
    for (int i = 0; i < n; ++i) lds_barrier();
  };

  if (slot >= 0) {
    const wide_rsrc_t rb[6] = {rx, rl, rw0, rw1, rw2, rw2};
    if constexpr (HZ) {
      qh_forward<T, NP, VL, QVecs<NP>::TV, NP == 1 ? 2 : 1, LG, false, false, true>(
          rb, ln, g, rev, grp, rn, QLamX<NP>{}, [](int, int, int) {},
          [&](int col, int, bool, const float (&h)[NP], const QPack<T, VL> (&)[NP]) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < NP; ++q) arr[ln.aoff[q] + col] = h[q];
          },
          [](int, int, bool, int) {}, exchange);
    } else {
      qv_forward<T, NP, QRing<T, NP>::RV, LG, false, false, true>(
          rb, ln, g, rev, grp, rn, QLamX<NP>{}, [](int, int, int) {},
          [&](int line, int, int, const float (&h)[NP], const QPack<T, NP>&) __attribute__((always_inline)) {
            float* d = arr + line * g.P;
#pragma unroll
            for (int q = 0; q < NP; ++q) d[ln.aoff[q]] = h[q];
          },
          [](int, int) {}, exchange);
    }
  } else {
    idle();
  }
  __syncthreads();

  constexpr int U = 2;
  const bool s0 = p.slot[HZ ? 2 : 0] >= 0, s1 = p.slot[HZ ? 3 : 1] >= 0;
  const int kc = HZ ? 1 << 20 : K, kr = HZ ? K : 1 << 20;
  // this axis's sum over the directions at an element
  auto sum_at = [&](int o) __attribute__((always_inline)) {
    return (s0 ? lds[o] : 0.f) + (s1 ? lds[ARR + o] : 0.f);
  };
  const bool add = finish && p.hsum != nullptr;
  if (finish) {
    const wide_rsrc_t rdu = q_rsrc((T*)p.du + gof, bytes), rs = q_rsrc(p.hsum + gof, add ? fbytes : 0);
    QPack<T, VE> v[U];
    float sv[U][VE];
    q_flat<VE, U>(
        g, threadIdx.x, 256,
        [&](int k, int e) __attribute__((always_inline)) {
          q_load<T, VE>(v[k], rdy, e * ES, 0);
          vp_load_f<VE>(sv[k], rs, e * 4, 0);  // zero when there is nothing to add
        },
        [&](int k, int e, const int (&li)[VE], int) __attribute__((always_inline)) {
          float o[VE];
#pragma unroll
          for (int q = 0; q < VE; ++q) o[q] = v[k].get(q) * (sv[k][q] + sum_at(li[q]));
          q_store<T, VE>(o, rdu, e * ES, 0);
        },
        kc, kr);
  } else {
    const wide_rsrc_t rs = q_rsrc(p.hsum + gof, fbytes);
    q_flat<VE, U>(
        g, threadIdx.x, 256, [](int, int) {},
        [&](int, int e, const int (&li)[VE], int) __attribute__((always_inline)) {
          float o[VE];
#pragma unroll
          for (int q = 0; q < VE; ++q) o[q] = sum_at(li[q]);
          vp_store_f<VE>(o, rs, e * 4, 0);
        },
        kc, kr);
  }
  __syncthreads();

  if (slot >= 0) {
    const wide_rsrc_t rb[5] = {ru, rdy, rw0, rw1, rw2};
    const wide_rsrc_t rd[3] = {q_rsrc(d0, bytes), q_rsrc(d0 + p.npc, bytes), q_rsrc(d0 + 2 * p.npc, bytes)};
    if constexpr (HZ) {
      qh_adjoint<T, NP, VL, QVecs<NP>::TV, NP == 1 ? 2 : 1, LG>(rb, rd, ln, g, arr, rev, grp, rn, exchange);
    } else {
      qv_adjoint<T, NP, QRing<T, NP>::RV, LG>(rb, rd, ln, g, arr, rev, grp, rn, exchange);
    }
  } else {
    idle();
  }
  __syncthreads();

  if (finish) {
    const wide_rsrc_t rs = q_rsrc(p.gsum + gof, add ? fbytes : 0);
    const wide_rsrc_t rdx = q_rsrc((T*)p.dx + gof, bytes), rdl = q_rsrc((T*)p.dlam + gof, bytes);
    QPack<T, VE> vx[U], vl[U];
    float sv[U][VE];
    q_flat<VE, U>(
        g, threadIdx.x, 256,
        [&](int k, int e) __attribute__((always_inline)) {
          q_load<T, VE>(vx[k], rx, e * ES, 0);
          q_load<T, VE>(vl[k], rl, e * ES, 0);
          vp_load_f<VE>(sv[k], rs, e * 4, 0);
        },
        [&](int k, int e, const int (&li)[VE], int) __attribute__((always_inline)) {
          float a[VE], b[VE];
#pragma unroll
          for (int q = 0; q < VE; ++q) {
            const float s = sv[k][q] + sum_at(li[q]);
            a[q] = vl[k].get(q) * s;
            b[q] = vx[k].get(q) * s;
          }
          q_store<T, VE>(a, rdx, e * ES, 0);
          q_store<T, VE>(b, rdl, e * ES, 0);
        },
        kc, kr);
  } else {
    const wide_rsrc_t rs = q_rsrc(p.gsum + gof, fbytes);
    q_flat<VE, U>(
        g, threadIdx.x, 256, [](int, int) {},
        [&](int, int e, const int (&li)[VE], int) __attribute__((always_inline)) {
          float o[VE];
#pragma unroll
          for (int q = 0; q < VE; ++q) o[q] = sum_at(li[q]);
          vp_store_f<VE>(o, rs, e * 4, 0);
        },
        kc, kr);
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
inline bool quad_bwd_size_fits(int H, int W) {
  QConfig c;
  return quad_config(H, W, &c) && quad_lds(c, H, 4) <= kQuadMaxLds;
}

template <typename T, int NPV, int NPH, int VL, bool LG, int TV = QVecs<NPH>::TV>
hipError_t launch_quad_bwd_k(const QBwdParams& p, int lds, hipStream_t st) {
  return quad_launch<T>(quad_bwd_kernel<T, NPV, NPH, VL, TV, LG>, p, 64 >> p.segsh, lds, st);
}

template <typename T, bool LG>
hipError_t launch_quad_bwd(QBwdParams p, hipStream_t st) {
  QConfig c;
  constexpr int VL = 16 / (int)sizeof(T);
  if (!quad_config(p.H, p.W, &c)) return hipErrorInvalidValue;
  p.P = c.P;
  p.segsh = c.segsh;
  if (quad_lds(c, p.H, 4) > kQuadMaxLds) return hipErrorInvalidValue;
  // An array for each direction present, and the registers of the scans that run:
  // both decide how many workgroups share a compute unit (2048 planes, four arrays and
  // every scan's registers -> this: top-to-bottom alone 72 x 72 fp32 286 -> 157 us, bf16
  // 297 -> 89, 200 x 4 fp32 367 -> 121; left-to-right alone 64 x 128 bf16 341 -> 186).
  const int lds = (int)quad_lds(c, p.H, p.n);
  const bool v = p.slot[0] >= 0 || p.slot[1] >= 0, h = p.slot[2] >= 0 || p.slot[3] >= 0;
  const int npv = v ? c.npv : 1, nph = h ? c.nph : 1;
  if constexpr (VL > 4) {  // bf16 rows of 4 to 7: 8-byte vectors
    if (p.W < VL && p.W >= 4 && nph == 1) return launch_quad_bwd_k<T, 1, 1, 4, LG, 2>(p, lds, st);
  }
  if (p.W < VL) {
    switch (nph) {
      case 1: return launch_quad_bwd_k<T, 1, 1, 1, LG>(p, lds, st);
      case 2: return launch_quad_bwd_k<T, 1, 2, 1, LG>(p, lds, st);
      default: return launch_quad_bwd_k<T, 1, 4, 1, LG>(p, lds, st);
    }
  }
  // two vectors of a row also for planes of few rows, whose horizontal waves have most
  // lanes idle: more workgroups count more than long loads (2048 planes, eight -> two:
  // four directions 16 x 32 fp32 77 -> 60 us, 14 x 60 bf16 97 -> 62, 4 x 200 bf16 262 -> 146;
  // left-to-right alone 16 x 32 fp32 59 -> 33)
  if (p.W <= 2 * VL || p.H <= 16 || !h) {
    if (nph == 1)
      return npv == 1 ? launch_quad_bwd_k<T, 1, 1, VL, LG, 2>(p, lds, st)
           : npv == 2 ? launch_quad_bwd_k<T, 2, 1, VL, LG, 2>(p, lds, st)
                      : launch_quad_bwd_k<T, 4, 1, VL, LG, 2>(p, lds, st);
  }
  // a single horizontal direction runs on one wave of a workgroup: more of them, with
  // shorter loads (2048 planes: 72 x 72 bf16 284 -> 188 us, 96 x 96 fp32 539 -> 452), but
  // for fp32 planes of one row a lane over 10 KB (60 x 60 155 -> 190), as in the forward
  if (p.n == 1 && nph == 1 && (sizeof(T) == 2 || p.H * p.W <= 2560))
    return launch_quad_bwd_k<T, 1, 1, VL, LG, 4>(p, lds, st);
  if (p.n == 1 && nph == 2) return launch_quad_bwd_k<T, 1, 2, VL, LG, 4>(p, lds, st);
  // four arrays of a plane with both sides over 128 do not fit
  if (npv == 1 && nph == 1 && p.W <= 4 * VL) return launch_quad_bwd_k<T, 1, 1, VL, LG, 4>(p, lds, st);
  if (npv == 1)
    return nph == 1 ? launch_quad_bwd_k<T, 1, 1, VL, LG>(p, lds, st)
         : nph == 2 ? launch_quad_bwd_k<T, 1, 2, VL, LG>(p, lds, st)
                    : launch_quad_bwd_k<T, 1, 4, VL, LG>(p, lds, st);
  if (npv == 2)
    return nph == 1 ? launch_quad_bwd_k<T, 2, 1, VL, LG>(p, lds, st)
         : nph == 2 ? launch_quad_bwd_k<T, 2, 2, VL, LG>(p, lds, st)
                    : launch_quad_bwd_k<T, 2, 4, VL, LG>(p, lds, st);
  return nph == 1 ? launch_quad_bwd_k<T, 4, 1, VL, LG>(p, lds, st)
       : nph == 2 ? launch_quad_bwd_k<T, 4, 2, VL, LG>(p, lds, st) : hipErrorInvalidValue;
}

// Pair kernel: lines of at least 32 positions on both axes (two halves with
// halos), both axes' arrays in LDS.
inline int pair_pitch(int W, bool hz) { return hz ? (W | 1) : ((W + 2 * kHalo + 1) | 1); }
inline int64_t pair_lds(int H, int W, bool hz) {
  return (int64_t)2 * (H + (hz ? 2 * kHalo : 0) + 1) * pair_pitch(W, hz) * 4;
}
inline bool pair_bwd_size_fits(int H, int W) {
  constexpr int64_t most = kQuadMaxLds - 2 * 2 * 2 * kHalo * 4;
  return H >= 32 && W >= 32 && H <= 256 && W <= 256 && pair_lds(H, W, false) <= most && pair_lds(H, W, true) <= most;
}

template <typename T, bool HZ, int NP, bool LG>
hipError_t launch_pair_axis_k(const QBwdParams& p, int finish, int lds, hipStream_t st) {
  constexpr int VL = 16 / (int)sizeof(T);
  auto kern = pair_bwd_kernel<T, HZ, NP, VL, LG>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)p.planes), dim3(256), lds, st, p, finish);
  return hipGetLastError();
}
template <typename T, bool HZ, bool LG>
hipError_t launch_pair_axis(QBwdParams p, int finish, hipStream_t st) {
  p.P = pair_pitch(p.W, HZ);
  const int lds = (int)pair_lds(p.H, p.W, HZ);
  const int half = ((HZ ? p.H : p.W) + 1) / 2;  // kept by a wave, rounded up to whole lanes
  if (half + kHalo <= 64) return launch_pair_axis_k<T, HZ, 1, LG>(p, finish, lds, st);
  if (half + 1 + kHalo <= 128) return launch_pair_axis_k<T, HZ, 2, LG>(p, finish, lds, st);
  return launch_pair_axis_k<T, HZ, 4, LG>(p, finish, lds, st);
}
// both axes: the vertical launch first (sums into the workspace), the
// horizontal one adds its own and finishes; an axis without directions is left out
template <typename T, bool LG>
hipError_t launch_pair_bwd(QBwdParams p, hipStream_t st) {
  if (!pair_bwd_size_fits(p.H, p.W) || p.lam_pd || p.u_pd || p.y_pd) return hipErrorInvalidValue;
  const bool v = p.slot[0] >= 0 || p.slot[1] >= 0, h = p.slot[2] >= 0 || p.slot[3] >= 0;
  if (!v || !h) p.hsum = p.gsum = nullptr;
  if (v) {
    hipError_t e = launch_pair_axis<T, false, LG>(p, h ? 0 : 1, st);
    if (e != hipSuccess || !h) return e;
  }
  return launch_pair_axis<T, true, LG>(p, 1, st);
}

inline QBwdParams quad_bwd_params(const ResidentBwdArgs& a) {
  QBwdParams p{};
  p.dy = a.dy; p.x = a.x; p.lam = a.lam; p.w = a.w; p.u = a.u;
  p.dx = a.dx; p.dw = a.dw; p.dlam = a.dlam; p.du = a.du;
  p.npc = a.planes * (int64_t)a.H * a.W;
  p.planes = a.planes;
  p.H = a.H; p.W = a.W;
  int n = 0;
  for (int d = 0; d < 4; ++d) p.slot[d] = (a.mask >> d) & 1 ? n++ : -1;
  p.n = n;
  p.gh = (a.group_h > 0 && a.group_h < a.H) ? a.group_h : a.H;
  p.gw = (a.group_w > 0 && a.group_w < a.W) ? a.group_w : a.W;
  p.renorm = a.renorm;
  p.lam_pd = a.lam_pd; p.u_pd = a.u_pd; p.y_pd = a.y_pd;
  return p;
}

}  // namespace gspn
