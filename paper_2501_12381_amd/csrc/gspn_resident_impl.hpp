// What the resident forwards share, and their dispatch.  A workgroup owns whole
// planes and runs every direction of the mask in one launch; a line (row or
// column) of a plane is held by one wave (or two, sharing it), each lane owning
// NP consecutive positions, so the neighbour exchange of Sec. 3.3's three-way
// connection is two DPP wave shifts per line, with no barrier.  The square
// sizes 16, 28, 32, 56 and 64 run on gspn_fixed_impl.hpp, 128 x 128 on
// gspn_wide_impl.hpp, every other one on gspn_quadfwd_impl.hpp.
#pragma once

#include "gspn_device.hpp"
#include "gspn_launch.hpp"

namespace gspn {

// ---------------------------------------------------------------------------
// packed element groups: N consecutive elements of T kept as raw 32-bit words
// until the step that uses them (the convert of bf16 is one shift or mask)
// ---------------------------------------------------------------------------
template <typename T, int N>
struct Pack;

template <int N>
struct Pack<float, N> {
  static constexpr int kWords = N;
  uint32_t w[N];
  __device__ __forceinline__ void load(const float* __restrict__ p) {
    if constexpr (N == 1) {
      w[0] = __float_as_uint(p[0]);
    } else if constexpr (N == 2) {
      const uint2 t = *reinterpret_cast<const uint2*>(p);
      w[0] = t.x; w[1] = t.y;
    } else {
#pragma unroll
      for (int i = 0; i < N; i += 4) {
        const uint4 t = *reinterpret_cast<const uint4*>(p + i);
        w[i] = t.x; w[i + 1] = t.y; w[i + 2] = t.z; w[i + 3] = t.w;
      }
    }
  }
  __device__ __forceinline__ float get(int i) const { return __uint_as_float(w[i]); }
};

template <int N>
struct Pack<bf16, N> {
  static constexpr int kWords = (N + 1) / 2;
  uint32_t w[kWords];
  __device__ __forceinline__ void load(const bf16* __restrict__ p) {
    if constexpr (N == 1) {
      w[0] = *reinterpret_cast<const uint16_t*>(p);
    } else if constexpr (N == 2) {
      w[0] = *reinterpret_cast<const uint32_t*>(p);
    } else if constexpr (N == 4) {
      const uint2 t = *reinterpret_cast<const uint2*>(p);
      w[0] = t.x; w[1] = t.y;
    } else {
#pragma unroll
      for (int i = 0; i < N; i += 8) {
        const uint4 t = *reinterpret_cast<const uint4*>(p + i);
        w[i / 2] = t.x; w[i / 2 + 1] = t.y; w[i / 2 + 2] = t.z; w[i / 2 + 3] = t.w;
      }
    }
  }
  __device__ __forceinline__ float get(int i) const { return (i & 1) ? bf_hi(w[i >> 1]) : bf_lo(w[i >> 1]); }
};

// One step of the recurrence for the lane's NP positions (Eq. 1):
//   h[q] = w0 * hprev[q-1] + w1 * hprev[q] + w2 * hprev[q+1] + lam * x
// with the neighbours outside the lane taken from the adjacent lanes.
template <int NP>
__device__ __forceinline__ void line_step(const float (&xv)[NP], const float (&lv)[NP],
                                          const float (&a)[NP], const float (&b)[NP],
                                          const float (&c)[NP], const bool (&valid)[NP],
                                          float (&hp)[NP]) {
  const float left = from_prev_lane(hp[NP - 1]);
  const float right = from_next_lane(hp[0]);
  float h[NP];
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const float hl = q == 0 ? left : hp[q - 1];
    const float hr = q == NP - 1 ? right : hp[q + 1];
    float v = lv[q] * xv[q];
    v = fmaf(a[q], hl, v);
    v = fmaf(b[q], hp[q], v);
    v = fmaf(c[q], hr, v);
    h[q] = valid[q] ? v : 0.f;
  }
#pragma unroll
  for (int q = 0; q < NP; ++q) hp[q] = h[q];
}

// Eq. 6 on the lane's NP positions (LG: the weight maps hold logits): w0..w2
// of each position in place, renormalised over on-line neighbours when
// renorm is set.  Positions past the line keep whatever they get (their h is
// forced to 0).
template <bool LG, int NP>
__device__ __forceinline__ void norm_weights(float (&a)[NP], float (&b)[NP], float (&c)[NP], int pos0, int Pn,
                                             bool renorm) {
  if constexpr (LG) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const Norm3 r = normalize3(a[q], b[q], c[q], pos0 + q == 0, pos0 + q == Pn - 1, renorm);
      a[q] = r.w[0];
      b[q] = r.w[1];
      c[q] = r.w[2];
    }
  }
}

// y = u * acc over one plane with VE-element vectors (W % VE == 0), in
// batches of U vectors per thread whose loads are issued together.
template <typename T, int VE>
__device__ __forceinline__ void epilogue(const T* __restrict__ ub, T* __restrict__ yb,
                                         const float* __restrict__ ac, int H, int W, int P, int tid) {
  constexpr int U = 16;
  const int per_row = W / VE;
  const int n = H * per_row;
  for (int base = tid; base < n; base += 128 * U) {
    Pack<T, VE> uv[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int e = base + k * 128 < n ? base + k * 128 : base;
      const int r = e / per_row, c = (e - r * per_row) * VE;
      uv[k].load(ub + (int64_t)r * W + c);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int e = base + k * 128;
      if (e < n) {
        const int r = e / per_row, c = (e - r * per_row) * VE;
        float yv[VE];
#pragma unroll
        for (int q = 0; q < VE; ++q) yv[q] = uv[k].get(q) * ac[r * P + c + q];
        stv<VE>(yb + (int64_t)r * W + c, yv);
      }
    }
  }
}

struct ResFwdParams {
  const void* x;
  const void* lam;
  const void* w;
  const void* u;
  void* y;
  int64_t npc;  // elements per (B, C, H, W) tensor = stride between weight maps
  int64_t planes;
  int H, W;
  int slot[4];  // T2B, B2T, L2R, R2L -> weight slot or -1
  int vec_y;
  int gh, gw;   // local-GSPN group lengths along rows and columns (the line count: global)
  int grouped;  // gh < H or gw < W
  // per direction (T2B, B2T, L2R, R2L): bit l of word l / 64 set when line l
  // (< 128) starts a group in that direction's scan order
  uint64_t gstart[4][2];
  int logits, renorm;  // w holds Eq. 6 logits (renorm: normalised over on-line neighbours)
};

}  // namespace gspn

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
namespace gspn {
// Sizes with a specialised forward kernel (square planes).
inline bool fixed_size_supported(int H, int W) {
  return H == W && (H == 16 || H == 28 || H == 32 || H == 56 || H == 64);
}
template <typename T, int S> hipError_t launch_fixed(const ResFwdParams& p, hipStream_t st);
template <typename T> hipError_t launch_wide(const ResFwdParams& p, hipStream_t st);
namespace resident_detail {

constexpr int kMaxLds = 160 * 1024;  // LDS per CU on gfx950
constexpr int kMaxLine = 256;        // longest line one wave holds (64 lanes x 4 positions)

inline bool al(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

}  // namespace resident_detail

template <typename T>
hipError_t resident_fwd_t(const ResidentFwdArgs& a) {
  using namespace resident_detail;
  if (a.u_pd && !a.y_pd) return hipErrorInvalidValue;  // a merged y with per-direction u: streaming family
  const bool fixed = a.use_fixed && !a.lam_pd && !a.y_pd && fixed_size_supported(a.H, a.W) && al(a.x, 16) &&
                     al(a.lam, 16) && al(a.w, 16);
  // persistent, every input read once
  const bool wide = a.use_fixed && !a.lam_pd && !a.y_pd && a.H == 128 && a.W == 128 && al(a.x, 16) && al(a.lam, 16) &&
                    al(a.w, 16) && al(a.u, 16) && al(a.y, 16) && (a.group_h <= 0 || a.group_h >= a.H) &&
                    (a.group_w <= 0 || a.group_w >= a.W);
  if (!fixed && !wide) return sizeof(T) == 4 ? quad_fwd_f32(a) : quad_fwd_bf16(a);
  ResFwdParams p{};
  p.x = a.x; p.lam = a.lam; p.w = a.w; p.u = a.u; p.y = a.y;
  p.npc = (int64_t)a.planes * a.H * a.W;
  p.planes = a.planes;
  p.H = a.H; p.W = a.W;
  int n = 0;
  for (int d = 0; d < 4; ++d) p.slot[d] = (a.mask >> d) & 1 ? n++ : -1;
  p.gh = (a.group_h > 0 && a.group_h < a.H) ? a.group_h : a.H;
  p.gw = (a.group_w > 0 && a.group_w < a.W) ? a.group_w : a.W;
  p.grouped = p.gh < a.H || p.gw < a.W;
  p.logits = a.logits;
  p.renorm = a.renorm;
  for (int d = 0; d < 4; ++d) {
    const bool hz = d >= 2, rev = d & 1;
    const int L = hz ? a.W : a.H, G = hz ? p.gw : p.gh;
    p.gstart[d][0] = p.gstart[d][1] = 0;
    for (int l = 0; l < L && l < 128; ++l)
      if (rev ? ((l + 1) % G == 0 || l == L - 1) : (l % G == 0)) p.gstart[d][l >> 6] |= 1ull << (l & 63);
  }
  // epilogue vectors: 16 bytes if rows allow, else 8 bytes, else scalars
  const int v16 = 16 / (int)sizeof(T), v8 = 8 / (int)sizeof(T);
  p.vec_y = (a.W % v16 == 0 && al(a.u, 16) && al(a.y, 16)) ? 2 : (a.W % v8 == 0 && al(a.u, 8) && al(a.y, 8)) ? 1 : 0;
  hipStream_t st = (hipStream_t)a.stream;
  if (wide) return launch_wide<T>(p, st);
  switch (a.H) {
    case 16: return launch_fixed<T, 16>(p, st);
    case 28: return launch_fixed<T, 28>(p, st);
    case 32: return launch_fixed<T, 32>(p, st);
    case 56: return launch_fixed<T, 56>(p, st);
    default: return launch_fixed<T, 64>(p, st);
  }
}

// Planes that a forced resident family takes (AUTO goes by quad_fwd_fits beyond).
// narr: the directions present for unmerged outputs, else 1.  The kernels of unmerged
// outputs hold no array; what a caller could force, and what was refused, stays so.
inline bool resident_fwd_fits(int H, int W, int narr = 1) {
  using namespace resident_detail;
  if (H > kMaxLine || W > kMaxLine) return false;
  return (int64_t)narr * (H + 1) * (W + 1 + (W & 1)) * 4 <= kMaxLds;
}

}  // namespace gspn
