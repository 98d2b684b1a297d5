// Scans of planes that fit a compute unit's LDS, for any size and alignment:
// the building blocks of the generic resident kernels (forward in
// gspn_quadfwd_impl.hpp, backward in gspn_quadbwd_impl.hpp).
//
// One wave runs one direction, a lane owning NP consecutive positions of the
// line, so the three-way neighbour exchange is two DPP shifts a line and the
// directions run side by side, one wave on each SIMD.  Small planes (lines of
// at most 31 positions) share a wave in segments of 16 or 32 lanes whose last
// lanes hold zeros.  Vertical scans read one vector of NP elements a row and
// map, horizontal ones TV vectors of 16 bytes of every row they own; both keep
// a ring of them in flight (idle rows or groups of columns before the first
// one fill the ring's turns, so that every load is unconditional: a load
// inside a branch would be waited for where the branch ends).  Buffer loads need no alignment, so odd widths and
// element-aligned tensors take the same path:
//   * a row's last vector, when it would cross the row's end, starts where it
//     ends at the row's end and is shifted into place;
//   * a row's last vector of columns starts W - VL columns in, and the columns
//     already done are skipped;
//   * lanes past the line (and planes past the tensor) read at an offset out
//     of the resource's range, which returns zero without traffic.
#pragma once

#include "gspn_device.hpp"
#include "gspn_launch.hpp"
#include "gspn_resident_impl.hpp"
#include "gspn_vpass_impl.hpp"

namespace gspn {

// NP elements as loaded: a Pack, or for one bf16 the 16 bits themselves (a
// Pack's 32-bit word would be widened at the load, and so wait for it)
template <typename T, int NP>
struct QPack : Pack<T, NP> {};
template <>
struct QPack<bf16, 1> {
  uint16_t h;
  __device__ __forceinline__ float get(int) const { return __uint_as_float((uint32_t)h << 16); }
};
template <typename T, int NP>
__device__ __forceinline__ void q_load(QPack<T, NP>& pk, wide_rsrc_t r, int voff, int soff) {
  if constexpr (sizeof(T) * NP == 2) pk.h = __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
  else wide_load<T, NP>(pk, r, voff, soff);
}

template <typename T, int NP>
__device__ __forceinline__ void q_store(const float (&v)[NP], wide_rsrc_t r, int voff, int soff) {
  if constexpr (sizeof(T) * NP == 2) {
    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)pack_bf2(v[0], 0.f), r, voff, soff, 0);
  } else if constexpr (sizeof(T) * NP == 4) {
    if constexpr (sizeof(T) == 2) __builtin_amdgcn_raw_buffer_store_b32(pack_bf2(v[0], v[1]), r, voff, soff, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[0]), r, voff, soff, 0);
  } else if constexpr (sizeof(T) * NP == 8) {
    vp_u32x2 t;
    if constexpr (sizeof(T) == 2) t = vp_u32x2{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
    else t = vp_u32x2{__float_as_uint(v[0]), __float_as_uint(v[1])};
    __builtin_amdgcn_raw_buffer_store_b64(t, r, voff, soff, 0);
  } else {
    vp_store<T, NP>(v, r, voff, soff);
  }
}

template <typename T>
__device__ __forceinline__ void q_store_elem(float v, wide_rsrc_t r, int voff, int soff) {
  const float t[1] = {v};
  q_store<T, 1>(t, r, voff, soff);
}

// drop the first sh elements of the pack (sh < NP, per lane), zeros behind the rest
template <typename T, int NP>
__device__ __forceinline__ void q_shift(QPack<T, NP>& p, int sh) {
  if constexpr (NP == 2 && sizeof(T) == 2) {
    p.w[0] >>= 16 * sh;
  } else if constexpr (NP == 4 && sizeof(T) == 2) {
    const uint64_t v = (((uint64_t)p.w[1] << 32) | p.w[0]) >> (16 * sh);
    p.w[0] = (uint32_t)v;
    p.w[1] = (uint32_t)(v >> 32);
  } else if constexpr (NP == 2) {
    p.w[0] = sh ? p.w[1] : p.w[0];
    p.w[1] = sh ? 0u : p.w[1];
  } else if constexpr (NP == 4) {
    const bool s1 = sh & 1, s2 = sh & 2;
    const uint32_t t0 = s1 ? p.w[1] : p.w[0], t1 = s1 ? p.w[2] : p.w[1], t2 = s1 ? p.w[3] : p.w[2],
                   t3 = s1 ? 0u : p.w[3];
    p.w[0] = s2 ? t2 : t0;
    p.w[1] = s2 ? t3 : t1;
    p.w[2] = s2 ? 0u : t2;
    p.w[3] = s2 ? 0u : t3;
  }
}

// A buffer resource of its own four scalars: resources of equal sizes would
// share their last two, and the compiler then copies them together before
// every load (as many scalar instructions as the line step has vector ones).
__device__ __forceinline__ wide_rsrc_t q_rsrc(const void* base, int bytes) {
  int flags = 0x00020000;
  asm("" : "+s"(bytes), "+s"(flags));
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, bytes, flags);
}

// What a workgroup's planes look like: np planes of H x W from plane g0 on,
// LDS arrays of (H + 1) x P floats (the last row and column W are padding).
struct QPlanes {
  int H, W, P, np;
  int segsh;  // log2 of the lanes per plane
};

// A line shared by two waves (pair kernel): wave 0 keeps positions [0, K) and
// carries kHalo of wave 1's, wave 1 the rest and kHalo of wave 0's.  Each
// scans its span alone; every kHalo lines they exchange their edges.  A wave
// has LDS columns (rows, for a horizontal scan) of its own for its whole span:
// position p of wave 1's lie 2 kHalo further on.
// An exchange has one barrier; the next one writes the other buffer (par, the
// running block's parity), since a wave may reach it before the other wave has
// read what this one brought.
constexpr int kHalo = 8;
struct QHalf {
  int hf, K;
  float* buf;  // [2 parities][2 sides][kHalo]
};
template <int NP, typename F>
__device__ __forceinline__ void q_exchange(float (&v)[NP], const QHalf& x, int pos0, int par, F&& barrier) {
  float* lo = x.buf + par * 2 * kHalo;  // positions [K - kHalo, K), then [K, K + kHalo)
  const int j = pos0 - (x.K - kHalo);
  const bool in0 = j >= 0 && j < kHalo, in1 = j >= kHalo && j < 2 * kHalo;
  if (x.hf ? in1 : in0) {
#pragma unroll
    for (int q = 0; q < NP; ++q) lo[j + q] = v[q];
  }
  barrier();
  if (x.hf ? in0 : in1) {
#pragma unroll
    for (int q = 0; q < NP; ++q) v[q] = lo[j + q];
  }
}

// Lane geometry of a vertical scan (positions are columns).
template <typename T, int NP>
struct QV {
  int voff;         // byte offset of the lane's vector in a row of its plane
  int sh;           // elements to drop from it
  int nval;         // positions of the lane on the line
  bool tail;        // some lane is partly past the line (uniform)
  int pos0;
  int aoff[NP];     // LDS offsets in a row (the padding column past the line)
  bool valid[NP];
  bool kept;        // the lane's values are this wave's to store
  __device__ __forceinline__ QV(const QPlanes& g, int lane) {
    const int seg = lane >> g.segsh, sl = lane & ((1 << g.segsh) - 1);
    pos0 = sl * NP;
    const int left = seg < g.np ? g.W - pos0 : 0;
    nval = left < 0 ? 0 : (left > NP ? NP : left);
    sh = (nval > 0 && nval < NP && g.W >= NP) ? NP - nval : 0;
    tail = g.W % NP != 0;
    voff = nval > 0 ? (seg * g.H * g.W + pos0 - sh) * (int)sizeof(T) : kWideOob;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      valid[q] = q < nval;
      aoff[q] = valid[q] ? pos0 + q : g.W;
    }
    kept = true;
  }
  // half of a plane's columns and kHalo of the other half's
  __device__ __forceinline__ QV(const QPlanes& g, int lane, const QHalf& x) {
    const int ss = x.hf ? x.K - kHalo : 0, se = x.hf ? g.W : x.K + kHalo;
    pos0 = ss + lane * NP;
    const int left = se - pos0;
    nval = left < 0 ? 0 : (left > NP ? NP : left);
    sh = (nval > 0 && nval < NP) ? NP - nval : 0;
    tail = g.W % NP != 0;
    voff = nval > 0 ? (pos0 - sh) * (int)sizeof(T) : kWideOob;
    kept = x.hf ? pos0 >= x.K : pos0 < x.K;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      valid[q] = q < nval;
      aoff[q] = valid[q] ? pos0 + q + (x.hf ? 2 * kHalo : 0) : g.W + 2 * kHalo;
    }
  }
};

// Lane geometry of a horizontal scan (positions are rows).
template <typename T, int NP>
struct QH {
  int voff[NP];
  int voffs[NP];    // the same for stores (out of range for rows of the other half)
  int pos0;
  int aoff[NP];     // LDS offsets of the rows (the padding row past the line)
  bool valid[NP];
  __device__ __forceinline__ QH(const QPlanes& g, int lane) {
    const int seg = lane >> g.segsh, sl = lane & ((1 << g.segsh) - 1);
    pos0 = sl * NP;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      valid[q] = seg < g.np && pos0 + q < g.H;
      voff[q] = valid[q] ? (seg * g.H + pos0 + q) * g.W * (int)sizeof(T) : kWideOob;
      voffs[q] = voff[q];
      aoff[q] = (valid[q] ? pos0 + q : g.H) * g.P;
    }
  }
  // half of a plane's rows and kHalo of the other half's
  __device__ __forceinline__ QH(const QPlanes& g, int lane, const QHalf& x) {
    const int ss = x.hf ? x.K - kHalo : 0, se = x.hf ? g.H : x.K + kHalo;
    pos0 = ss + lane * NP;
    const bool kept = x.hf ? pos0 >= x.K : pos0 < x.K;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      valid[q] = pos0 + q < se;
      voff[q] = valid[q] ? (pos0 + q) * g.W * (int)sizeof(T) : kWideOob;
      voffs[q] = kept ? voff[q] : kWideOob;
      aoff[q] = (valid[q] ? pos0 + q + (x.hf ? 2 * kHalo : 0) : g.H + 2 * kHalo) * g.P;
    }
  }
};

// Vectors of a row read together by a horizontal scan of five or six maps (a
// cache line, less where the rows of a lane would not fit the registers).
template <int NP>
struct QVecs {
  static constexpr int TV = NP <= 2 ? 8 : 3;
};

// Rows in flight of a vertical scan, by the registers they take (a row of a
// narrow plane is few bytes: 16 rows of 46 lanes x 4 bytes x 5 maps are 15 KB).
template <typename T, int NP>
struct QRing {
  static constexpr int VW = Pack<T, NP>::kWords;
  static constexpr int RV = VW == 1 ? 16 : (VW == 2 ? 8 : 4);
};

// A lane's NP values of a row: one vector, unless the line's end cuts it.
template <typename T, int NP>
__device__ __forceinline__ void qv_store(const float (&v)[NP], wide_rsrc_t r, const QV<T, NP>& ln, int so) {
  q_store<T, NP>(v, r, ln.nval == NP && ln.kept ? ln.voff : kWideOob, so);
  if (NP > 1 && ln.tail) {
#pragma unroll
    for (int q = 0; q < NP - 1; ++q)
      q_store_elem<T>(v[q], r, (ln.nval < NP && q < ln.nval && ln.kept) ? ln.voff + (ln.sh + q) * (int)sizeof(T) : kWideOob, so);
  }
}

// Called with the values of the last line of every block of lines (at most
// kHalo of them) but the last: exchanges the edges of two waves that share the
// lines, where there are two.
struct QNoExchange {
  template <int NP>
  __device__ __forceinline__ void operator()(int, float (&)[NP]) const {}
};

// Where a scan reads lam * x from: the maps themselves, or an LDS array that
// holds the product (offsets of the lane's positions in it; one line ahead).
template <int NP>
struct QLamX {
  const float* lx;
  int off[NP];
};

// The rows of a vertical scan, in blocks of kHalo rows that are the same for
// both senses (rev: from the last block and its last row on); rows past the
// plane are idle: their loads are out of range and their line is H, the
// padding row.
struct QRows {
  int H, nb, rowb;
  bool rev;
  template <int R>
  __device__ __forceinline__ static QRows make(int H, int rowb, bool rev) {
    constexpr int UB = R > kHalo ? R / kHalo : 1;  // whole turns of the ring
    const int n = (H + kHalo - 1) / kHalo;
    return QRows{H, (n + UB - 1) / UB * UB, rowb, rev};
  }
  __device__ __forceinline__ int row(int s) const { return rev ? nb * kHalo - 1 - s : s; }
  __device__ __forceinline__ int line(int s) const { return min(max(row(s), 0), H); }
  __device__ __forceinline__ bool on(int s) const { return (unsigned)row(s) < (unsigned)H; }
  __device__ __forceinline__ int soff(int s) const { return on(s) ? row(s) * rowb : kWideOob; }
};

// Vertical scan of one direction (rev: rows from the last to the first).  rb:
// x, lam, w0, w1, w2, u (LX: x and lam unused, lam * x from LDS; UM: u is read
// too).  begin(block, blocks, first line) before every block, emit(line, next
// line, row offset, h, u pack) after every row, end(block, blocks) after every
// block.
// XE: the exchange precedes the last row's emit (whose receiver keeps the halo
// positions too), else it follows end().  With a QMerge it has to follow: in the
// middle block the exchange's barrier would otherwise come before the merge's
// second one and pair with the opposite direction's, which then reads the
// block's last row while it is still being stored.
template <typename T, int NP, int R, bool LG, bool UM, bool LX, bool XE = false, typename FB, typename F, typename FE,
          typename FX = QNoExchange>
__device__ __forceinline__ void qv_forward(const wide_rsrc_t (&rb)[6], const QV<T, NP>& ln, const QPlanes& g,
                                           bool rev, int grp, bool renorm, const QLamX<NP>& lam_x, FB&& begin,
                                           F&& emit, FE&& end, FX exchange = FX{}) {
  constexpr int M0 = LX ? 2 : 0, NM = UM ? 6 : 5, UB = R > kHalo ? R / kHalo : 1;
  typedef QPack<T, NP> PK;
  const int W = g.W;
  const QRows rows = QRows::make<R>(g.H, W * (int)sizeof(T), rev);
  PK ring[R][NM];
  auto load = [&](int k, int s) __attribute__((always_inline)) {
    const int so = rows.soff(s);
#pragma unroll
    for (int m = M0; m < NM; ++m) q_load<T, NP>(ring[k][m], rb[m], ln.voff, so);
  };
#pragma unroll
  for (int k = 0; k < R; ++k) {
    load(k, k);
    __builtin_amdgcn_sched_barrier(0);  // in the ring's order, so that the loop's waits match
  }
  float hp[NP], lxn[NP];
#pragma unroll
  for (int q = 0; q < NP; ++q) hp[q] = 0.f;
  auto read_lx = [&](int s) __attribute__((always_inline)) {  // idle rows: the (zeroed) padding row
    const int o = rows.line(s) * g.P;
#pragma unroll
    for (int q = 0; q < NP; ++q) lxn[q] = lam_x.lx[lam_x.off[q] + o];
  };
  if constexpr (LX) read_lx(0);
  // the row at which the state restarts next
  int nxt = rev ? (g.H - 1) / grp * grp - 1 : grp;
  const int nstep = rev ? -grp : grp;
  for (int b0 = 0; b0 < rows.nb; b0 += UB) {
#pragma unroll
    for (int ub = 0; ub < UB; ++ub) {
      const int s0 = (b0 + ub) * kHalo;
      begin(b0 + ub, rows.nb, rows.line(s0));
#pragma unroll
      for (int kk = 0; kk < kHalo; ++kk) {
        const int s = s0 + kk, k = (ub * kHalo + kk) % R;
        PK v[NM];
#pragma unroll
        for (int m = M0; m < NM; ++m) v[m] = ring[k][m];
        if (NP > 1 && ln.tail) {
#pragma unroll
          for (int m = M0; m < NM; ++m) q_shift<T, NP>(v[m], ln.sh);
        }
        float xv[NP], lv[NP], a[NP], b[NP], c[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          xv[q] = LX ? lxn[q] : v[0].get(q);
          lv[q] = LX ? 1.f : v[1].get(q);
          a[q] = v[2].get(q);
          b[q] = v[3].get(q);
          c[q] = v[4].get(q);
        }
        if constexpr (LX) read_lx(s + 1);
        if (rows.row(s) == nxt) {  // a group starts at this row
#pragma unroll
          for (int q = 0; q < NP; ++q) hp[q] = 0.f;
          nxt += nstep;
        }
        norm_weights<LG, NP>(a, b, c, ln.pos0, W, renorm);
        line_step<NP>(xv, lv, a, b, c, ln.valid, hp);
        load(k, s + R);
        if (XE && kk == kHalo - 1 && b0 + ub + 1 < rows.nb) exchange((b0 + ub) & 1, hp);
        emit(rows.line(s), rows.line(s + 1), rows.soff(s), hp, v[NM - 1]);
      }
      end(b0 + ub, rows.nb);
      if (!XE && b0 + ub + 1 < rows.nb) exchange((b0 + ub) & 1, hp);
    }
  }
}

// A vector's elements in reverse.
template <int VL>
__device__ __forceinline__ void q_reverse(QPack<float, VL>& p) {
#pragma unroll
  for (int i = 0; i < VL / 2; ++i) {
    const uint32_t t = p.w[i];
    p.w[i] = p.w[VL - 1 - i];
    p.w[VL - 1 - i] = t;
  }
}
template <int VL>
__device__ __forceinline__ void q_reverse(QPack<bf16, VL>& p) {
  if constexpr (VL > 1) {
    constexpr int N = VL / 2;
    uint32_t t[N];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = __builtin_amdgcn_alignbit(p.w[N - 1 - i], p.w[N - 1 - i], 16);
#pragma unroll
    for (int i = 0; i < N; ++i) p.w[i] = t[i];
  }
}
template <int VL>
__device__ __forceinline__ void q_reverse(float (&v)[VL]) {
#pragma unroll
  for (int i = 0; i < VL / 2; ++i) {
    const float t = v[i];
    v[i] = v[VL - 1 - i];
    v[VL - 1 - i] = t;
  }
}

// The columns of a horizontal scan, in vectors of VL in visiting order (the
// row's last vector starts VL columns before its end and overlaps the one
// before it), read in groups of TV: each map's vectors of a row back to back,
// since they share cache lines that the many rows of a wave would otherwise
// push out of the L1 before the next vector is read (one vector at a time
// measured 540 us on 1280 planes of 96 x 168 bf16: every line read from the L2
// once per vector).  The vectors of a group go through one copy of the code
// (visit), a switch picks the registers; unrolled, the steps of a group would
// not fit the instruction cache.
template <typename T, int NP, int VL, int TV, int R, int M0, int NM, typename FV>
__device__ __forceinline__ void qh_columns(const wide_rsrc_t* rb, const QH<T, NP>& ln, int W, bool rev, FV&& visit) {
  typedef QPack<T, VL> PK;
  constexpr int ES = (int)sizeof(T);
  const int nt = (W + VL - 1) / VL, ng = (nt + TV - 1) / TV;
  auto lo = [&](int ti) { return (rev ? nt - 1 - ti : ti) * VL; };
  PK ring[R][NM][NP][TV];
  auto load = [&](int k, int gi) __attribute__((always_inline)) {
#pragma unroll
    for (int m = M0; m < NM; ++m)
#pragma unroll
      for (int q = 0; q < NP; ++q)
#pragma unroll
        for (int v = 0; v < TV; ++v) {
          const int ti = gi * TV + v;
          q_load<T, VL>(ring[k][m][q][v], rb[m], ln.voff[q],
                        (unsigned)ti < (unsigned)nt ? min(lo(ti), W - VL) * ES : kWideOob);
        }
  };
  const int gb = -((R - ng % R) % R);  // idle groups fill the ring's first turn
#pragma unroll
  for (int k = 0; k < R; ++k) {
    load(k, gb + k);
    __builtin_amdgcn_sched_barrier(0);  // in the ring's order, so that the loop's waits match
  }
  for (int G0 = gb; G0 < ng; G0 += R) {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int t0 = (G0 + k) * TV, n = G0 + k < 0 ? 0 : min(TV, nt - t0);
      for (int vi = 0; vi < n; ++vi) {
        PK v[NM][NP];
        static_for<0, TV>([&](auto vc) __attribute__((always_inline)) {
          constexpr int c = decltype(vc)::value;
          if (vi == c) {
#pragma unroll
            for (int m = M0; m < NM; ++m)
#pragma unroll
              for (int q = 0; q < NP; ++q) v[m][q] = ring[k][m][q][c];
          }
        });
        if (VL > 1 && rev) {
#pragma unroll
          for (int m = M0; m < NM; ++m)
#pragma unroll
            for (int q = 0; q < NP; ++q) q_reverse<VL>(v[m][q]);
        }
        const int ti = t0 + vi, l = lo(ti);
        visit(ti, nt, l, min(l, W - VL), v);
      }
      load(k, G0 + k + R);
    }
  }
}

// Horizontal scan of one direction (rev: columns from the last to the first).
// begin(ti, nt, first column) before every vector, emit(col, visited element e of the vector,
// whether the vector overlaps the one before it, h, last map's vectors in
// visiting order) after every column, end(ti, nt, overlaps, first column)
// after every vector.
// XE: the exchange precedes the last column's emit (whose receiver keeps the
// halo positions too), else it follows end().
template <typename T, int NP, int VL, int TV, int R, bool LG, bool UM, bool LX, bool XE = false, typename FB,
          typename F, typename FT, typename FX = QNoExchange>
__device__ __forceinline__ void qh_forward(const wide_rsrc_t (&rb)[6], const QH<T, NP>& ln, const QPlanes& g, bool rev,
                                           int grp, bool renorm, const QLamX<NP>& lam_x, FB&& begin, F&& emit, FT&& end,
                                           FX exchange = FX{}) {
  constexpr int M0 = LX ? 2 : 0, NM = UM ? 6 : 5, XV = kHalo / VL;
  typedef QPack<T, VL> PK;
  const int W = g.W, H = g.H;
  float hp[NP], lxn[NP];
#pragma unroll
  for (int q = 0; q < NP; ++q) hp[q] = 0.f;
  auto read_lx = [&](int c) __attribute__((always_inline)) {
    const int o = (unsigned)c < (unsigned)W ? c : 0;
#pragma unroll
    for (int q = 0; q < NP; ++q) lxn[q] = lam_x.lx[lam_x.off[q] + o];
  };
  if constexpr (LX) read_lx(rev ? W - 1 : 0);
  int nxt = rev ? (W - 1) / grp * grp - 1 : grp;  // the column at which the state restarts next
  const int nstep = rev ? -grp : grp;
  qh_columns<T, NP, VL, TV, R, M0, NM>(rb, ln, W, rev, [&](int ti, int nt, int lo, int c0, const PK (&v)[NM][NP])
                                       __attribute__((always_inline)) {
    begin(ti, nt, rev ? c0 + VL - 1 : lo);
    const bool cut = c0 != lo;
    const bool xch = (ti + 1) % XV == 0 && ti + 1 < nt;
    auto step = [&](int e) __attribute__((always_inline)) {
      const int col = rev ? c0 + VL - 1 - e : c0 + e;
      if (VL > 1 && col < lo) return;
      if (col == nxt) {  // a group starts at this column
#pragma unroll
        for (int q = 0; q < NP; ++q) hp[q] = 0.f;
        nxt += nstep;
      }
      float xv[NP], lv[NP], a[NP], b[NP], c[NP];
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        xv[q] = LX ? lxn[q] : v[0][q].get(e);
        lv[q] = LX ? 1.f : v[1][q].get(e);
        a[q] = v[2][q].get(e);
        b[q] = v[3][q].get(e);
        c[q] = v[4][q].get(e);
      }
      if constexpr (LX) read_lx(rev ? col - 1 : col + 1);
      norm_weights<LG, NP>(a, b, c, ln.pos0, H, renorm);
      line_step<NP>(xv, lv, a, b, c, ln.valid, hp);
      if (XE && xch && col == (rev ? lo : c0 + VL - 1)) exchange((ti / XV) & 1, hp);
      emit(col, e, cut, hp, v[NM - 1]);
    };
#pragma unroll
    for (int e = 0; e < VL; ++e) step(e);
    end(ti, nt, cut, c0);
    if (!XE && xch) exchange((ti / XV) & 1, hp);
  });
}

// The adjoint's line: g of the lane's positions from the products of the line
// done before (a_k = w_k g) ...
template <int NP>
__device__ __forceinline__ void q_adjoint_g(const float (&uv)[NP], const float (&dyv)[NP], const bool (&valid)[NP],
                                            const float (&a0)[NP], const float (&a1)[NP], const float (&a2)[NP],
                                            float (&g)[NP]) {
  const float ar = from_next_lane(a0[0]), al = from_prev_lane(a2[NP - 1]);
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const float an = q == NP - 1 ? ar : a0[q + 1];
    const float ap = q == 0 ? al : a2[q - 1];
    const float gv = fmaf(uv[q], dyv[q], a1[q] + an + ap);
    g[q] = valid[q] ? gv : 0.f;
  }
}
// ... and from g and the state the line read, its own products and dw.
template <int NP, bool LG>
__device__ __forceinline__ void q_adjoint_w(const float (&w0)[NP], const float (&w1)[NP], const float (&w2)[NP],
                                            const float (&hv)[NP], const float (&g)[NP], int pos0, int Pn, bool renorm,
                                            bool rst, float (&a0)[NP], float (&a1)[NP], float (&a2)[NP],
                                            float (&dv)[3][NP]) {
  const float hr = from_next_lane(hv[0]), hl = from_prev_lane(hv[NP - 1]);
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    float wa = w0[q], wb = w1[q], wc = w2[q];
    Norm3 nr;
    if constexpr (LG) {
      nr = normalize3(wa, wb, wc, pos0 + q == 0, pos0 + q == Pn - 1, renorm);
      wa = nr.w[0];
      wb = nr.w[1];
      wc = nr.w[2];
    }
    a0[q] = wa * g[q];
    a1[q] = wb * g[q];
    a2[q] = wc * g[q];
    dv[0][q] = g[q] * (q == 0 ? hl : hv[q - 1]);
    dv[1][q] = g[q] * hv[q];
    dv[2][q] = g[q] * (q == NP - 1 ? hr : hv[q + 1]);
    if constexpr (LG) norm3_vjp(nr, dv[0][q], dv[1][q], dv[2][q]);
  }
  if (rst) {  // uniform
#pragma unroll
    for (int q = 0; q < NP; ++q) a0[q] = a1[q] = a2[q] = 0.f;
  }
}

// Adjoint of a vertical direction (rev: of the bottom-to-top scan; rows are
// visited against the scan order): reads h from arr, leaves g there, writes dw.
// rb: u, dy, w0, w1, w2; rd: the three dw maps.
template <typename T, int NP, int R, bool LG, typename FX = QNoExchange>
__device__ __forceinline__ void qv_adjoint(const wide_rsrc_t (&rb)[5], const wide_rsrc_t (&rd)[3], const QV<T, NP>& ln,
                                           const QPlanes& g, float* __restrict__ arr, bool rev, int grp, bool renorm,
                                           FX exchange = FX{}) {
  constexpr int UB = R > kHalo ? R / kHalo : 1;
  typedef QPack<T, NP> PK;
  const int H = g.H, W = g.W, P = g.P;
  const QRows rows = QRows::make<R>(H, W * (int)sizeof(T), !rev);
  PK ring[R][5];
  auto load = [&](int k, int s) __attribute__((always_inline)) {
    const int so = rows.soff(s);
#pragma unroll
    for (int m = 0; m < 5; ++m) q_load<T, NP>(ring[k][m], rb[m], ln.voff, so);
  };
#pragma unroll
  for (int k = 0; k < R; ++k) {
    load(k, k);
    __builtin_amdgcn_sched_barrier(0);  // in the ring's order, so that the loop's waits match
  }
  float a0[NP], a1[NP], a2[NP], hn[NP];
#pragma unroll
  for (int q = 0; q < NP; ++q) a0[q] = a1[q] = a2[q] = 0.f;
  // h of the row visited next: the previous row of the current one in scan
  // order (past the last row whatever is there: that row starts a group; the
  // padding column holds the zeros the scan left for positions past the line)
  auto read_h = [&](int s) __attribute__((always_inline)) {
    const int o = rows.line(s) * P;
#pragma unroll
    for (int q = 0; q < NP; ++q) hn[q] = arr[o + ln.aoff[q]];
  };
  read_h(1);
  // the row visited next that starts a group (the last one does): it read a
  // zero state
  int nxt = rev ? min(grp, H) - 1 : (H - 1) / grp * grp;
  auto next_start = [&](int r) { return rev ? min(r + grp, H - 1) : r - grp; };
  for (int b0 = 0; b0 < rows.nb; b0 += UB) {
#pragma unroll
    for (int ub = 0; ub < UB; ++ub) {
#pragma unroll
      for (int kk = 0; kk < kHalo; ++kk) {
        const int s = (b0 + ub) * kHalo + kk, k = (ub * kHalo + kk) % R;
        PK v[5];
#pragma unroll
        for (int m = 0; m < 5; ++m) v[m] = ring[k][m];
        if (NP > 1 && ln.tail) {
#pragma unroll
          for (int m = 0; m < 5; ++m) q_shift<T, NP>(v[m], ln.sh);
        }
        float uv[NP], dyv[NP], w0[NP], w1[NP], w2[NP], hv[NP], gv[NP], dv[3][NP];
        const bool rst = rows.row(s) == nxt;
        if (rst) {
          nxt = next_start(nxt);
#pragma unroll
          for (int q = 0; q < NP; ++q) hn[q] = 0.f;
        }
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          uv[q] = v[0].get(q);
          dyv[q] = v[1].get(q);
          w0[q] = v[2].get(q);
          w1[q] = v[3].get(q);
          w2[q] = v[4].get(q);
          hv[q] = hn[q];
        }
        read_h(s + 2);
        q_adjoint_g<NP>(uv, dyv, ln.valid, a0, a1, a2, gv);
        if (kk == kHalo - 1 && b0 + ub + 1 < rows.nb) exchange((b0 + ub) & 1, gv);
        q_adjoint_w<NP, LG>(w0, w1, w2, hv, gv, ln.pos0, W, renorm, rst, a0, a1, a2, dv);
        load(k, s + R);
        const int line = rows.line(s), so = rows.soff(s);
#pragma unroll
        for (int q = 0; q < NP; ++q) arr[line * P + ln.aoff[q]] = gv[q];
#pragma unroll
        for (int m = 0; m < 3; ++m) qv_store<T, NP>(dv[m], rd[m], ln, so);
      }
    }
  }
}

// Adjoint of a horizontal direction (rev: of the right-to-left scan; columns
// are visited against the scan order).
template <typename T, int NP, int VL, int TV, int R, bool LG, typename FX = QNoExchange>
__device__ __forceinline__ void qh_adjoint(const wide_rsrc_t (&rb)[5], const wide_rsrc_t (&rd)[3], const QH<T, NP>& ln,
                                           const QPlanes& g, float* __restrict__ arr, bool rev, int grp, bool renorm,
                                           FX exchange = FX{}) {
  constexpr int ES = (int)sizeof(T), XV = kHalo / VL;
  typedef QPack<T, VL> PK;
  const int W = g.W, H = g.H;
  const bool desc = !rev;
  float a0[NP], a1[NP], a2[NP], hn[NP];
#pragma unroll
  for (int q = 0; q < NP; ++q) a0[q] = a1[q] = a2[q] = 0.f;
  // past the last column (which starts a group) whatever is there; the padding
  // row holds the zeros the scan left for positions past the line
  auto read_h = [&](int c) __attribute__((always_inline)) {
    const int o = max(c, 0);  // column W is padding
#pragma unroll
    for (int q = 0; q < NP; ++q) hn[q] = arr[ln.aoff[q] + o];
  };
  read_h(desc ? W - 2 : 1);
  int nxt = desc ? (W - 1) / grp * grp : min(grp, W) - 1;
  qh_columns<T, NP, VL, TV, R, 0, 5>(rb, ln, W, desc, [&](int ti, int nt, int lo, int c0, const PK (&v)[5][NP])
                                     __attribute__((always_inline)) {
    const bool cut = c0 != lo;
    const bool xch = (ti + 1) % XV == 0 && ti + 1 < nt;
    float dwb[3][NP][VL];
    auto step = [&](int e) __attribute__((always_inline)) {
      const int col = desc ? c0 + VL - 1 - e : c0 + e;
      if (VL > 1 && col < lo) return;
      const bool rst = col == nxt;
      if (rst) {
        nxt = desc ? nxt - grp : min(nxt + grp, W - 1);
#pragma unroll
        for (int q = 0; q < NP; ++q) hn[q] = 0.f;
      }
      float uv[NP], dyv[NP], w0[NP], w1[NP], w2[NP], hv[NP], gv[NP], dv[3][NP];
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        uv[q] = v[0][q].get(e);
        dyv[q] = v[1][q].get(e);
        w0[q] = v[2][q].get(e);
        w1[q] = v[3][q].get(e);
        w2[q] = v[4][q].get(e);
        hv[q] = hn[q];
      }
      read_h(desc ? col - 2 : min(col + 2, W));
      q_adjoint_g<NP>(uv, dyv, ln.valid, a0, a1, a2, gv);
      // the vector's last column visited
      if (xch && col == (desc ? lo : c0 + VL - 1)) exchange((ti / XV) & 1, gv);
      q_adjoint_w<NP, LG>(w0, w1, w2, hv, gv, ln.pos0, H, renorm, rst, a0, a1, a2, dv);
#pragma unroll
      for (int q = 0; q < NP; ++q) arr[ln.aoff[q] + col] = gv[q];
#pragma unroll
      for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          dwb[m][q][e] = dv[m][q];
          if (cut) q_store_elem<T>(dv[m][q], rd[m], ln.voffs[q], col * ES);
        }
    };
#pragma unroll
    for (int e = 0; e < VL; ++e) step(e);
    if (!cut) {
#pragma unroll
      for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          if (VL > 1 && desc) q_reverse<VL>(dwb[m][q]);
          q_store<T, VL>(dwb[m][q], rd[m], ln.voffs[q], c0 * ES);
        }
    }
  });
}

// Elementwise passes over the workgroup's planes: VE elements a thread and
// turn, in the flat order of the tensors (a plane's last vector ends at its
// end), U turns at a time: first pre(k, element) for each (loads), then
// post(k, element, LDS index of each value within its plane's arrays, plane).
// kc, kr: columns from kc on, rows from kr on lie 2 kHalo further (QHalf).
template <int VE, int U, typename FA, typename FB>
__device__ __forceinline__ void q_flat(const QPlanes& g, int tid, int nthreads, FA&& pre, FB&& post, int kc = 1 << 20,
                                       int kr = 1 << 20) {
  const int HW = g.H * g.W;
  const int nv = (HW + VE - 1) / VE, n = g.np * nv;
  const float inv_nv = 1.f / (float)nv, inv_w = 1.f / (float)g.W;
  for (int i0 = tid; i0 < n; i0 += nthreads * U) {
    int pl[U], e0[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int i = min(i0 + k * nthreads, n - 1);
      pl[k] = (int)(((float)i + 0.5f) * inv_nv);
      e0[k] = min((i - pl[k] * nv) * VE, HW - VE);
      pre(k, pl[k] * HW + e0[k]);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      if (i0 + k * nthreads < n) {
        int r = (int)(((float)e0[k] + 0.5f) * inv_w);
        int c = e0[k] - r * g.W, o = (r + (r >= kr ? 2 * kHalo : 0)) * g.P;
        int li[VE];
#pragma unroll
        for (int q = 0; q < VE; ++q) {
          li[q] = o + c + (c >= kc ? 2 * kHalo : 0);
          if (++c == g.W) {
            c = 0;
            ++r;
            o = (r + (r >= kr ? 2 * kHalo : 0)) * g.P;
          }
        }
        post(k, pl[k] * HW + e0[k], li, pl[k]);
      }
    }
  }
}

// A pair of opposite directions adding into one LDS array, blocks of lines at
// a time (the blocks are the same for both senses): a direction comes first to
// the blocks of its first half; in the middle both pass two barriers, between
// which the forward one does the middle block of an odd count.  So every
// element gets its terms in a fixed order.  The first to come stores (or adds,
// when the array holds a sum already), the other adds, reading one line ahead
// but never across the barriers.
// The barriers are anonymous: every wave of the pair, the idle ones too, has to
// pass them and those of an edge exchange in one sequence, in which a block's
// exchange follows its end().
template <int NP>
struct QMerge {
  float* arr;
  int off[NP];
  bool rev, other, base;  // base: the array holds a sum already
  bool adding;
  float cur[NP];
  __device__ __forceinline__ void fetch(int o) {
#pragma unroll
    for (int q = 0; q < NP; ++q) cur[q] = arr[off[q] + o];
  }
  // before block b of n, whose first line is at o
  __device__ __forceinline__ void begin(int b, int n, int o) {
    const int mid = n >> 1;
    const bool odd = n & 1;
    if (b == 0) adding = base;
    bool first = b == 0;
    if (b == mid) {
      lds_barrier();
      if (rev || !odd) {
        lds_barrier();
        adding = base || other;
      }
      first = true;
    }
    if (b == mid + 1 && !rev && odd) {
      adding = base || other;
      first = true;
    }
    if (first && adding) fetch(o);
  }
  __device__ __forceinline__ void end(int b, int n) const {
    if (b == (n >> 1) && !rev && (n & 1)) lds_barrier();
  }
  __device__ __forceinline__ void put(int o, int onext, const float (&h)[NP]) {
    if (adding) {
#pragma unroll
      for (int q = 0; q < NP; ++q) arr[off[q] + o] = cur[q] + h[q];
      fetch(onext);
    } else {
#pragma unroll
      for (int q = 0; q < NP; ++q) arr[off[q] + o] = h[q];
    }
  }
};

}  // namespace gspn
