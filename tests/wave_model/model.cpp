// The generic resident kernels on the host (see hip/hip_runtime.h), behind C
// functions: MODEL_T (0: fp32, 1: bf16) and MODEL_LG (Eq. 6 logits) choose the
// instantiation.
#include "gspn_quadbwd_impl.hpp"

namespace gspn {
alignas(16) float lds[(sim::kLdsBytes + sim::kGuard) / 4];
}
using namespace gspn;

namespace {
typedef std::conditional_t<MODEL_T == 0, float, bf16> T;

void setup(const int* order) {
  sim::order.assign(order, order + 4);
  sim::allowed.clear();
  sim::grids.clear();
  sim::dry = false;
}
}  // namespace

extern "C" {

int model_fwd(const void* x, const void* w, const void* lam, const void* u, void* y, int64_t planes, int H, int W,
              unsigned mask, int group_h, int group_w, int lam_pd, int y_pd, const int* order) {
  setup(order);
  ResidentFwdArgs a{};
  a.x = x; a.w = w; a.lam = lam; a.u = u; a.y = y;
  a.planes = planes; a.H = H; a.W = W; a.mask = mask; a.group_h = group_h; a.group_w = group_w;
  a.lam_pd = lam_pd; a.y_pd = y_pd;
  const size_t b = (size_t)planes * H * W * sizeof(T), n = __builtin_popcount(mask);
  sim::allow(x, b);
  sim::allow(w, b * 3 * n);
  sim::allow(lam, lam_pd ? b * n : b);
  sim::allow(u, b);
  sim::allow(y, y_pd ? b * n : b);
  const QFwdParams p = quad_fwd_params(a);
  return y_pd ? launch_quad_fwd_pd<T, MODEL_LG>(p, nullptr) : launch_quad_fwd<T, MODEL_LG>(p, nullptr);
}

// pair: one axis a launch, with the sums of h and g (planes * H * W floats each)
int model_bwd(const void* dy, const void* x, const void* w, const void* lam, const void* u, void* dx, void* dw,
              void* dlam, void* du, float* hsum, float* gsum, int64_t planes, int H, int W, unsigned mask,
              int group_h, int group_w, int pair, const int* order) {
  setup(order);
  ResidentBwdArgs a{};
  a.dy = dy; a.x = x; a.w = w; a.lam = lam; a.u = u; a.dx = dx; a.dw = dw; a.dlam = dlam; a.du = du;
  a.planes = planes; a.H = H; a.W = W; a.mask = mask; a.group_h = group_h; a.group_w = group_w;
  const size_t e = (size_t)planes * H * W, b = e * sizeof(T), n = __builtin_popcount(mask);
  for (const void* q : {dy, x, lam, u, (const void*)dx, (const void*)dlam, (const void*)du}) sim::allow(q, b);
  sim::allow(w, b * 3 * n);
  sim::allow(dw, b * 3 * n);
  sim::allow(hsum, e * 4);
  sim::allow(gsum, e * 4);
  QBwdParams p = quad_bwd_params(a);
  if (!pair) return launch_quad_bwd<T, MODEL_LG>(p, nullptr);
  p.hsum = hsum;
  p.gsum = gsum;
  return launch_pair_bwd<T, MODEL_LG>(p, nullptr);
}

// The launches of a forward (which 0) or backward (1) over so many planes,
// recorded and not run: their number, -1 where one is too large; groups:
// their workgroups in all.
int model_launches(int which, int64_t planes, int H, int W, int64_t* groups) {
  const int order[4] = {0, 1, 2, 3};
  setup(order);
  sim::dry = true;
  ResidentFwdArgs f{};
  ResidentBwdArgs b{};
  f.planes = b.planes = planes;
  f.H = b.H = H;
  f.W = b.W = W;
  f.mask = b.mask = 15;
  const hipError_t e = which ? launch_quad_bwd<T, MODEL_LG>(quad_bwd_params(b), nullptr)
                             : launch_quad_fwd<T, MODEL_LG>(quad_fwd_params(f), nullptr);
  *groups = 0;
  for (uint64_t g : sim::grids) *groups += (int64_t)(g / 256);
  return e == hipSuccess ? (int)sim::grids.size() : -1;
}

}  // extern "C"
