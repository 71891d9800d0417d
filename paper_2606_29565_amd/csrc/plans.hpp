// The launch plans of one pass's projections, and the size of the work buffer that their
// split-K partials share.  Host only.
#pragma once

#include <algorithm>

#include "kernels.hpp"

namespace spp {

struct StepPlans {
  k::GemmPlan qkv, o, dn;
  k::GemmPlan sw;  // gate/up with the SwiGLU fused (no K-splits); splits = 0 where it does not apply
  k::GemmPlan gu;  // the gate/up projection there
};

inline StepPlans step_plans(const Shape& s, bool fp4, int M) {
  const auto plan = fp4 ? k::gemm_plan_fp4 : k::gemm_plan;
  const int nq = s.n_q * s.dh, nkv = s.n_kv * s.dh;
  StepPlans p{};
  p.qkv = plan(s, M, nq + 2 * nkv, s.d);
  p.o = plan(s, M, s.d, nq);
  p.dn = plan(s, M, s.d, s.ffn);
  p.sw = fp4 ? k::gemm_plan_swiglu_fp4(s, M, s.ffn, s.d) : k::gemm_plan_swiglu(s, M, s.ffn, s.d);
  if (p.sw.splits != 1) p.gu = plan(s, M, 2 * s.ffn, s.d);
  return p;
}

// Floats of the largest partials among a pass's projections with these plans, at M rows.
inline size_t partial_elems(const Shape& s, const StepPlans& p, int M) {
  const size_t nqkv = (size_t)(s.n_q + 2 * s.n_kv) * s.dh;
  return M * std::max({p.qkv.splits * nqkv, p.o.splits * (size_t)s.d, p.dn.splits * (size_t)s.d,
                       p.gu.splits * (size_t)s.ffn * 2});
}

// Floats that hold the partials of every pass of up to max_rows rows.  The split counts do not
// grow with the row count inside a bucket of the planners' row tiles (16, 32, then whole 64s):
// the plans of a bucket's first row count, at its last one, bound the bucket (the planners charge
// partials by the row, so a larger count turns only to fewer splits).  Asking every count up to 8192
// took 2 ms of a model's creation.
inline size_t partial_elems_upto(const Shape& s, bool fp4, int max_rows) {
  size_t most = 0;
  for (int lo = 1; lo <= max_rows;) {
    const int hi = lo == 1 ? 16 : lo == 17 ? 32 : (lo + 63) / 64 * 64;
    most = std::max(most, partial_elems(s, step_plans(s, fp4, lo), std::min(hi, max_rows)));
    lo = hi + 1;
  }
  return most;
}

}  // namespace spp
