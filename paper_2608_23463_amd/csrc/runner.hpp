// Launch context: either enqueues kernels on a stream, or (dry run) only
// records how much split-K workspace the same sequence of GEMMs needs, so the
// size queries and the real calls can never disagree.
#pragma once

#include "gemm.hpp"
#include "trace.hpp"

namespace pf {

struct Runner {
  bool dry;
  hipStream_t stream;
  float* gemm_ws;      // split-K partials (may be NULL in a dry run)
  size_t gemm_need;    // dry run: max bytes any GEMM asked for
  hipError_t err;

  explicit Runner(bool dry_run, hipStream_t s = nullptr, float* ws = nullptr)
      : dry(dry_run), stream(s), gemm_ws(ws), gemm_need(0), err(hipSuccess) {}

  bool ok() const { return err == hipSuccess; }

  // C = A B^T through `epi`, with a deterministic split-K through gemm_ws when
  // the plan asks for it. `label` names the launch for tracing.
  template <typename T, int LA, int LB, class Epi>
  void gemm(const char* label, const GemmProblem& pr, const Epi& epi) {
    gemm_group<T, LA, LB>(label, &pr, &epi, 1);
  }

  // Up to kGemmGroup independent products in one launch (and one reduction
  // when K is split): small products leave most of the chip idle on their own
  // and pay a launch and a pipeline fill each. `plan`: made by the caller.
  template <typename T, int LA, int LB, class Epi>
  void gemm_group(const char* label, const GemmProblem* prs, const Epi* epis, int count,
                  const GemmPlan* plan = nullptr) {
    if (!ok() || count <= 0) return;
    for (int i = 0; i < count; ++i)
      if (prs[i].M <= 0 || prs[i].N <= 0) return;
    GemmPlan pl = plan ? *plan : plan_gemm<T>(prs, count, kPlanCUsGemm);
    if (dry) {
      if (pl.splits > 1) {
        size_t need = 0;
        for (int i = 0; i < count; ++i) need += plan_partials(prs[i], pl) * sizeof(float);
        if (need > gemm_need) gemm_need = need;
      }
      return;
    }
    if (pl.splits <= 1 || gemm_ws == nullptr) {
      pl.splits = 1;
      timed(label, [&] { return launch_gemm_plan<T, LA, LB>(prs, count, pl, epis, stream); });
      return;
    }
    EpiPartial part[kGemmGroup];
    GemmProblem sl[kGemmGroup];
    float* parts[kGemmGroup];
    float* at = gemm_ws;
    for (int i = 0; i < count; ++i) {
      sl[i] = prs[i];
      if (sl[i].colsum) sl[i].colsum = prs[i].cs_part;  // per-slice sums, joined by the reduction
      parts[i] = at;
      part[i] = EpiPartial{at, prs[i].N, (int64_t)prs[i].M * prs[i].N, 0};
      at += plan_partials(prs[i], pl);
    }
    timed(label, [&] { return launch_gemm_plan<T, LA, LB>(sl, count, pl, part, stream); });
    if (!ok()) return;
    timed("splitk_reduce", [&] { return launch_splitk_reduce(prs, count, pl, parts, epis, stream); });
  }

  template <class F>
  void launch(const char* label, F&& f) {
    if (!ok() || dry) return;
    timed(label, f);
  }

  template <class F>
  void timed(const char* label, F&& f) {
    const bool tr = trace_on();
    if (tr) trace_begin(label, stream);
    err = f();
    if (tr) trace_end(stream);
  }

  static constexpr int kPlanCUsGemm = 256;
};

}  // namespace pf
