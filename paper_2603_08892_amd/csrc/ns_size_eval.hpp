// ns_size_eval.hpp -- the passes of one size of ns_size_plans.hpp, with the stage
// operation as an argument; instantiated by size_passes.hip for one size and type.
#pragma once

#include "ns_fast_eval.hpp"
#include "ns_size_plans.hpp"

namespace nsh {

template <typename R, int N>
struct SizeEval {
  using P = ns::SizePlan<R, N>;
  using C = ns::FastCfg<typename P::X, typename P::Y, typename P::Z, P::PZ, typename P::X, typename P::ZA, P::PZA>;

  static ns_status eval(ns_ctx* c, int op, const Cx<R>* in, ns::Lay lin, const ns::Shift& sh, EpiArgs<R> a,
                        Chain* ch) {
    const bool front = !(ch && ch->front_done);
    const int feed = (ch && !a.full && c->lay.ntiles_active > 0) ? ch->feed : 0;
    a.op = op;
    a.feed = feed;
    if (ch) ch->fused = feed != 0;
    if (feed != 0)
      return eval_fast<C, ns::OP_ANY, ns::FEED_ANY>(c, in, lin, sh, a, front, make_shift(ch->next_s));
    return eval_fast<C, ns::OP_ANY, 0>(c, in, lin, sh, a, front, sh);
  }

  static ns_status adj(ns_ctx* c, int aop, const Cx<R>* st, ns::Lay lst, const ns::Shift& sh, const LamArgs<R>& la,
                       AdjArgs<R> aa) {
    aa.op = aop;
    return adj_eval_fast<C, ns::AOP_ANY>(c, st, lst, sh, la, aa);
  }
};

template <typename R, int N>
const SizePasses<R>* size_passes() {
  static const SizePasses<R> passes = {&SizeEval<R, N>::eval, &SizeEval<R, N>::adj};
  return &passes;
}

}  // namespace nsh
