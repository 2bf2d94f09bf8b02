// One-pass steps of interleaved batches (k_colstep, k_colstep_fix).
#include "kern_table.hpp"
#include "nshaped_colstep.hpp"

namespace nsk {
namespace {
template <int I>
void reg_one(Tables& t) {
  constexpr int M = kColStepCfgs[I].M, W = kColStepCfgs[I].W;
  t.colstep[I][0][0] = (const void*)&nsd::k_colstep<M, W, false>;
  t.colstep[I][1][0] = (const void*)&nsd::k_colstep<M, W, true>;
  t.colstep[I][0][1] = (const void*)&nsd::k_colstep_fix<M, W, false>;
  t.colstep[I][1][1] = (const void*)&nsd::k_colstep_fix<M, W, true>;
}
template <int... I>
void reg_range(Tables& t, std::integer_sequence<int, I...>) {
  (reg_one<I>(t), ...);
}
}  // namespace

void reg_colstep(Tables& t) { reg_range(t, std::make_integer_sequence<int, kNumColStepCfg>{}); }

}  // namespace nsk
