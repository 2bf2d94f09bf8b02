// One-pass steps of contiguous systems (k_rowstep, k_rowstep_fix) and of the partial waves' field
// part (k_lstep).
#include "kern_table.hpp"
#include "nshaped_lstep.hpp"
#include "nshaped_rowstep.hpp"

namespace nsk {
namespace {
template <int I>
void reg_one(Tables& t) {
  constexpr int M = kRowStepCfgs[I].M, W = kRowStepCfgs[I].W;
  t.rowstep[I][0][0] = (const void*)&nsd::k_rowstep<M, W, false>;
  t.rowstep[I][1][0] = (const void*)&nsd::k_rowstep<M, W, true>;
  t.rowstep[I][0][1] = (const void*)&nsd::k_rowstep_fix<M, W, false>;
  t.rowstep[I][1][1] = (const void*)&nsd::k_rowstep_fix<M, W, true>;
}
template <int... I>
void reg_range(Tables& t, std::integer_sequence<int, I...>) {
  (reg_one<I>(t), ...);
}
}  // namespace

void reg_rowstep(Tables& t) {
  reg_range(t, std::make_integer_sequence<int, kNumRowStepCfg>{});
  t.aux[AUX_LSTEP] = (const void*)&nsd::k_lstep<nsd::kLRows>;
}

}  // namespace nsk
