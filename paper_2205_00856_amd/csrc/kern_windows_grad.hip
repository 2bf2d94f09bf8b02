// Window kernels (k_window): backward sequences (state and gradient).
#include "kern_table.hpp"
#include "nshaped_windows.hpp"

namespace nsk {
namespace {
template <int I, int LV>
void reg_lv(Tables& t) {
  constexpr int M = kWinCfgs[1][I].M, W = kWinCfgs[1][I].W;
  t.win[1][I][LV - kWinLevelMin][0] = (const void*)&nsd::k_window<M, W, LV, 2, false>;
  t.win[1][I][LV - kWinLevelMin][1] = (const void*)&nsd::k_window<M, W, LV, 2, true>;
}
template <int I, int... LV>
void reg_one(Tables& t, std::integer_sequence<int, LV...>) {
  (reg_lv<I, LV + kWinLevelMin>(t), ...);
}
template <int... I>
void reg_range(Tables& t, std::integer_sequence<int, I...>) {
  (reg_one<I>(t, std::make_integer_sequence<int, kNumWinLevel>{}), ...);
}
}  // namespace

void reg_windows_grad(Tables& t) { reg_range(t, std::make_integer_sequence<int, kNumWinCfg>{}); }

}  // namespace nsk
