// Window kernels (k_window): sequences of Crank-Nicolson steps on independent windows.
#include "kern_table.hpp"
#include "nshaped_windows.hpp"

namespace nsk {
namespace {
template <int I, int LV>
void reg_lv(Tables& t) {
  constexpr int M = kWinCfgs[0][I].M, W = kWinCfgs[0][I].W;
  t.win[0][I][LV - kWinLevelMin][0] = (const void*)&nsd::k_window<M, W, LV, 1, false>;
  t.win[0][I][LV - kWinLevelMin][1] = (const void*)&nsd::k_window<M, W, LV, 1, true>;
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

void reg_windows(Tables& t) { reg_range(t, std::make_integer_sequence<int, kNumWinCfg>{}); }

}  // namespace nsk
