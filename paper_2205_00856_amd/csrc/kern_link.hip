// One-pass kernels of multi-tile systems (k_tile<PH_LINK>, k_tile_fix): the tiles that the
// automatic plans of large batches use.
#include "kern_table.hpp"
#include "nshaped_kernels.hpp"

namespace nsk {
namespace {
template <int M, int W, int S>
void reg_one(Tables& t) {
  constexpr int I = cfg_index<M, W>();
  static_assert(I >= 0, "a configuration of the row-tile table");
  t.link[I][S][0] = (const void*)&nsd::k_tile<M, W, S, nsd::PH_LINK>;
  t.link[I][S][1] = (const void*)&nsd::k_tile_fix<M, W, S>;
  t.link[I][S][3] = (const void*)&nsd::k_tile<M, W, S, nsd::PH_SUBST_LK>;
  if constexpr (nsd::cn_src(S)) t.link[I][S][2] = (const void*)&nsd::k_tile<M, W, S, nsd::PH_HAND>;
}
}  // namespace

void reg_link(Tables& t) {
  reg_one<4, 2, nsd::SRC_EXPL>(t);
  reg_one<4, 4, nsd::SRC_EXPL>(t);
  reg_one<4, 2, nsd::SRC_EXPL_CT>(t);
  reg_one<4, 4, nsd::SRC_EXPL_CT>(t);
  reg_one<8, 4, nsd::SRC_CN>(t);
  reg_one<8, 4, nsd::SRC_CNW>(t);
}

}  // namespace nsk
