// Small problems: the reduction split over the waves of a workgroup.
#include "instances.hpp"
namespace bolt {
// W(waves, row fragments, column fragments): what came first or within 5 % of the first on 76 problems with up to 512 tiles;
// 64-row and 64-column tiles and 16 waves on a 32 x 32 tile never did.
#define BOLT_WS_LIST(W) \
  W(4, 1, 1), W(8, 1, 1), W(16, 1, 1), W(4, 1, 2), W(8, 1, 2), W(16, 1, 2), W(4, 2, 2), W(8, 2, 2)
#define KN(NW, FM, FN) BOLT_FPROP_WS_INSTANCE(NW, FM, FN, 0, true)
#define NK(NW, FM, FN) BOLT_FPROP_WS_INSTANCE(NW, FM, FN, 0, false)
#define CV(NW, FM, FN) BOLT_FPROP_WS_INSTANCE(NW, FM, FN, 1, false)
void register_gemm_ws_instances(std::vector<FpropInstance>& v) {
  static const FpropInstance table[] = {BOLT_WS_LIST(KN), BOLT_WS_LIST(NK)};
  for (const auto& t : table) v.push_back(t);
}
void register_conv_ws_instances(std::vector<FpropInstance>& v) {
  static const FpropInstance table[] = {BOLT_WS_LIST(CV), BOLT_WS_LIST(NK)};
  for (const auto& t : table) v.push_back(t);
}
}  // namespace bolt
