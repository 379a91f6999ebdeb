// Thin convolutions, alone and fused with the 1x1 behind them: weights in registers, pixels streamed.
#include "conv_patch_kernel.hpp"
#include "instances.hpp"
namespace bolt {
void register_b2b_conv_patch_instances(std::vector<B2bInstance>& v) {
// P(channels, first op's output channels, filter extent, stride)
#define P(CP, N0T, RS, ST) BOLT_CONV_PATCH_PAIR_INSTANCE(CP, N0T, RS, ST)
  static const B2bInstance table[] = {
      P(64, 64, 3, 1), P(48, 64, 3, 1), P(32, 64, 3, 1), P(64, 32, 3, 1), P(32, 32, 3, 1),
      P(64, 64, 3, 2), P(32, 64, 3, 2), P(64, 64, 1, 1), P(128, 64, 1, 1), P(64, 32, 1, 1), P(128, 32, 1, 1),
  };
  for (const auto& t : table) v.push_back(t);
}
void register_conv_patch_instances(std::vector<FpropInstance>& v) {
#define S(CP, RS, ST) BOLT_CONV_PATCH_INSTANCE(CP, RS, ST)
  static const FpropInstance table[] = {S(64, 3, 1), S(32, 3, 1)};
  for (const auto& t : table) v.push_back(t);
}
}  // namespace bolt
