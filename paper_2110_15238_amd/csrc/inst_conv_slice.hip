// 3x3 convolutions split over independent waves by input channels.
#include "instances.hpp"
namespace bolt {
void register_conv_slice_instances(std::vector<FpropInstance>& v) {
  static const FpropInstance table[] = {
      BOLT_CONV_SLICE_INSTANCE(128, 64, 1), BOLT_CONV_SLICE_INSTANCE(128, 64, 2), BOLT_CONV_SLICE_INSTANCE(64, 64, 1),
      BOLT_CONV_SLICE_INSTANCE(64, 64, 2),  BOLT_CONV_SLICE_INSTANCE(64, 64, 4),  BOLT_CONV_SLICE_INSTANCE(128, 128, 1),
  };
  for (const auto& t : table) v.push_back(t);
}
}  // namespace bolt
