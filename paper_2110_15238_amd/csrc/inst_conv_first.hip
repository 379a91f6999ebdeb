// First-layer convolutions of 3 or 4 channels in strips (k-steps of 32 = 8 taps x 4 channels each, stride along W).
#include "instances.hpp"
namespace bolt {
void register_conv_first_instances(std::vector<FpropInstance>& v) {
  static const FpropInstance table[] = {BOLT_CONV_FIRST_INSTANCE(2, 2), BOLT_CONV_FIRST_INSTANCE(4, 2), BOLT_CONV_FIRST_INSTANCE(7, 2),
                                        BOLT_CONV_FIRST_INSTANCE(2, 1), BOLT_CONV_FIRST_INSTANCE(4, 1), BOLT_CONV_FIRST_INSTANCE(7, 1)};
  for (const auto& t : table) v.push_back(t);
}
}  // namespace bolt
