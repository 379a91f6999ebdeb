// Convolutions with an even channel count that is no multiple of 8, padded on the way to LDS.
#include "instances.hpp"
namespace bolt {
// E(waves, pixel fragments, channel fragments): what is left of {4, 8} x {2, 3, 4, 5, 6, 8} x {1, 2, 3, 4} after keeping
// what came first or within 3 % of the first on 31 problems (the ranges of Table 3, 8 to 288 images, 10 to 174 channels).
#define E(NW, FM, FN) BOLT_CONV_EVEN_INSTANCE(NW, FM, FN)
void register_conv_even_instances(std::vector<FpropInstance>& v) {
  static const FpropInstance table[] = {
      E(4, 4, 1), E(4, 5, 1), E(4, 6, 1), E(4, 5, 2), E(4, 6, 2), E(4, 8, 2), E(4, 4, 3),
      E(8, 2, 1), E(8, 4, 1), E(8, 5, 1), E(8, 6, 1), E(8, 5, 2), E(8, 6, 2), E(8, 8, 2), E(8, 8, 3), E(8, 5, 4),
  };
  for (const auto& t : table) v.push_back(t);
}
}  // namespace bolt
