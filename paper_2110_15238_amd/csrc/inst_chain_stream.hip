// GEMM chains and pairs whose rows stream through independent waves (chain_stream_kernel.hpp).
#include "chain_stream_kernel.hpp"
#include "instances.hpp"
namespace bolt {
// Thin first ops, K0 <= 128; widths that the tiled chains (inst_b2b_chain.hip) and pairs have too, so that what is accepted does
// not depend on K0
#define BOLT_CHAIN_STREAM_WIDTHS(WKN)                                                                   \
  BOLT_CHAIN_STREAM_INSTANCE(4, 128, 32, 128, 32, WKN), BOLT_CHAIN_STREAM_INSTANCE(4, 128, 64, 64, 64, WKN), \
  BOLT_CHAIN_STREAM_INSTANCE(4, 128, 64, 128, 64, WKN), BOLT_CHAIN_STREAM_INSTANCE(4, 128, 64, 64, 128, WKN)
#define BOLT_PAIR_STREAM_WIDTHS(WKN)                                                                 \
  BOLT_PAIR_STREAM_INSTANCE(4, 128, 32, 128, WKN), BOLT_PAIR_STREAM_INSTANCE(4, 128, 64, 32, WKN),     \
  BOLT_PAIR_STREAM_INSTANCE(4, 128, 64, 64, WKN), BOLT_PAIR_STREAM_INSTANCE(4, 128, 64, 128, WKN),     \
  BOLT_PAIR_STREAM_INSTANCE(4, 128, 128, 64, WKN)
void register_b2b_gemm_stream_instances(std::vector<B2bInstance>& v) {
  static const B2bInstance table[] = {BOLT_PAIR_STREAM_WIDTHS(false), BOLT_PAIR_STREAM_WIDTHS(true)};
  for (const auto& t : table) v.push_back(t);
}
void register_gemm_chain_stream_instances(std::vector<ChainInstance>& v) {
  static const ChainInstance table[] = {BOLT_CHAIN_STREAM_WIDTHS(false), BOLT_CHAIN_STREAM_WIDTHS(true)};
  for (const auto& t : table) v.push_back(t);
}
}  // namespace bolt
