// Whole transforms in the register kernels over BN254 Fr.
#include "ntt_pass_impl.hpp"

namespace zk {
hipError_t launch_pass_bn(int log_r, const PassLaunch& a, hipStream_t s) {
  return detail::dispatch_registers<Bn254Fr>(log_r, a, s);
}
}  // namespace zk
