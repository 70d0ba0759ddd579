// Whole transforms in the register kernels over BLS12-377 Fr.
#include "ntt_pass_impl.hpp"

namespace zk {
hipError_t launch_pass_b377(int log_r, const PassLaunch& a, hipStream_t s) {
  return detail::dispatch_registers<Bls12_377Fr>(log_r, a, s);
}
}  // namespace zk
