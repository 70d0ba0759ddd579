// Whole transforms in the register kernels over BLS12-381 Fr.
#include "ntt_pass_impl.hpp"

namespace zk {
hipError_t launch_pass_bls(int log_r, const PassLaunch& a, hipStream_t s) {
  return detail::dispatch_registers<Bls12_381Fr>(log_r, a, s);
}
}  // namespace zk
