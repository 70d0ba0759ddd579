// Matrix-core pass kernels for BN254 Fr.
#include "ntt_mfma_impl.hpp"

namespace zk {
hipError_t launch_mfma_bn(int log_r, const PassLaunch& a, hipStream_t s) { return mfma::dispatch<Bn254Fr>(log_r, a, s); }
}  // namespace zk
