// Matrix-core pass kernels for BLS12-377 Fr.
#include "ntt_mfma_impl.hpp"

namespace zk {
hipError_t launch_mfma_b377(int log_r, const PassLaunch& a, hipStream_t s) { return mfma::dispatch<Bls12_377Fr>(log_r, a, s); }
}  // namespace zk
