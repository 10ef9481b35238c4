// gemm_slim.hpp for f16.
#include "gemm_slim.hpp"

namespace ci {

int launch_gemm_slim_f16(int tm, int tn, int epi, const GemmArgs& g, hipStream_t s) {
  return launch_tm<F16>(tm, tn, epi, g, s);
}

}  // namespace ci
