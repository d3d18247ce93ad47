// Launches of k_pipe (laud_pipe.h): modes CONV2, SD2, G2.
#include "laud_pipe.h"

namespace laud {

int launch_pipe_b(int mode, int dtype, const GemmArgs& a, long long cap_rows, int nsamples, hipStream_t st) {
  switch (mode) {
    case M_CONV2: return launch_pipe_mode<M_CONV2>(dtype, a, cap_rows, nsamples, st);
    case M_SD2: return launch_pipe_mode<M_SD2>(dtype, a, cap_rows, nsamples, st);
    case M_G2: return launch_pipe_mode<M_G2>(dtype, a, cap_rows, nsamples, st);
    default: return LAUD_ERR_UNSUPPORTED;
  }
}

}  // namespace laud
