// Launches of k_pipe (laud_pipe.h): modes CONV1, DENSE1, SD1.
#include "laud_pipe.h"

namespace laud {

int launch_pipe_a(int mode, int dtype, const GemmArgs& a, long long cap_rows, int nsamples, hipStream_t st) {
  switch (mode) {
    case M_CONV1: return launch_pipe_mode<M_CONV1>(dtype, a, cap_rows, nsamples, st);
    case M_DENSE1: return launch_pipe_mode<M_DENSE1>(dtype, a, cap_rows, nsamples, st);
    case M_SD1: return launch_pipe_mode<M_SD1>(dtype, a, cap_rows, nsamples, st);
    default: return LAUD_ERR_UNSUPPORTED;
  }
}

}  // namespace laud
