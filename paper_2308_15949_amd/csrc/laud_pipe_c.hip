// Launches of k_pipe (laud_pipe.h): modes CONV3, SD3, CS1, CS2, CS3, U1, U2, U3.
#include "laud_pipe.h"

namespace laud {

int launch_pipe_c(int mode, int dtype, const GemmArgs& a, long long cap_rows, int nsamples, hipStream_t st) {
  switch (mode) {
    case M_CONV3: return launch_pipe_mode<M_CONV3>(dtype, a, cap_rows, nsamples, st);
    case M_SD3: return launch_pipe_mode<M_SD3>(dtype, a, cap_rows, nsamples, st);
    case M_CS1: return launch_pipe_mode<M_CS1>(dtype, a, cap_rows, nsamples, st);
    case M_CS2: return launch_pipe_mode<M_CS2>(dtype, a, cap_rows, nsamples, st);
    case M_CS3: return launch_pipe_mode<M_CS3>(dtype, a, cap_rows, nsamples, st);
    case M_U1: return launch_pipe_mode<M_U1>(dtype, a, cap_rows, nsamples, st);
    case M_U2: return launch_pipe_mode<M_U2>(dtype, a, cap_rows, nsamples, st);
    case M_U3: return launch_pipe_mode<M_U3>(dtype, a, cap_rows, nsamples, st);
    default: return LAUD_ERR_UNSUPPORTED;
  }
}

}  // namespace laud
