// One (element type, pass length) instantiation of the kernels: the build
// compiles this file once per pair with -DTFFT_INST_R=<float|double> and
// -DTFFT_INST_M=<length>.
#include "tfft_cols.h"

namespace tfft {
TFFT_INSTANTIATE_M(TFFT_INST_R, TFFT_INST_M)
// (the column kernels: complex64 alone, cfg_cols)
#define TFFT_COLS_OF_float(M) TFFT_INSTANTIATE_COLS(float, M)
#define TFFT_COLS_OF_double(M)
#define TFFT_COLS_OF_(R, M) TFFT_COLS_OF_##R(M)
#define TFFT_COLS_OF(R, M) TFFT_COLS_OF_(R, M)
#if TFFT_INST_M >= 64 && TFFT_INST_M <= 512
TFFT_COLS_OF(TFFT_INST_R, TFFT_INST_M)
#endif
}  // namespace tfft
