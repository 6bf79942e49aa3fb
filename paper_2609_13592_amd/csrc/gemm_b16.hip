// The matrix-core GEMM of 1 batch tile (one translation unit per count, so
// that they build in parallel).
#include "gemm.h"

template int bst::gv::launch_gemm<1>(GemvParams&, const Route&, int, bool, const boost_ctx*,
                                      hipStream_t);
