// The split-product fused kernel (wino_split.h) of one tile size per object file: the
// build compiles this file once for every m of WINO_SPLIT_M, with WS_M defined.
#include "wino_split.h"

#if !defined(WS_M)
#error "compile with -DWS_M=<m>"
#endif

namespace wino {

template hipError_t launch_split_t<WS_M>(const Geometry &, const float *, const float *, float *, int, bool,
                                         const SplitBuffers &, hipStream_t);

}  // namespace wino
