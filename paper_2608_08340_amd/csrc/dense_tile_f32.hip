// The tiled scoring and rescoring kernels for fp32 storage.
#include "dense_tile.h"

namespace oprag {
template hipError_t tile_launch<kDtypeF32>(int, int, long long, DenseArgs&, hipStream_t, hipEvent_t, hipEvent_t);
template hipError_t rescore_launch<kDtypeF32>(const RescoreArgs&, int, hipStream_t);
}  // namespace oprag
