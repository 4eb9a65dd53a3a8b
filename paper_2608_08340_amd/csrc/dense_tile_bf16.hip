// The tiled scoring and rescoring kernels for bf16 storage.
#include "dense_tile.h"

namespace oprag {
template hipError_t tile_launch<kDtypeBF16>(int, int, long long, DenseArgs&, hipStream_t, hipEvent_t, hipEvent_t);
template hipError_t rescore_launch<kDtypeBF16>(const RescoreArgs&, int, hipStream_t);
}  // namespace oprag
