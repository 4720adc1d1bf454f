// The layer kernel's variants: KV in HBM, summaries read past the caches.
#include "fkv_layer_dev.h"

namespace fkv {

bool launch_layer_hbm_stream(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st) {
  return launch_layer_variant<false, STREAM_SUMMARIES>(io, l, dtype, G, st);
}

}  // namespace fkv
