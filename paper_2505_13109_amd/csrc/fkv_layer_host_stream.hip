// The layer kernel's variants: KV in a host pool, summaries read past the caches.
#include "fkv_layer_dev.h"

namespace fkv {

bool launch_layer_host_stream(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st) {
  return launch_layer_variant<true, STREAM_SUMMARIES>(io, l, dtype, G, st);
}

}  // namespace fkv
