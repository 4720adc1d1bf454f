// The layer kernel's variants: KV in a host pool.
#include "fkv_layer_dev.h"

namespace fkv {

bool launch_layer_host(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st) {
  return launch_layer_variant<true, 0>(io, l, dtype, G, st);
}

}  // namespace fkv
