// The layer kernel's variants: KV in a host pool.
#include "fkv_layer_dev.h"

namespace fkv {

bool launch_layer_host(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st) {
  return dtype == 0 ? launch_layer_variant<0, true, 0>(io, l, G, st) : launch_layer_variant<1, true, 0>(io, l, G, st);
}

}  // namespace fkv
