// The layer kernel's variants: KV in a host pool, the poolings beside the method's.
#include "fkv_layer_dev.h"

namespace fkv {

bool launch_layer_host_pool(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st) {
  return launch_layer_variant<true, OTHER_POOLING>(io, l, dtype, G, st);
}

}  // namespace fkv
