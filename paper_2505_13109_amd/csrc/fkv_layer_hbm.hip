// The layer kernel's variants: KV in HBM.
#include "fkv_layer_dev.h"

namespace fkv {

bool launch_layer_hbm(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st) {
  return launch_layer_variant<false, 0>(io, l, dtype, G, st);
}

}  // namespace fkv
