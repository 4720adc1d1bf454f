// The layer kernel's variants: KV in HBM.
#include "fkv_layer_dev.h"

namespace fkv {

bool launch_layer_hbm(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st) {
  return dtype == 0 ? launch_layer_variant<0, false, 0>(io, l, G, st) : launch_layer_variant<1, false, 0>(io, l, G, st);
}

}  // namespace fkv
