// product_kernel instantiations: MODE_GATEUP_PRE, weights row-major ([K, N])
#include "bb_product_inst.h"
namespace bb {
template void product_dispatch<MODE_GATEUP_PRE, false>(int, int, int, dim3, hipStream_t, const GemmArgs&);
}
