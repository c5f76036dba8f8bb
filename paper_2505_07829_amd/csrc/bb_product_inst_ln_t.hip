// product_kernel instantiations: MODE_LN_PRE, weights transposed ([N, K])
#include "bb_product_inst.h"
namespace bb {
template void product_dispatch<MODE_LN_PRE, true>(int, int, int, dim3, hipStream_t, const GemmArgs&);
}
