// product_kernel instantiations: MODE_PLAIN, weights transposed ([N, K])
#include "bb_product_inst.h"
namespace bb {
template void product_dispatch<MODE_PLAIN, true>(int, int, int, dim3, hipStream_t, const GemmArgs&);
}
