// attention kernel instantiations: head dimensions d = 64, dv = 64
#include "bb_attn_inst.h"
namespace bb {
template void attn_tiled_launch<64, 64>(int, int, int, bool, dim3, dim3, hipStream_t, const AttnArgs&);
template void attn_decode_launch<64, 64>(dim3, hipStream_t, const AttnArgs&);
template void attn_group_launch<64, 64>(int, dim3, hipStream_t, const AttnArgs&);
}
