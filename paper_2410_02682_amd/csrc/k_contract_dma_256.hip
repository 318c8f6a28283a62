// k_contract_dma with 256 x 256 tiles.
#include "k_contract_dma.h"

namespace eg {
namespace dma {

int launch_256(ContractParams &p, int nw, void *stream)
{
    if (p.in_dtype == EG_F32) return launch_layout<256, 256, 128, 2, 2, 8, true>(p, stream);
    if (nw == 4) return launch_layout<256, 256, 128, 2, 2, 4, false>(p, stream);
    return launch_layout<256, 256, 128, 2, 2, 8, false>(p, stream);
}

}  // namespace dma
}  // namespace eg
