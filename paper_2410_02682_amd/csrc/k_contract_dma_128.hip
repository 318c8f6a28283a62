// k_contract_dma with 128 x 128 and 256 x 128 tiles.
#include "k_contract_dma.h"

namespace eg {
namespace dma {

int launch_128(ContractParams &p, int ns, void *stream)
{
    if (p.in_dtype == EG_F32) return launch_layout<128, 128, 128, 2, 2, 4, true>(p, stream);
    if (ns == 4) return launch_layout<128, 128, 128, 4, 2, 8, false>(p, stream);
    return launch_layout<128, 128, 128, 2, 2, 4, false>(p, stream);
}

int launch_256x128(ContractParams &p, void *stream) { return launch_layout<256, 128, 64, 3, 2, 4, false>(p, stream); }

}  // namespace dma
}  // namespace eg
