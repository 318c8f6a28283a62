// k_contract_dma with the totals of the blocks along aggregated labels.
#include "k_contract_dma.h"

namespace eg {
namespace dma {

int launch_totals(ContractParams &p, int ns, void *stream)
{
    if (p.in_dtype == EG_F32) return launch_layout<128, 128, 128, 2, 2, 4, true, 1>(p, stream);
    if (ns == 4) return launch_layout<128, 128, 128, 4, 2, 8, false, 1>(p, stream);
    return launch_layout<128, 128, 128, 2, 2, 4, false, 1>(p, stream);
}

}  // namespace dma
}  // namespace eg
