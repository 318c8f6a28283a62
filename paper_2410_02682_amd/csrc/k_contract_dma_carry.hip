// k_contract_dma with 256 x 256 tiles and two blocks along the aggregated labels: the first one's sums wait in memory for the second.
#include "k_contract_dma.h"

namespace eg {
namespace dma {

int launch_carry(ContractParams &p, void *stream) { return launch_layout<256, 256, 128, 2, 2, 8, false, 2>(p, stream); }

}  // namespace dma
}  // namespace eg
