// Tile kernels of one operand-kind pair and layout for ragged shapes (see EDGE in gemm_tile.h).
#include "gemm_tile.h"

namespace llmq {
template bool launch_edge_tile<0, 0, false, true>(LLMQ_EDGE_LAUNCH_PARAMS);
}
