// Explicit instantiation of general whole-network kernel variants, with and without intermediate taps.
#include "fused_mlp.hpp"

namespace aq {
AQ_FUSED_INST(1, 1, false, false, true);
AQ_FUSED_INST(1, 1, false, true, true);
AQ_FUSED_INST(1, 1, false, false, false);
AQ_FUSED_INST(1, 1, false, true, false);
}  // namespace aq
