// Explicit instantiation of general whole-network kernel variants, with and without intermediate taps.
#include "fused_mlp.hpp"

namespace aq {
AQ_FUSED_INST(1, 2, true, false, true);
AQ_FUSED_INST(1, 2, true, true, true);
AQ_FUSED_INST(1, 2, true, false, false);
AQ_FUSED_INST(1, 2, true, true, false);
}  // namespace aq
