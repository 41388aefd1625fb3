// Explicit instantiation of general whole-network kernel variants, with and without intermediate taps.
#include "fused_mlp.hpp"

namespace aq {
AQ_FUSED_INST(4, 1, false, false, false);
AQ_FUSED_INST(4, 1, false, true, false);
}  // namespace aq
