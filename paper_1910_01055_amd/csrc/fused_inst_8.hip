// Explicit instantiation of general whole-network kernel variants, with and without intermediate taps.
#include "fused_mlp.hpp"

namespace aq {
AQ_FUSED_INST(2, 2, true, false, false);
AQ_FUSED_INST(2, 2, true, true, false);
}  // namespace aq
