#include "skinny_layer.hpp"

namespace aq {
void skinny_go_asym(const SkinnyCall& c) {
    if (c.taps) skinny_tile<true, true, false>(c);
    else skinny_tile<true, false, false>(c);
}
}  // namespace aq
