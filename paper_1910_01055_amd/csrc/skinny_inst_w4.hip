#include "skinny_layer.hpp"

namespace aq {
void skinny_go_w4(const SkinnyCall& c) {
    if (c.taps) skinny_tile<false, true, true>(c);
    else skinny_tile<false, false, true>(c);
}
}  // namespace aq
