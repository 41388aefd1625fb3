#include "skinny_layer.hpp"

namespace aq {
void skinny_go_sym(const SkinnyCall& c) {
    if (c.taps) skinny_tile<false, true, false>(c);
    else skinny_tile<false, false, false>(c);
}
}  // namespace aq
