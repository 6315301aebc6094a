// Pre-pass of the weighted fields, float.
#include "fields_pre.hpp"

namespace pkm {
PKM_PRE_INST(float)
}  // namespace pkm
