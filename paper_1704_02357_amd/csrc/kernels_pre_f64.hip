// Pre-pass of the weighted fields, double.
#include "fields_pre.hpp"

namespace pkm {
PKM_PRE_INST(double)
}  // namespace pkm
