// Post-pass of the weighted fields in blocks of fewer lines, double.
#include "fields_post.hpp"

namespace pkm {
PKM_POST_FEW_INST(double)
}  // namespace pkm
