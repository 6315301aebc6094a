// Post-pass of the weighted fields, double.
#include "fields_post.hpp"

namespace pkm {
PKM_POST_INST(double)
}  // namespace pkm
