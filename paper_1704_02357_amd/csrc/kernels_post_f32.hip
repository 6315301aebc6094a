// Post-pass of the weighted fields, float.
#include "fields_post.hpp"

namespace pkm {
PKM_POST_INST(float)
}  // namespace pkm
