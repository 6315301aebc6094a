// Column passes, float.
#include "columns.hpp"

namespace pkm {
PKM_COLUMNS_INST(float)
}  // namespace pkm
