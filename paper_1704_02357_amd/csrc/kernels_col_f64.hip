// Column passes, double.
#include "columns.hpp"

namespace pkm {
PKM_COLUMNS_INST(double)
}  // namespace pkm
