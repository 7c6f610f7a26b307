// Stencil kernels of dimension 3, order 4, 65 to 96 rows (one file per kernel, so that they
// compile in parallel).
#include "stencil_impl.hpp"

namespace cutcell {
CC_ROWS(3, 4, 96, )
}  // namespace cutcell
