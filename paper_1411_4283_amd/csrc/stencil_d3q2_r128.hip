// Stencil kernels of dimension 3, order 2, 97 to 128 rows (one file per kernel, so that they
// compile in parallel).
#include "stencil_impl.hpp"

namespace cutcell {
CC_ROWS(3, 2, 128, )
}  // namespace cutcell
