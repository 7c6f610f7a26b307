// Stencil kernels of dimension 2, order 4, 97 to 128 rows (one file per kernel, so that they
// compile in parallel).
#include "stencil_impl.hpp"

namespace cutcell {
CC_ROWS(2, 4, 128, )
}  // namespace cutcell
