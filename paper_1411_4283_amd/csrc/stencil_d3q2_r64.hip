// Stencil kernels of dimension 3, order 2, up to 64 rows (one file per kernel, so that they
// compile in parallel).
#include "stencil_impl.hpp"

namespace cutcell {
CC_DISPATCH(3, 2, )
CC_ROWS(3, 2, 64, )
}  // namespace cutcell
