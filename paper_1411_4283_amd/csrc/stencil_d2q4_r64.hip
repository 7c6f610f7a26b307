// Stencil kernels of dimension 2, order 4, up to 64 rows (one file per kernel, so that they
// compile in parallel).
#include "stencil_impl.hpp"

namespace cutcell {
CC_DISPATCH(2, 4, )
CC_ROWS(2, 4, 64, )
}  // namespace cutcell
