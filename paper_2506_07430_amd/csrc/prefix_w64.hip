// Prefix-shared kernels of one width class (see prefix_bf16.hpp).
#include "prefix_bf16.hpp"

namespace elocal {

ELOCAL_PREFIX_CLASS(w64, 2, 1, 1)
ELOCAL_PREFIX_CLASS(w64c2, 2, 2, 1)

}  // namespace elocal
