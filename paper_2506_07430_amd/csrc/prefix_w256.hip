// Prefix-shared kernels of one width class (see prefix_bf16.hpp).
#include "prefix_bf16.hpp"

namespace elocal {

ELOCAL_PREFIX_CLASS(w256, 8, 1, 2)

}  // namespace elocal
