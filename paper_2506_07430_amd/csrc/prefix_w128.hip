// Prefix-shared kernels of one width class (see prefix_bf16.hpp).
#include "prefix_bf16.hpp"

namespace elocal {

ELOCAL_PREFIX_CLASS(w128, 4, 1, 1)

}  // namespace elocal
