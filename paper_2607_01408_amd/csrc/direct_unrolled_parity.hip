// The unrolled direct kernels (direct_unrolled.h) of the parity basis.
#include "direct_unrolled.h"

namespace spingtp {

const UnrolledKernel* find_unrolled_parity(int L) { return find_unrolled<pattern::kParity>(L); }

}  // namespace spingtp
