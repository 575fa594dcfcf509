// The unrolled direct kernels (direct_unrolled.h) of the paired basis.
#include "direct_unrolled.h"

namespace spingtp {

const UnrolledKernel* find_unrolled_paired(int L) { return find_unrolled<pattern::kPaired>(L); }

}  // namespace spingtp
