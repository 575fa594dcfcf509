// The unrolled direct kernels (direct_unrolled.h) of the paper basis.
#include "direct_unrolled.h"

namespace spingtp {

const UnrolledKernel* find_unrolled_paper(int L) { return find_unrolled<pattern::kPaper>(L); }

}  // namespace spingtp
