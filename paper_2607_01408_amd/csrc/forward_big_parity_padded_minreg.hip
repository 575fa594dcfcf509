// The mixed-degree parity-basis kernels of L = 10, 12 and 16 (see forward_big_parity_padded.hip),
// built with the register-minimising scheduling strategy (build.py).  Forward, 65,536 units,
// (L, 2, L), fp32 / bf16, us, default strategy -> this one: L = 10 383 / 425 -> 368 / 407,
// L = 12 637 / 781 -> 623 / 766, L = 16 2,149 / 2,923 -> 2,136 / 2,883 (grad_x1 and grad_x2
// 4,363 -> 4,158); the other degrees are slower with it: L = 11 497 / 611 -> 513 / 618,
// L = 14 985 / 1,234 -> 1,055 / 1,373, L = 9 and 13 within 2%.
#include <hip/hip_runtime.h>

#include "forward_pair.h"
#include "internal.h"

namespace spingtp {
namespace {

template <typename TIO>
const KernelEntry* find_minreg(int L) {
    static const KernelEntry k[3] = {big_parity_padded_entry<10, TIO>(), big_parity_padded_entry<12, TIO>(),
                                     big_parity_padded_entry<16, TIO>()};
    return L == 10 ? &k[0] : L == 12 ? &k[1] : L == 16 ? &k[2] : nullptr;
}

}  // namespace

const KernelEntry* find_big_parity_padded_minreg_kernel(int L, int dtype) {
    return dtype == 0 ? find_minreg<float>(L) : dtype == 1 ? find_minreg<uint16_t>(L) : nullptr;
}

}  // namespace spingtp
