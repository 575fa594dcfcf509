// The mixed-degree instantiations of the parity-basis large-degree kernel (spins
// {-1, 0, +1}, L = 9..16, fp32 and bf16 I/O; PAD in forward_pair.h); those of L = 10, 12 and 16
// are in forward_big_parity_padded_minreg.hip.
#include <hip/hip_runtime.h>

#include "forward_pair.h"
#include "internal.h"

namespace spingtp {
namespace {

template <typename TIO>
const KernelEntry* find_default(int L) {
    static const KernelEntry k[5] = {big_parity_padded_entry<9, TIO>(), big_parity_padded_entry<11, TIO>(),
                                     big_parity_padded_entry<13, TIO>(), big_parity_padded_entry<14, TIO>(),
                                     big_parity_padded_entry<15, TIO>()};
    switch (L) {
        case 9: return &k[0];
        case 11: return &k[1];
        case 13: case 14: case 15: return &k[L - 11];
        default: return nullptr;
    }
}

}  // namespace

const KernelEntry* find_big_parity_padded_kernel(int L, int dtype) {
    if (dtype != 0 && dtype != 1) return nullptr;
    const KernelEntry* k = find_big_parity_padded_minreg_kernel(L, dtype);
    return k != nullptr ? k : dtype == 0 ? find_default<float>(L) : find_default<uint16_t>(L);
}

}  // namespace spingtp
