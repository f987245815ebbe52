// beamSearch on RaBitQ codes: the instances of beam_kernels.h for 4- and 8-bit codes (nibble planes) and 1- and 2-bit
// codes (bit planes).
#include "beam_launch.h"

namespace jx {

hipError_t launch_beam_codes(int kind, int qbits, const BeamArgs& a, hipStream_t st, char* kernel_name) {
    if (kind == K_RQ4) return qbits == 8 ? launch_shape<K_RQ4, 8>(a, st, kernel_name) : launch_shape<K_RQ4, 4>(a, st, kernel_name);
    if (kind == K_RQ1) return qbits == 8 ? launch_shape<K_RQ1, 8>(a, st, kernel_name) : launch_shape<K_RQ1, 4>(a, st, kernel_name);
    return hipErrorInvalidValue;
}

}  // namespace jx
