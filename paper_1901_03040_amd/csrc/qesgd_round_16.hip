// The round kernels for level widths of 16 bits.
#include "qesgd_round_device.h"

namespace qesgd {
template void launch_round<16>(const RParams&, uint32_t, uint32_t, hipStream_t);
}  // namespace qesgd
