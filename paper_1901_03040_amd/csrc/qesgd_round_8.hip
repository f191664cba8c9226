// The round kernels for level widths of 8 bits.
#include "qesgd_round_device.h"

namespace qesgd {
template void launch_round<8>(const RParams&, uint32_t, uint32_t, hipStream_t);
}  // namespace qesgd
