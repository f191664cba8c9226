// The round kernels for level widths of 1 and 2 bits.
#include "qesgd_round_device.h"

namespace qesgd {
template void launch_round<1>(const RParams&, uint32_t, uint32_t, hipStream_t);
template void launch_round<2>(const RParams&, uint32_t, uint32_t, hipStream_t);
}  // namespace qesgd
