// The round kernels for level widths of 3 and 5 bits.
#include "qesgd_round_device.h"

namespace qesgd {
template void launch_round<3>(const RParams&, uint32_t, uint32_t, hipStream_t);
template void launch_round<5>(const RParams&, uint32_t, uint32_t, hipStream_t);
}  // namespace qesgd
