// The round kernels for level widths of 6 and 7 bits.
#include "qesgd_round_device.h"

namespace qesgd {
template void launch_round<6>(const RParams&, uint32_t, uint32_t, hipStream_t);
template void launch_round<7>(const RParams&, uint32_t, uint32_t, hipStream_t);
}  // namespace qesgd
