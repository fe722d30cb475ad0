// ftp_back16_1x1.h: odd deltas.
#include "ftp_back16_1x1.h"

namespace ftp {

template void launch_back16_1x1<BF_ODD>(const Back16OneArgs&, int, BfShape, unsigned, size_t, hipStream_t);

}  // namespace ftp
