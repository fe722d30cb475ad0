// ftp_back16_1x1.h: through a pool.
#include "ftp_back16_1x1.h"

namespace ftp {

template void launch_back16_1x1<BF_POOL>(const Back16OneArgs&, int, BfShape, unsigned, size_t, hipStream_t);

}  // namespace ftp
