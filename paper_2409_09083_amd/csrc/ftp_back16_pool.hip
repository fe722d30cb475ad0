// ftp_back16.h: through a pool, the caller's input map.
#include "ftp_back16.h"

namespace ftp {

template bool launch_back16<BF_POOL, false, false>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);

}  // namespace ftp
