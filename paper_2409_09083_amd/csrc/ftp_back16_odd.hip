// ftp_back16.h: odd deltas, the caller's input map.
#include "ftp_back16.h"

namespace ftp {

template bool launch_back16<BF_ODD, false, false>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);

}  // namespace ftp
