// ftp_back16.h: odd deltas, input maps in the workspace.
#include "ftp_back16.h"

namespace ftp {

template bool launch_back16<BF_ODD, true, false>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);

}  // namespace ftp
