// ftp_back16.h: even deltas, input maps in the workspace, the gradient in rows.
#include "ftp_back16.h"

namespace ftp {

template bool launch_back16<BF_WS, true, true>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);

}  // namespace ftp
