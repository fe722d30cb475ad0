// ftp_back_split.h: no pool, input maps in the workspace.
#include "ftp_back_split.h"

namespace ftp {

template bool launch_back_split<false, true>(const BackSplitArgs&, int, int, SplitShape, unsigned, hipStream_t);

}  // namespace ftp
