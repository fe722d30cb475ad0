// ftp_back_split.h: through a pool, the caller's input map.
#include "ftp_back_split.h"

namespace ftp {

template bool launch_back_split<true, false>(const BackSplitArgs&, int, int, SplitShape, unsigned, hipStream_t);

}  // namespace ftp
