// Filter relayout as a launch of its own (ftp_prep.h).
#include "ftp_prep.h"

namespace ftp {

template <int CAP>
__global__ void __launch_bounds__(256)
k_prep_filters(PrepArgs<CAP> a)
{
    prep_block(a, (int)blockIdx.x);
}

namespace {

template <int CAP>
void launch_prep(const PrepJob* jobs, int n, hipStream_t s)
{
    PrepArgs<CAP> a;
    const int blocks = fill_prep(a, jobs, n);
    hipLaunchKernelGGL((k_prep_filters<CAP>), dim3((unsigned)blocks), dim3(256), 0, s, a);
}

}  // namespace

// n <= kPrepJobs
void prep_filters(const PrepJob* jobs, int n, hipStream_t s)
{
    if (n == 1) launch_prep<1>(jobs, n, s);
    else if (n <= kPrepFew) launch_prep<kPrepFew>(jobs, n, s);
    else launch_prep<kPrepJobs>(jobs, n, s);
}

}  // namespace ftp
