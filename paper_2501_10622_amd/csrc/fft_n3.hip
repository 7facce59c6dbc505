// The transform's kernels for some of the grid sizes.
#include "fft_passes.h"

template hf_status hf::run_cwt_n<18>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<96>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<288>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<768>(hf_ctx *, const CwtJobs &, const CwtLayout &);
