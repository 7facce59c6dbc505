// The transform's kernels for some of the grid sizes.
#include "fft_passes.h"

template hf_status hf::run_cwt_n<16>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<72>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<256>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<648>(hf_ctx *, const CwtJobs &, const CwtLayout &);
