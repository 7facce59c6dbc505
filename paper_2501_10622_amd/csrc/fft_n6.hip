// The transform's kernels for some of the grid sizes.
#include "fft_passes.h"

template hf_status hf::run_cwt_n<36>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<144>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<432>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<1024>(hf_ctx *, const CwtJobs &, const CwtLayout &);
