// The transform's kernels for some of the grid sizes.
#include "fft_passes.h"

template hf_status hf::run_cwt_n<8>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<54>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<192>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<512>(hf_ctx *, const CwtJobs &, const CwtLayout &);
