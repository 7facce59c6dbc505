// The transform's kernels for some of the grid sizes.
#include "fft_passes.h"

template hf_status hf::run_cwt_n<48>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<162>(hf_ctx *, const CwtJobs &, const CwtLayout &);
template hf_status hf::run_cwt_n<486>(hf_ctx *, const CwtJobs &, const CwtLayout &);
