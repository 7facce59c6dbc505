// The kernels of the grid CWT by FFT (Eqs. (2)-(4)) for one grid size N, and the
// types that the host side shares.  Each supported size is a set of kernels of
// its own, made by run_cwt_n<N> (instantiated in the fft_n*.hip units): the radix
// plan, strides, tile counts and thread counts are constants, so that an index
// costs a few shifts and adds.  With one set of kernels for all sizes, whose
// indices went through multiply-high divisions, integer work was most of what the
// passes did: 238 vector instructions per complex element in the x forward pass
// at 432^3 (the vector ALUs busy for 65% of its time), 100 in a y pass.
//
// Data flow (n^3 grid, H = n/2 + 1, half spectrum S complex64 stored in tiles
// of YZ_TILE columns, see spec_at):
//   tables  : twiddles and the multiplier's 1D tables.
//   x_fwd   : rows of int64 rho -> float, two real rows packed as one complex
//             row, complex FFT along x, split into two half-spectrum rows;
//             also the exact 128-bit mass of the rows.
//   y_fwd   : complex FFT along y on tiles of YZ_TILE columns; one workgroup per
//             job also sums the row masses: mean density in FP64 -> overall scale.
//   z_mul   : forward FFT along z, times the multiplier and the scale,
//             inverse FFT along z, in LDS (one HBM round trip).
//   y_inv   : inverse along y.
//   x_inv   : two half-spectrum rows -> one complex row, inverse FFT, the
//             real and imaginary parts are the two output rows.
// Every 1D transform is a Stockham autosort FFT over radices 16/8/4/3/2 on a
// tile of pencils in LDS.  A pass's first stage reads straight from HBM into
// registers and its last one writes straight back (but for the split of x_fwd
// and the join of x_inv, which need a row's two ends at once), and the z pass
// turns from forward to inverse in registers.  Two radix-3 stages in a row are
// one step on 9 elements in registers.
#pragma once

#include "hf_internal.h"

namespace hf {

constexpr int YZ_LOG = 3;
constexpr int YZ_TILE = 1 << YZ_LOG;  // pencils per workgroup in the y and z passes
constexpr int FFT_ELEMS = 16;         // complex values per thread

// The half spectrum in HBM, in tiles of YZ_TILE columns: element (kx, y, z) of
// an n^3 grid at spec_at(n, kx / YZ_TILE, z, y) + kx % YZ_TILE.  A tile is an
// [z][y][column] block whose z planes are n + 1 rows apart, and tiles are
// n (n + 1) + 1 rows apart.  A y-pass tile (YZ_TILE columns at one z) is one
// contiguous run of n * YZ_TILE elements, a z-pass tile's elements are
// (n + 1) YZ_TILE apart inside one tile, and the x passes move YZ_TILE-column
// blocks of consecutive rows.  The spare rows keep those strides off powers of
// two, which would put a workgroup's accesses on few HBM channels.  Columns
// H .. tiles * YZ_TILE - 1 and the spare rows are padding that no pass reads.
constexpr int spec_tiles(int n) { return (n / 2 + 1 + YZ_TILE - 1) / YZ_TILE; }
constexpr size_t spec_tile_rows(int n) { return size_t(n) * (n + 1) + 1; }

// log2 of the row pairs per x-pass workgroup: at most `elems` complex values,
// between 4 and 16 pairs.  More pairs make longer runs in each spectrum tile.
constexpr int x_log_pairs(int n, int elems) {
    int lp = 4;
    while (lp > 2 && (n << lp) > elems) --lp;
    return lp;
}
constexpr int x_fwd_log_pairs(int n) { return x_log_pairs(n, 8192); }
constexpr int x_inv_log_pairs(int n) { return x_log_pairs(n, 8192); }

constexpr int64_t x_blocks(int n, int lp) { return (int64_t(n) * n / 2 + (1 << lp) - 1) >> lp; }

// Per-job workspace layout (offsets from the job's workspace base).
struct CwtLayout {
    size_t scalars, tw, btab, ptab, mass, spec, total;
};

// Up to MAX_BATCH same-n transforms in one launch per pass; the job index is a
// grid dimension and job j's workspace starts at ws + j * stride.
constexpr int MAX_BATCH = HF_CWT_BATCH_MAX;
struct CwtJobs {
    const int64_t *rho[MAX_BATCH];
    float *cwt[MAX_BATCH];
    double box_len[MAX_BATCH];
    double w[MAX_BATCH];
    int images[MAX_BATCH];
    char *ws;
    size_t stride;
    int mode;  // hf_kernel
    int count;
    // every job transforms job 0's density (one grid, several scales): the
    // forward x and y passes run for job 0 only and each job's z pass reads
    // job 0's half spectrum (and its normalisation) into its own; job 0's own
    // z pass, in place, runs in a launch after the others
    int shared_forward;
    int job_base;  // the z pass's first job (its launch covers job_base .. job_base + grid jobs - 1)
};

// Enqueues the whole transform for J.count jobs of size N (one launch per pass).
template <int N>
hf_status run_cwt_n(hf_ctx *ctx, const CwtJobs &J, const CwtLayout &L);

}  // namespace hf
