// Step 3 (Eqs. (2)-(4)): the grid CWT as a real 3D FFT, a multiply by the
// wavelet's DFT-domain multiplier, and an inverse FFT, all in FP32 with
// FP64 only for the mean density and for table generation: the tables and the
// entry points.  The passes are in fft_passes.h, one set of kernels per size.
#include <cmath>

#include "fft_plan.h"

using namespace hf;

namespace {

// ---------------------------------------------------------------------------
// Tables, generated in FP64 and stored as FP32.
// ---------------------------------------------------------------------------
// One workgroup of TAB_THREADS per frequency k and job.  Twiddle tw[k] = exp(-2
// pi i k / n), and the separable multiplier M(kx,ky,kz) = P_x B_y B_z + B_x P_y
// B_z + B_x B_y P_z:
//  sampled : B = DFT(G), A = DFT(Hs), P = (alpha/3) B + beta A with
//            alpha = 6 dx^3 w^1.5, beta = -dx^3 w^3.5 (Eq. (4) split into
//            6 g g g - w^2 (x^2 g g g + ...), periodised and transformed), with
//            the periodised 1D Gaussian factors G_j = sum_m g(x_j + m L), Hs_j =
//            sum_m (x_j + m L)^2 g(...), g(t) = exp(-w^2 t^2 / 4) and x_j the
//            minimum-image offset of node j;
//  analytic: B = exp(-k^2/w^2), P = 32 pi^1.5 w^-3.5 k^2 B (the transform of Eq. (4)).
// Thread t sums the terms j = t, t + TAB_THREADS, ... and the partial sums are
// added in a fixed order.  Every workgroup forms the G_j and Hs_j it sums over,
// n (2 images + 1) FP64 exponentials, or (READ) takes them from where
// factors_kernel put them.
constexpr int TAB_THREADS = 256;

// n times the images up to which the workgroups form the factors themselves.  Each
// does all of them, which takes longer than a launch for them where there are many
// images (scales larger than the box) and the device is full of workgroups.  With
// the timer's events, 25 to 30 us a launch: n = 1024 71 us with one image, 83 with two,
// 110 with four (76 in two launches), 720 with 53 (110), 19.4 ms with 1600 (1.36); n =
// 256 39 us with six, 50 with 16 (69), 1.53 ms with 1600 (1.30).
constexpr int64_t TAB_OWN_MOST = 2048;

struct Factors {
    double G, Hs;
};

__device__ __forceinline__ Factors factors_of(int j, int n, double box_len, double w, int images) {
    const double dx = box_len / n;
    const int jc = (j + n / 2) % n - n / 2;
    Factors f{0.0, 0.0};
    for (int m = -images; m <= images; ++m) {
        const double x = jc * dx + m * box_len;
        const double g = exp(-0.25 * w * w * x * x);
        f.G += g;
        f.Hs += x * x * g;
    }
    return f;
}

// Where the factors of a job lie: in its half spectrum, which the x pass writes later.
__device__ __forceinline__ Factors *factors_at(const CwtJobs &J, const CwtLayout &L, int job) {
    return reinterpret_cast<Factors *>(J.ws + size_t(job) * J.stride + L.spec);
}

__global__ void __launch_bounds__(64) factors_kernel(CwtJobs J, CwtLayout L, int n) {
    const int j = blockIdx.x * 64 + threadIdx.x, job = blockIdx.y;
    if (j < n) factors_at(J, L, job)[j] = factors_of(j, n, J.box_len[job], J.w[job], J.images[job]);
}

template <bool READ>
__global__ void __launch_bounds__(TAB_THREADS) tables_kernel(CwtJobs J, CwtLayout L, int n) {
    const int k = blockIdx.x, job = blockIdx.y;
    char *ws = J.ws + size_t(job) * J.stride;
    auto *tw = reinterpret_cast<float2 *>(ws + L.tw);
    auto *btab = reinterpret_cast<float *>(ws + L.btab), *ptab = reinterpret_cast<float *>(ws + L.ptab);
    const double w = J.w[job], box_len = J.box_len[job];
    if (threadIdx.x == 0) {
        double s, c;
        sincospi(2.0 * double(k) / double(n), &s, &c);
        tw[k] = make_float2(float(c), float(-s));
    }
    if (J.mode == HF_KERNEL_ANALYTIC) {
        if (threadIdx.x != 0) return;
        const int ks = k <= n / 2 ? k : k - n;
        const double kk = 2.0 * M_PI * ks / box_len;
        const double B = exp(-(kk * kk) / (w * w));
        const double beta = 32.0 * pow(M_PI, 1.5) * pow(w, -3.5);
        btab[k] = float(B);
        ptab[k] = float(beta * kk * kk * B);
        return;
    }
    const double dx = box_len / n;
    double B = 0.0, A = 0.0;
    const int step = int((int64_t(TAB_THREADS) * k) % n);  // phase step between a thread's terms
    int ph = int((int64_t(threadIdx.x) * k) % n);
    for (int j = threadIdx.x; j < n; j += TAB_THREADS) {
        const Factors f = READ ? factors_at(J, L, job)[j] : factors_of(j, n, box_len, w, J.images[job]);
        const double c = cospi(2.0 * double(ph) / double(n));
        B += f.G * c;
        A += f.Hs * c;
        ph += step;
        if (ph >= n) ph -= n;
    }
    __shared__ double rb[TAB_THREADS], ra[TAB_THREADS];
    rb[threadIdx.x] = B;
    ra[threadIdx.x] = A;
    __syncthreads();
    for (int h = TAB_THREADS / 2; h > 0; h >>= 1) {
        if (int(threadIdx.x) < h) {
            rb[threadIdx.x] += rb[threadIdx.x + h];
            ra[threadIdx.x] += ra[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    B = rb[0];
    A = ra[0];
    const double dx3 = dx * dx * dx;
    const double alpha = 6.0 * dx3 * pow(w, 1.5);
    const double beta = -dx3 * pow(w, 3.5);
    btab[k] = float(B);
    ptab[k] = float(alpha / 3.0 * B + beta * A);
}

// ---------------------------------------------------------------------------
// workspace layout
// ---------------------------------------------------------------------------
CwtLayout cwt_layout(int n) {
    CwtLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes);
        return at;
    };
    L.scalars = take(64);
    L.tw = take(sizeof(float2) * n);
    L.btab = take(sizeof(float) * n);
    L.ptab = take(sizeof(float) * n);
    L.mass = take(sizeof(Mass128) * size_t(x_blocks(n, x_fwd_log_pairs(n))));
    L.spec = take(sizeof(float2) * size_t(spec_tiles(n)) * spec_tile_rows(n) * YZ_TILE);
    L.total = off;
    return L;
}

// Every n = 2^a 3^b with a >= 1 and 8 <= n <= 1024 (supported_n).
#define HF_FFT_SIZES(X)                                                                                      \
    X(8) X(12) X(16) X(18) X(24) X(32) X(36) X(48) X(54) X(64) X(72) X(96) X(108) X(128) X(144) X(162) X(192) \
    X(216) X(256) X(288) X(324) X(384) X(432) X(486) X(512) X(576) X(648) X(768) X(864) X(972) X(1024)

// Enqueues the whole transform for J.count same-n jobs.
hf_status run_cwt(hf_ctx *ctx, int n, const CwtJobs &J) {
    const CwtLayout L = cwt_layout(n);
    const dim3 each(n, unsigned(J.count));
    int images = 0;
    for (int j = 0; j < J.count; ++j) images = J.images[j] > images ? J.images[j] : images;
    if (J.mode == HF_KERNEL_SAMPLED && int64_t(n) * images > TAB_OWN_MOST) {
        HF_LAUNCH(ctx, K_TABLES_1, factors_kernel, dim3((n + 63) / 64, unsigned(J.count)), dim3(64), 0, ctx->stream, J, L, n);
        HF_LAUNCH(ctx, K_TABLES_2, tables_kernel<true>, each, dim3(TAB_THREADS), 0, ctx->stream, J, L, n);
    } else {
        HF_LAUNCH(ctx, K_TABLES_1, tables_kernel<false>, each, dim3(TAB_THREADS), 0, ctx->stream, J, L, n);
    }
    switch (n) {
#define HF_FFT_CASE(N) \
    case N: return run_cwt_n<N>(ctx, J, L);
        HF_FFT_SIZES(HF_FFT_CASE)
#undef HF_FFT_CASE
    }
    return HF_ERR_SIZE;
}

bool fill_job(CwtJobs &J, int j, const int64_t *rho, float *cwt, double box_len, double kw) {
    if (!rho || !cwt || !(kw > 0.0) || !std::isfinite(kw) || !(box_len > 0.0) || !(box_len < 1e300)) return false;
    J.rho[j] = rho;
    J.cwt[j] = cwt;
    J.box_len[j] = box_len;
    J.w[j] = 1000.0 * kw / box_len;  // step 1: k_w = w L / 1000
    // periodic images within w (I + 1/2) L >= 16, where the wavelet is < 1e-25 of its peak
    J.images[j] = std::max(1, int(std::ceil(16.0 / (J.w[j] * box_len) - 0.5)));
    return true;
}

}  // namespace

size_t hf::cwt_ws_bytes(const hf_box &box) { return cwt_layout(box.n).total; }

extern "C" hf_status hf_cwt(hf_ctx *ctx, const hf_box *box, const int64_t *rho, double kw, hf_kernel kernel,
                            float *cwt, void *ws, size_t ws_bytes) {
    if (!ctx || !rho || !cwt) return HF_ERR_ARG;
    if (kernel != HF_KERNEL_SAMPLED && kernel != HF_KERNEL_ANALYTIC && kernel != HF_KERNEL_STENCIL) return HF_ERR_ARG;
    if (!(kw > 0.0) || !std::isfinite(kw)) return HF_ERR_ARG;
    if (kernel == HF_KERNEL_STENCIL) {
        if (!box) return HF_ERR_ARG;
        const int32_t h = stencil_half_width(kw, box->n);  // Table 1's extent on this grid
        if (h < 0) return HF_ERR_ARG;
        return hf_cwt_stencil(ctx, box, rho, kw, h, cwt, ws, ws_bytes);
    }
    hf_status s = check_box(box);
    if (s != HF_OK) return s;
    const size_t need = cwt_layout(box->n).total;
    s = check_ws(ws, ws_bytes, need);
    if (s != HF_OK) return s;
    if (hipSetDevice(ctx->device) != hipSuccess) return HF_ERR_DEVICE;
    CwtJobs J{};
    if (!fill_job(J, 0, rho, cwt, box->box_len, kw)) return HF_ERR_ARG;
    J.ws = static_cast<char *>(ws);
    J.stride = need;
    J.mode = kernel;
    J.count = 1;
    return run_cwt(ctx, box->n, J);
}

extern "C" hf_status hf_cwt_scales(hf_ctx *ctx, const hf_box *box, const int64_t *rho, int32_t count,
                                   const double *kws, hf_kernel kernel, float *const *cwts, void *ws,
                                   size_t ws_bytes) {
    if (!ctx || !rho || !kws || !cwts || count < 1 || count > HF_CWT_BATCH_MAX) return HF_ERR_ARG;
    if (kernel != HF_KERNEL_SAMPLED && kernel != HF_KERNEL_ANALYTIC) return HF_ERR_ARG;
    hf_status s = check_box(box);
    if (s != HF_OK) return s;
    const size_t per = cwt_layout(box->n).total;
    s = check_ws(ws, ws_bytes, per * size_t(count));
    if (s != HF_OK) return s;
    CwtJobs J{};
    for (int j = 0; j < count; ++j)
        if (!fill_job(J, j, rho, cwts[j], box->box_len, kws[j])) return HF_ERR_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return HF_ERR_DEVICE;
    J.ws = static_cast<char *>(ws);
    J.stride = per;
    J.mode = kernel;
    J.count = count;
    J.shared_forward = 1;
    return run_cwt(ctx, box->n, J);
}

extern "C" hf_status hf_cwt_batch_ws_size(int32_t n, int32_t count, size_t *bytes) {
    if (!bytes || count < 1 || count > HF_CWT_BATCH_MAX) return HF_ERR_ARG;
    if (!supported_n(n)) return HF_ERR_SIZE;
    *bytes = cwt_layout(n).total * size_t(count);
    return HF_OK;
}

extern "C" hf_status hf_cwt_batch(hf_ctx *ctx, int32_t n, int32_t count, const hf_cwt_item *items, hf_kernel kernel,
                                  void *ws, size_t ws_bytes) {
    if (!ctx || !items || count < 1 || count > HF_CWT_BATCH_MAX) return HF_ERR_ARG;
    if (kernel != HF_KERNEL_SAMPLED && kernel != HF_KERNEL_ANALYTIC) return HF_ERR_ARG;
    if (!supported_n(n)) return HF_ERR_SIZE;
    const size_t per = cwt_layout(n).total;
    hf_status s = check_ws(ws, ws_bytes, per * size_t(count));
    if (s != HF_OK) return s;
    CwtJobs J{};
    for (int j = 0; j < count; ++j)
        if (!fill_job(J, j, items[j].rho, items[j].cwt, items[j].box_len, items[j].kw)) return HF_ERR_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return HF_ERR_DEVICE;
    J.ws = static_cast<char *>(ws);
    J.stride = per;
    J.mode = kernel;
    J.count = count;
    return run_cwt(ctx, n, J);
}
