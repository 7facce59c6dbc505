// Kernels and launches of run_cwt_n<N>; included by the units that instantiate it.
#pragma once

#include "fft_plan.h"

using namespace hf;

namespace {

// ---------------------------------------------------------------------------
// plans
// ---------------------------------------------------------------------------
constexpr int MAX_STAGES = 12;

struct FftPlan {
    int nst;
    int radix[MAX_STAGES];
};

constexpr FftPlan make_plan(int n) {
    FftPlan p{};
    int m = n;
    while (m % 3 == 0) {
        p.radix[p.nst++] = 3;
        m /= 3;
    }
    const int two[4] = {16, 8, 4, 2};
    for (int i = 0; i < 4; ++i)
        while (m % two[i] == 0) {
            p.radix[p.nst++] = two[i];
            m /= two[i];
        }
    return p;
}

// The same factors with the last one moved to the front: the inverse transform
// that follows a forward one in registers starts with the radix the forward
// one ended with.
constexpr FftPlan rotate_plan(FftPlan f) {
    FftPlan p = f;
    p.radix[0] = f.radix[f.nst - 1];
    for (int s = 1; s < f.nst; ++s) p.radix[s] = f.radix[s - 1];
    return p;
}

template <int N, bool ROT>
struct PlanOf {
    static constexpr FftPlan p = ROT ? rotate_plan(make_plan(N)) : make_plan(N);
    static constexpr int radix(int s) { return p.radix[s]; }
    static constexpr int before(int s) {  // product of the radices before stage s
        int ns = 1;
        for (int i = 0; i < s; ++i) ns *= p.radix[i];
        return ns;
    }
};

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
// a (wr + i wi) with the roundings spelled out: of the two products of the real
// part, and of the imaginary part, the one with a.x (X) or a.y (Y) is rounded and
// goes into the fused multiply-add of the other.  Left to the compiler, the choice
// would follow the code around it, and so would the last bits of the field and,
// where two cells are that close, the labels.
enum class Round { XX, YX, XY, YY };
template <Round M>
__device__ __forceinline__ float2 turn(float2 a, float wr, float wi) {
    constexpr bool rx = M == Round::XX || M == Round::XY, ix = M == Round::XX || M == Round::YX;
    return make_float2(rx ? fmaf(-a.y, wi, a.x * wr) : fmaf(a.x, wr, -(a.y * wi)),
                       ix ? fmaf(a.y, wr, a.x * wi) : fmaf(a.x, wi, a.y * wr));
}

// multiply by -i (forward) or +i (inverse)
template <bool INV>
__device__ __forceinline__ float2 mul_mi(float2 a) {
    return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

template <bool INV>
__device__ __forceinline__ void dft2(float2 &a, float2 &b) {
    float2 t = a;
    a = cadd(t, b);
    b = csub(t, b);
}

template <bool INV>
__device__ __forceinline__ void dft4(float2 &v0, float2 &v1, float2 &v2, float2 &v3) {
    float2 t0 = cadd(v0, v2), t1 = csub(v0, v2);
    float2 t2 = cadd(v1, v3), t3 = mul_mi<INV>(csub(v1, v3));
    v0 = cadd(t0, t2);
    v2 = csub(t0, t2);
    v1 = cadd(t1, t3);
    v3 = csub(t1, t3);
}

// Where a transform stands: between stages, at a pass's end with its outputs
// going to global memory, at the z pass's seam, or as the z pass's only stage.
// The radix-16 transform has roundings of its own in each, those of the kernels
// for all sizes that made the fields before (the same bits at every size when these
// took their place; the tests hold the fields to a tolerance against FP64).  Radix 8
// and the multiplier leave the choice to the compiler.
enum class Place { Mid, End, Seam, Only };

template <int R, bool INV, Place PLACE = Place::Mid>
__device__ __forceinline__ void dft(float2 (&v)[R]) {
    if constexpr (R == 2) {
        dft2<INV>(v[0], v[1]);
    } else if constexpr (R == 4) {
        dft4<INV>(v[0], v[1], v[2], v[3]);
    } else if constexpr (R == 8) {
        // radix-8 as two radix-4 transforms of the even and odd inputs
        float2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
        float2 o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
        dft4<INV>(e0, e1, e2, e3);
        dft4<INV>(o0, o1, o2, o3);
        const float r = 0.70710678118654752440f;
        // o_s *= exp(-+ 2 pi i s / 8)
        o1 = INV ? make_float2(r * (o1.x - o1.y), r * (o1.x + o1.y)) : make_float2(r * (o1.x + o1.y), r * (o1.y - o1.x));
        o2 = mul_mi<INV>(o2);
        o3 = INV ? make_float2(-r * (o3.x + o3.y), r * (o3.x - o3.y)) : make_float2(r * (o3.y - o3.x), -r * (o3.x + o3.y));
        v[0] = cadd(e0, o0);
        v[4] = csub(e0, o0);
        v[1] = cadd(e1, o1);
        v[5] = csub(e1, o1);
        v[2] = cadd(e2, o2);
        v[6] = csub(e2, o2);
        v[3] = cadd(e3, o3);
        v[7] = csub(e3, o3);
    } else if constexpr (R == 16) {
        // 16 = 4 x 4: element 4 a + b; length-4 transforms over a, the twiddles
        // W16^(b c), length-4 transforms over b; output c + 4 d sits at 4 c + d
        dft4<INV>(v[0], v[4], v[8], v[12]);
        dft4<INV>(v[1], v[5], v[9], v[13]);
        dft4<INV>(v[2], v[6], v[10], v[14]);
        dft4<INV>(v[3], v[7], v[11], v[15]);
        const float c1 = 0.92387953251128675613f, s1 = 0.38268343236508977173f, h = 0.70710678118654752440f;
        const float sg = INV ? 1.f : -1.f;  // exp(-+ 2 pi i m / 16) = cos - + i sin
        constexpr Round A = INV ? Round::YX : Round::XX;  // m = 1, 3
        constexpr Round B = INV || PLACE == Place::End || PLACE == Place::Only ? Round::YY : Round::XX;
        constexpr Round C = INV ? Round::XY : Round::YY;  // m = 9
        constexpr Round D = INV && (PLACE == Place::Seam || PLACE == Place::Only) ? Round::YY : Round::XX;
        constexpr Round E = INV && (PLACE == Place::End || PLACE == Place::Only) ? Round::YY : Round::XX;
        v[5] = turn<A>(v[5], c1, sg * s1);            // m = 1
        v[9] = turn<D>(v[9], h, sg * h);              // m = 2
        v[13] = turn<A>(v[13], s1, sg * c1);          // m = 3
        v[6] = turn<E>(v[6], h, sg * h);              // m = 2
        v[10] = mul_mi<INV>(v[10]);                   // m = 4
        v[14] = turn<B>(v[14], -h, sg * h);           // m = 6
        v[7] = turn<A>(v[7], s1, sg * c1);            // m = 3
        v[11] = turn<INV ? Round::YY : Round::XX>(v[11], -h, sg * h);  // m = 6
        v[15] = turn<C>(v[15], -c1, -sg * s1);        // m = 9
        dft4<INV>(v[0], v[1], v[2], v[3]);
        dft4<INV>(v[4], v[5], v[6], v[7]);
        dft4<INV>(v[8], v[9], v[10], v[11]);
        dft4<INV>(v[12], v[13], v[14], v[15]);
        float2 t[16];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int d = 0; d < 4; ++d) t[c + 4 * d] = v[4 * c + d];
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = t[e];
    } else if constexpr (R == 3) {
        const float c = -0.5f;
        const float s = INV ? 0.86602540378443864676f : -0.86602540378443864676f;
        float2 t = cadd(v[1], v[2]);
        float2 d = csub(v[1], v[2]);
        float2 m = make_float2(fmaf(c, t.x, v[0].x), fmaf(c, t.y, v[0].y));
        v[0] = cadd(v[0], t);
        v[1] = make_float2(fmaf(-s, d.y, m.x), fmaf(s, d.x, m.y));  // m + i s d
        v[2] = make_float2(fmaf(s, d.y, m.x), fmaf(-s, d.x, m.y));  // m - i s d
    }
}

// Two layouts of the pencils of a tile.  The y and z passes, whose columns lie
// side by side in memory, keep element x of pencil p at buf[x P + p] (P
// pencils) and give consecutive lanes consecutive pencils.  The x passes (ROWS),
// whose pencils are rows of memory, keep it at buf[p pitch + row_at(x)] and give
// consecutive lanes consecutive butterflies of one row: their global accesses
// are whole runs of the rows, and the place left free after every 16 elements
// spreads a stage's strided stores (powers of two up to 16) over the banks.
// The twiddles of ROWS stages are spread the same way.
__host__ __device__ constexpr int row_at(int x) { return x + (x >> 4); }

// Places of a row: rows start 8 places apart modulo 16, so that the x passes'
// accesses of 8 columns by several rows fall on distinct banks.
constexpr int row_pitch(int n) { return (row_at(n) + 7) / 16 * 16 + 8; }

constexpr int log2_of(int x) {
    int l = 0;
    while ((1 << l) < x) ++l;
    return l;
}

// FFT_ELEMS values per thread and, above two wavefronts, a multiple of four of
// them: the wavefronts of a workgroup go round the CU's four SIMDs, and with five
// to seven of them some SIMDs get twice the work of the others.  At 768^3, six
// wavefronts against eight that are not all in use: x forward 1814 -> 1056 us,
// z 1381 -> 941, x inverse 995 -> 697; at 384^3 x forward 247 -> 151.
constexpr int threads_for(int elems) {
    const int t = (elems + FFT_ELEMS - 1) / FFT_ELEMS;
    return t <= 64 ? 64 : t <= 128 ? 128 : t > 768 ? 1024 : (t + 255) / 256 * 256;
}

// One transform of a tile: size, direction, plan, layout, pencils and threads,
// whether its input and output are in LDS, and the stages [FROM, TO) it runs.
template <int N_, bool INV_, bool ROT, bool ROWS_, int P_, int T_, bool LOAD_LDS_, bool STORE_LDS_, int FROM_, int TO_>
struct Tile {
    static constexpr int N = N_, P = P_, T = T_, FROM = FROM_, TO = TO_;
    static constexpr bool INV = INV_, ROWS = ROWS_, LOAD_LDS = LOAD_LDS_, STORE_LDS = STORE_LDS_;
    using Plan = PlanOf<N_, ROT>;
    static __device__ __forceinline__ int at(int p, int x) {
        return ROWS ? p * row_pitch(N) + row_at(x) : (x << log2_of(P)) + p;
    }
};

// The butterflies of thread tid in a step of NBF per pencil: pencil p[i], index
// j[i] of the first element, on[i] whether there is one.  The indices are made
// opaque: from j = tid + i T - p NBF the compiler would else take the constant
// i T into an LDS access's offset, which leaves a negative base register, and
// such accesses have returned wrong values (the x passes at 96^3).
template <class C, int NBF>
struct Butterflies {
    static constexpr int TOTAL = NBF * C::P, MAXB = (TOTAL + C::T - 1) / C::T;
    int p[MAXB], j[MAXB];
    bool on[MAXB];
    __device__ __forceinline__ explicit Butterflies(uint32_t tid) {
#pragma unroll
        for (int i = 0; i < MAXB; ++i) {
            const uint32_t b = tid + uint32_t(i * C::T);
            uint32_t pp, jj;
            if constexpr (!C::ROWS) {
                pp = tid & uint32_t(C::P - 1);
                jj = b >> log2_of(C::P);
            } else {
                pp = b / uint32_t(NBF);
                jj = b - pp * uint32_t(NBF);
            }
            p[i] = C::ROWS ? opaque(int(pp)) : int(pp);
            j[i] = opaque(int(jj));
            on[i] = TOTAL % C::T == 0 || b < uint32_t(TOTAL);
        }
    }
};

// A product by a twiddle, rounded as it stands: the adds of the transform it
// goes into are not contracted with it, whatever the compiler sees of them.
__device__ __forceinline__ float2 twiddled(float2 a, float2 w) {
    float2 v = turn<Round::YX>(a, w.x, w.y);
    asm("" : "+v"(v.x), "+v"(v.y));
    return v;
}

// One step: a radix-R1 stage (Ns = NS, the product of the radices before it),
// or, with R2 > 1, that stage and the radix-R2 stage after it on R1 R2 elements
// in registers.  With R = R1 R2 and NBF = N / R, butterfly j takes the elements
// j + e NBF through load(p, index); stage one transforms the elements q + R2 r
// over r (twiddles r k, k = j mod NS), stage two, for each r, its outputs over q
// (twiddles q (k + r NS)); output (r, s) is element (j - k) R + k + r NS + s R1
// NS and goes to store(p, index, value).  Each value meets the operations of the
// two separate stages in the same order.  With sync, the loads of the whole
// workgroup end before the first store (LDS in place).
template <class C, int R1, int R2, int NS, bool SYNC, Place PLACE, class Load, class Store>
__device__ __forceinline__ void fft_step(const float2 *tw, int tid, Load &load, Store &store) {
    constexpr int N = C::N, R = R1 * R2, NBF = N / R;
    using B = Butterflies<C, NBF>;
    const B b(opaque(tid));  // index arithmetic stays in its step
    auto twiddle = [tw](int m) {
        float2 w = tw[C::ROWS ? row_at(m) : m];
        if (C::INV) w.y = -w.y;
        return w;
    };
    float2 v[B::MAXB][R];
#pragma unroll
    for (int i = 0; i < B::MAXB; ++i) {
        if (b.on[i]) {
#pragma unroll
            for (int e = 0; e < R; ++e) v[i][e] = load(b.p[i], b.j[i] + e * NBF);
        }
    }
    if constexpr (NS > 1) {
#pragma unroll
        for (int i = 0; i < B::MAXB; ++i) {
            if (b.on[i]) {
                const int k = int(uint32_t(b.j[i]) % uint32_t(NS));
#pragma unroll
                for (int r = 1; r < R1; ++r) {
                    const float2 w = twiddle(r * k * (N / (NS * R1)));
#pragma unroll
                    for (int q = 0; q < R2; ++q) v[i][q + R2 * r] = twiddled(v[i][q + R2 * r], w);
                }
            }
        }
    }
    if (SYNC) __syncthreads();
#pragma unroll
    for (int i = 0; i < B::MAXB; ++i) {
        if (!b.on[i]) continue;
        const int p = b.p[i], j = b.j[i];
        const int k = NS > 1 ? int(uint32_t(j) % uint32_t(NS)) : 0;
        const int base = (j - k) * R + k;
        if constexpr (R2 == 1) {
            dft<R1, C::INV, PLACE>(v[i]);
#pragma unroll
            for (int r = 0; r < R1; ++r) store(p, base + r * NS, v[i][r]);
        } else {
#pragma unroll
            for (int q = 0; q < R2; ++q) {
                float2 t[R1];
#pragma unroll
                for (int r = 0; r < R1; ++r) t[r] = v[i][q + R2 * r];
                dft<R1, C::INV>(t);
#pragma unroll
                for (int r = 0; r < R1; ++r) v[i][q + R2 * r] = t[r];
            }
#pragma unroll
            for (int r = 0; r < R1; ++r) {
                float2 t[R2];
                t[0] = v[i][R2 * r];
#pragma unroll
                for (int q = 1; q < R2; ++q) {
                    t[q] = v[i][q + R2 * r];
                    if (NS > 1 || r > 0) t[q] = twiddled(t[q], twiddle(q * (k + r * NS) * (N / (NS * R))));
                }
                dft<R2, C::INV, PLACE>(t);
#pragma unroll
                for (int s = 0; s < R2; ++s) store(p, base + r * NS + s * R1 * NS, t[s]);
            }
        }
    }
}

// The steps of C's plan from stage S on: the first reads through load, the
// last writes through store, the others go from LDS to LDS, with a barrier after
// every step but the last.
template <class C, int S, class Load, class Store>
__device__ __forceinline__ void fft_steps(float2 *buf, const float2 *tw, int tid, Load &load, Store &store) {
    using Plan = typename C::Plan;
    constexpr int R1 = Plan::radix(S);
    constexpr bool two = S + 1 < C::TO && R1 == 3 && Plan::radix(S + 1 < C::TO ? S + 1 : S) == 3;
    constexpr int R2 = two ? 3 : 1, NS = Plan::before(S), NEXT = S + (two ? 2 : 1);
    constexpr bool first = S == C::FROM, last = NEXT == C::TO;
    auto lload = [buf](int p, int x) { return buf[C::at(p, x)]; };
    auto lstore = [buf](int p, int x, float2 v) { buf[C::at(p, x)] = v; };
    constexpr Place end = C::STORE_LDS || C::ROWS ? Place::Mid : Place::End;
    if constexpr (first && last) fft_step<C, R1, R2, NS, (C::LOAD_LDS && C::STORE_LDS) || two, end>(tw, tid, load, store);
    // (a first step of two stages reads twiddles, which the workgroup has just put into LDS)
    else if constexpr (first) fft_step<C, R1, R2, NS, C::LOAD_LDS || two, Place::Mid>(tw, tid, load, lstore);
    else if constexpr (last) fft_step<C, R1, R2, NS, C::STORE_LDS, end>(tw, tid, lload, store);
    else fft_step<C, R1, R2, NS, true, Place::Mid>(tw, tid, lload, lstore);
    if constexpr (!last) {
        __syncthreads();
        fft_steps<C, NEXT>(buf, tw, tid, load, store);
    }
}

// The seam of the z pass: the last forward stage (Ns = N/R, so k = j and its
// outputs are elements j + r N/R), the multiplier, and the first inverse stage
// (Ns = 1, inputs j + r N/R, outputs j R + r), in registers.
template <class C, int R, bool SYNC, class Load, class Store, class Mul>
__device__ __forceinline__ void fft_seam(const float2 *tw, int tid, Load &load, Store &store, Mul &mul) {
    constexpr int NBF = C::N / R;
    using B = Butterflies<C, NBF>;
    const B b(opaque(tid));
    float2 v[B::MAXB][R];
#pragma unroll
    for (int i = 0; i < B::MAXB; ++i) {
        if (b.on[i]) {
#pragma unroll
            for (int r = 0; r < R; ++r) v[i][r] = load(b.p[i], b.j[i] + r * NBF);
            if constexpr (NBF > 1) {  // the twiddles' stride is 1 and k = j
#pragma unroll
                for (int r = 1; r < R; ++r) v[i][r] = twiddled(v[i][r], tw[r * b.j[i]]);
            }
        }
    }
    if (SYNC) __syncthreads();
#pragma unroll
    for (int i = 0; i < B::MAXB; ++i) {
        if (!b.on[i]) continue;
        const int p = b.p[i], j = b.j[i];
        constexpr Place PLACE = SYNC ? Place::Seam : Place::Only;
        dft<R, false, PLACE>(v[i]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float m = mul(p, j + r * NBF);
            v[i][r] = make_float2(v[i][r].x * m, v[i][r].y * m);
        }
        dft<R, true, PLACE>(v[i]);
#pragma unroll
        for (int r = 0; r < R; ++r) store(p, j * R + r, v[i][r]);
    }
}

// Loads of a workgroup's tile are issued as one batch into registers before
// any is written to LDS, so each thread keeps all of its loads in flight
// (a load-store loop would wait for every load in turn).
template <int N, int T, bool ROWS>
__device__ __forceinline__ void load_twiddles(float2 *tw_s, const float2 *tw_g) {
    constexpr int PER = (N + T - 1) / T;
    float2 t[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = threadIdx.x + i * T;
        if (e < N) t[i] = tw_g[e];
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = threadIdx.x + i * T;
        if (e < N) tw_s[ROWS ? row_at(e) : e] = t[i];
    }
}

// ---------------------------------------------------------------------------
// jobs
// ---------------------------------------------------------------------------
struct JobView {
    double *scalars;
    float2 *tw;
    float *btab, *ptab;
    Mass128 *mass;
    float2 *spec;
};

__device__ __forceinline__ JobView job_view(const CwtJobs &J, const CwtLayout &L, int j) {
    char *b = J.ws + size_t(j) * J.stride;
    JobView v;
    v.scalars = reinterpret_cast<double *>(b + L.scalars);
    v.tw = reinterpret_cast<float2 *>(b + L.tw);
    v.btab = reinterpret_cast<float *>(b + L.btab);
    v.ptab = reinterpret_cast<float *>(b + L.ptab);
    v.mass = reinterpret_cast<Mass128 *>(b + L.mass);
    v.spec = reinterpret_cast<float2 *>(b + L.spec);
    return v;
}

template <int N>
__device__ __forceinline__ size_t spec_at(int tile, int z, int y) {
    return (size_t(tile) * spec_tile_rows(N) + size_t(z) * (N + 1) + size_t(y)) * YZ_TILE;
}

// ---------------------------------------------------------------------------
// x passes
// ---------------------------------------------------------------------------
template <int N, int LP>
struct XTile {
    static constexpr int P = 1 << LP, T = threads_for(N << LP), H = N / 2 + 1, NT = spec_tiles(N), ROWS = 2 * P;
    static constexpr int64_t PAIRS = int64_t(N) * N / 2;
    static constexpr bool WHOLE = PAIRS % P == 0;  // no workgroup has absent pairs
};

constexpr int x_fwd_threads(int n) { return threads_for(n << x_fwd_log_pairs(n)); }
constexpr int x_inv_threads(int n) { return threads_for(n << x_inv_log_pairs(n)); }

// One workgroup = P row pairs (rows 2q, 2q + 1 of the N N rows of x); the first
// stage takes the two rows of a pair straight from the grid.  Bound by HBM at
// powers of two and by LDS at the others: it reads 8 bytes and writes 4 per cell.
// Measured, one set of kernels for all sizes with pencils side by side in LDS
// against this one: 1024^3 3353 -> 2384 us (5.4 TB/s), 512^3 452 -> 343, 432^3
// 345 -> 206, 256^3 60 -> 45.
template <int N>
__global__ void __launch_bounds__(x_fwd_threads(N)) fft_x_fwd_kernel(CwtJobs J, CwtLayout L, uint32_t *status) {
    using X = XTile<N, x_fwd_log_pairs(N)>;
    using Plan = PlanOf<N, false>;
    constexpr int T = X::T, P = X::P;
    __shared__ float2 tw[row_at(N)];
    __shared__ float2 buf[P * row_pitch(N)];
    __shared__ unsigned long long red_lo[T / 64], red_hi[T / 64];
    const JobView jv = job_view(J, L, blockIdx.y);
    const int tid = threadIdx.x;
    const int64_t q0 = int64_t(blockIdx.x) * P;
    const int64_t *__restrict__ rho = J.rho[blockIdx.y] + q0 * (2 * N);
    const int pairs = X::WHOLE ? P : int(X::PAIRS - q0 < P ? X::PAIRS - q0 : P);
    load_twiddles<N, T, true>(tw, jv.tw);  // read after a barrier of the first step
    unsigned long long lo = 0, hi = 0;
    long long sign = 0;
    auto gload = [&](int p, int x) {
        if (!X::WHOLE && p >= pairs) return make_float2(0.f, 0.f);
        const int64_t a = rho[p * (2 * N) + x], b = rho[p * (2 * N) + N + x];
        sign |= a | b;
        add128(lo, hi, static_cast<unsigned long long>(a));
        add128(lo, hi, static_cast<unsigned long long>(b));
        return make_float2(float(a), float(b));
    };
    auto lstore = [](int p, int x, float2 v) { buf[p * row_pitch(N) + row_at(x)] = v; };
    using C = Tile<N, false, false, true, P, T, false, true, 0, Plan::p.nst>;
    fft_steps<C, 0>(buf, tw, tid, gload, lstore);
    if (sign < 0) atomicOr(status, ST_INPUT);
    // workgroup sum of the 128-bit masses (fixed order: deterministic)
    for (int off = 32; off > 0; off >>= 1) {
        unsigned long long olo = __shfl_down(lo, off, 64);
        unsigned long long ohi = __shfl_down(hi, off, 64);
        add128(lo, hi, olo);
        hi += ohi;
    }
    if ((tid & 63) == 0) {
        red_lo[tid >> 6] = lo;
        red_hi[tid >> 6] = hi;
    }
    __syncthreads();
    if (tid == 0) {
        unsigned long long a = 0, b = 0;
        for (int w = 0; w < T / 64; ++w) {
            add128(a, b, red_lo[w]);
            b += red_hi[w];
        }
        jv.mass[blockIdx.x].lo = a;
        jv.mass[blockIdx.x].hi = b;
    }
    // split Z = A + iB into the two real rows' spectra; a wavefront writes one
    // column tile of the workgroup's consecutive rows
    float2 *__restrict__ spec = jv.spec;
    const uint32_t row0 = uint32_t(2 * q0);
    for (int e = tid; e < X::NT * YZ_TILE * X::ROWS; e += T) {
        const int c = e & (YZ_TILE - 1), r = (e >> YZ_LOG) & (X::ROWS - 1), tile = (e >> YZ_LOG) / X::ROWS;
        const int k = tile * YZ_TILE + c, p = r >> 1;
        if (k >= X::H || (!X::WHOLE && p >= pairs)) continue;
        const float2 zk = buf[p * row_pitch(N) + row_at(k)];
        const float2 zm = buf[p * row_pitch(N) + row_at(k ? N - k : 0)];
        const float2 v = (r & 1) ? make_float2(0.5f * (zk.y + zm.y), -0.5f * (zk.x - zm.x))  // B, row 2q + 1
                                 : make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));  // A, row 2q
        const uint32_t row = row0 + uint32_t(r), z = row / uint32_t(N);
        spec[spec_at<N>(tile, int(z), int(row - z * uint32_t(N))) + c] = v;
    }
}

// The last stage writes the two rows of a pair straight to the field: 4 bytes
// read and 4 written per cell, bound like x_fwd.  1024^3 2580 -> 1553 us (5.5
// TB/s), 432^3 309 -> 136, 256^3 47 -> 32.
template <int N>
__global__ void __launch_bounds__(x_inv_threads(N)) fft_x_inv_kernel(CwtJobs J, CwtLayout L) {
    using X = XTile<N, x_inv_log_pairs(N)>;
    using Plan = PlanOf<N, false>;
    constexpr int T = X::T, P = X::P;
    __shared__ float2 tw[row_at(N)];
    __shared__ float2 buf[P * row_pitch(N)];
    const JobView jv = job_view(J, L, blockIdx.y);
    const float2 *__restrict__ spec = jv.spec;
    const int tid = threadIdx.x;
    const int64_t q0 = int64_t(blockIdx.x) * P;
    float *__restrict__ out = J.cwt[blockIdx.y] + q0 * (2 * N);
    const int pairs = X::WHOLE ? P : int(X::PAIRS - q0 < P ? X::PAIRS - q0 : P);
    const uint32_t row0 = uint32_t(2 * q0);
    load_twiddles<N, T, true>(tw, jv.tw);
    // element e: column c of tile `tile` for pair p; a wavefront reads one column
    // tile of consecutive rows
    constexpr int SPAN = X::NT * YZ_TILE * P, PER = (SPAN + T - 1) / T;
    float2 va[PER], vb[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = tid + i * T;
        const int c = e & (YZ_TILE - 1), p = (e >> YZ_LOG) & (P - 1), tile = (e >> YZ_LOG) / P;
        if (tile * YZ_TILE + c < X::H && (X::WHOLE || p < pairs)) {
            // rows 2q and 2q + 1 share z (N is even)
            const uint32_t row = row0 + 2 * uint32_t(p), z = row / uint32_t(N);
            const size_t at = spec_at<N>(tile, int(z), int(row - z * uint32_t(N))) + c;
            va[i] = spec[at];
            vb[i] = spec[at + YZ_TILE];
        }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = tid + i * T;
        const int c = e & (YZ_TILE - 1), p = (e >> YZ_LOG) & (P - 1), tile = (e >> YZ_LOG) / P;
        const int k = tile * YZ_TILE + c;
        if (k >= X::H || (!X::WHOLE && p >= pairs)) continue;
        const float2 A = va[i], B = vb[i];
        float2 *row = buf + p * row_pitch(N);
        if (k == 0 || 2 * k == N) {
            // DC and Nyquist of a real row are real
            row[row_at(k)] = make_float2(A.x, B.x);
        } else {
            row[row_at(k)] = make_float2(A.x - B.y, A.y + B.x);
            row[row_at(N - k)] = make_float2(A.x + B.y, B.x - A.y);
        }
    }
    __syncthreads();
    auto lload = [](int p, int x) { return buf[p * row_pitch(N) + row_at(x)]; };
    auto gstore = [=](int p, int x, float2 v) {
        if (!X::WHOLE && p >= pairs) return;
        out[p * (2 * N) + x] = v.x;
        out[p * (2 * N) + N + x] = v.y;
    };
    using C = Tile<N, true, false, true, P, T, true, false, 0, Plan::p.nst>;
    fft_steps<C, 0>(buf, tw, tid, lload, gstore);
}

// ---------------------------------------------------------------------------
// mean density and overall scale
// ---------------------------------------------------------------------------
// By one workgroup of T threads, from the x pass's partial masses.
template <int T>
__device__ void mean_scale(const JobView &jv, int64_t nparts, int n, uint32_t *status) {
    __shared__ unsigned long long red_lo[T / 64], red_hi[T / 64];
    const Mass128 *__restrict__ mass = jv.mass;
    unsigned long long lo = 0, hi = 0;
    constexpr int U = 8;  // partial sums in flight per thread
    for (int64_t i0 = threadIdx.x; i0 < nparts; i0 += T * U) {
        Mass128 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = i0 + u * T < nparts ? mass[i0 + u * T] : Mass128{0ull, 0ull};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            add128(lo, hi, v[u].lo);
            hi += v[u].hi;
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        unsigned long long olo = __shfl_down(lo, off, 64);
        unsigned long long ohi = __shfl_down(hi, off, 64);
        add128(lo, hi, olo);
        hi += ohi;
    }
    if ((threadIdx.x & 63) == 0) {
        red_lo[threadIdx.x >> 6] = lo;
        red_hi[threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long a = 0, b = 0;
        for (int w = 0; w < T / 64; ++w) {
            add128(a, b, red_lo[w]);
            b += red_hi[w];
        }
        const double total = u128_to_double(a, b);
        const double cells = double(n) * double(n) * double(n);
        const double mbar = total / cells;  // mean cell mass, FP64
        if (!(mbar > 0.0)) {
            atomicOr(status, ST_INPUT);
            jv.scalars[0] = 0.0;
        } else {
            // C = IDFT(DFT(rho) M) / (mbar n^3): the mean normalisation and the
            // inverse-transform 1/n^3 folded into one factor
            jv.scalars[0] = 1.0 / (mbar * cells);
        }
        jv.scalars[1] = mbar;
    }
}

// ---------------------------------------------------------------------------
// y and z passes on tiles of YZ_TILE columns of the half spectrum
// ---------------------------------------------------------------------------
constexpr int yz_threads(int n) { return threads_for(n * YZ_TILE); }

// Logical block (x, y, job) of an (X, Y, jobs) grid, XCD-contiguous over the
// whole launch: x = column tile, y = row in the y pass; x = row, y = column
// tile in the z pass.
template <int X, int Y>
__device__ __forceinline__ void yz_tile(int &x, int &y, int &job) {
    const uint32_t lt = xcd_remap(blockIdx.x + X * (blockIdx.y + Y * blockIdx.z), X * Y * gridDim.z);
    x = int(lt % X);
    y = int((lt / X) % Y);
    job = int(lt / (X * Y));
}

// 4 bytes read and 4 written per cell, bound by HBM: 1024^3 1890 -> 1807 us forward
// and 1854 -> 1730 inverse (4.8 and 5.0 TB/s), 768^3 710 inverse (5.1), 432^3 141
// -> 107, 256^3 31.5 -> 26.
template <int N, bool INV>
__device__ __forceinline__ void y_pass(const JobView &jv, int tile, int zrow, float2 *tw, float2 *buf) {
    constexpr int T = yz_threads(N);
    using C = Tile<N, INV, false, false, YZ_TILE, T, false, false, 0, PlanOf<N, false>::p.nst>;
    const int valid = min(YZ_TILE, N / 2 + 1 - tile * YZ_TILE);
    float2 *__restrict__ col = jv.spec + spec_at<N>(tile, zrow, 0);  // element y of pencil p at col[y YZ_TILE + p]
    load_twiddles<N, T, false>(tw, jv.tw);                // read after a barrier of the first step
    auto gload = [=](int p, int y) { return p < valid ? col[y * YZ_TILE + p] : make_float2(0.f, 0.f); };
    auto gstore = [=](int p, int y, float2 v) {
        if (p < valid) col[y * YZ_TILE + p] = v;
    };
    fft_steps<C, 0>(buf, tw, threadIdx.x, gload, gstore);
}

// The workgroup of a job's first tile also forms the mean: its partial sums are
// ready (the x pass's launch is over), and the z pass needs it.
template <int N>
__global__ void __launch_bounds__(yz_threads(N)) fft_y_fwd_kernel(CwtJobs J, CwtLayout L, uint32_t *status) {
    __shared__ float2 tw[N], buf[N * YZ_TILE];
    int tile, zrow, job;
    yz_tile<spec_tiles(N), N>(tile, zrow, job);
    const JobView jv = job_view(J, L, job);
    if (tile == 0 && zrow == 0) mean_scale<yz_threads(N)>(jv, x_blocks(N, x_fwd_log_pairs(N)), N, status);
    y_pass<N, false>(jv, tile, zrow, tw, buf);
}

template <int N>
__global__ void __launch_bounds__(yz_threads(N)) fft_y_inv_kernel(CwtJobs J, CwtLayout L) {
    __shared__ float2 tw[N], buf[N * YZ_TILE];
    int tile, zrow, job;
    yz_tile<spec_tiles(N), N>(tile, zrow, job);
    y_pass<N, true>(job_view(J, L, job), tile, zrow, tw, buf);
}

// Forward z transform, multiplier, inverse z transform (the rotated plan).
// The z pass walks its tiles ky-fastest (grid (n, tiles, jobs)): the tiles of
// rows ky and ky + 1 read the two halves of the same 128-byte lines, so they
// run together on one XCD and each line comes from HBM once.  The y pass's bytes,
// with twice its LDS traffic and in 64-byte runs: 1024^3 2585 -> 2183 us (3.9
// TB/s), 512^3 (three scales) 1006 -> 763, 432^3 259 -> 168, 256^3 44 -> 29.
template <int N>
__global__ void __launch_bounds__(yz_threads(N)) fft_z_mul_kernel(CwtJobs J, CwtLayout L) {
    constexpr int T = yz_threads(N), H = N / 2 + 1, ZS = (N + 1) * YZ_TILE;
    using Plan = PlanOf<N, false>;
    __shared__ float2 tw[N], buf[N * YZ_TILE];
    int tile, ky, job;
    yz_tile<N, spec_tiles(N)>(ky, tile, job);
    job += J.job_base;
    const JobView jv = job_view(J, L, job);
    const JobView src = J.shared_forward ? job_view(J, L, 0) : jv;  // forward spectrum and normalisation
    const float *__restrict__ tab_b = jv.btab;
    const float *__restrict__ tab_p = jv.ptab;
    const int tid = threadIdx.x;
    const int kx0 = tile * YZ_TILE;
    const int valid = min(YZ_TILE, H - kx0);
    // element z of pencil p at col[z ZS + p]; col_in is the same place, or job 0's
    float2 *col = jv.spec + spec_at<N>(tile, 0, ky);
    const float2 *col_in = src.spec + spec_at<N>(tile, 0, ky);
    load_twiddles<N, T, false>(tw, jv.tw);
    const float scale = float(src.scalars[0]);
    const float by = tab_b[ky], py = tab_p[ky];
    // the thread's pencil is the same in every stage (T is a multiple of YZ_TILE)
    const int kx = min(kx0 + (tid & (YZ_TILE - 1)), H - 1);
    const float bx = tab_b[kx], px = tab_p[kx];
    const float cxy = (px * by + bx * py) * scale, bxy = bx * by * scale;
    auto gload = [=](int p, int z) { return p < valid ? col_in[z * ZS + p] : make_float2(0.f, 0.f); };
    auto gstore = [=](int p, int z, float2 v) {
        if (p < valid) col[z * ZS + p] = v;
    };
    auto mul = [=](int, int kz) { return cxy * tab_b[kz] + bxy * tab_p[kz]; };
    auto lload = [](int p, int x) { return buf[(x << YZ_LOG) + p]; };
    auto lstore = [](int p, int x, float2 v) { buf[(x << YZ_LOG) + p] = v; };
    constexpr int last = Plan::p.nst - 1, R = Plan::radix(last);
    using Seam = Tile<N, false, false, false, YZ_TILE, T, true, true, 0, 1>;
    if constexpr (last == 0) {
        fft_seam<Seam, R, false>(tw, tid, gload, gstore, mul);
    } else {
        using F = Tile<N, false, false, false, YZ_TILE, T, false, true, 0, last>;
        using I = Tile<N, true, true, false, YZ_TILE, T, true, false, 1, last + 1>;
        fft_steps<F, 0>(buf, tw, tid, gload, lstore);
        __syncthreads();
        fft_seam<Seam, R, true>(tw, tid, lload, lstore, mul);
        __syncthreads();
        fft_steps<I, 1>(buf, tw, tid, lload, gstore);
    }
}

}  // namespace

template <int N>
hf_status hf::run_cwt_n(hf_ctx *ctx, const CwtJobs &J, const CwtLayout &L) {
    hipStream_t st = ctx->stream;
    const unsigned jobs = unsigned(J.count), fwd_jobs = J.shared_forward ? 1u : jobs;
    constexpr unsigned tiles = unsigned(spec_tiles(N)), yz = unsigned(yz_threads(N));
    using XF = XTile<N, x_fwd_log_pairs(N)>;
    using XI = XTile<N, x_inv_log_pairs(N)>;
    constexpr unsigned fblocks = unsigned(x_blocks(N, x_fwd_log_pairs(N))),
                       iblocks = unsigned(x_blocks(N, x_inv_log_pairs(N)));
    HF_LAUNCH(ctx, K_X_FWD, fft_x_fwd_kernel<N>, dim3(fblocks, fwd_jobs), dim3(XF::T), 0, st, J, L, ctx->d_status);
    HF_LAUNCH(ctx, K_Y_FWD, fft_y_fwd_kernel<N>, dim3(tiles, N, fwd_jobs), dim3(yz), 0, st, J, L, ctx->d_status);
    if (J.shared_forward && jobs > 1) {
        // the other scales read job 0's forward spectrum before job 0 overwrites it
        CwtJobs Jr = J;
        Jr.job_base = 1;
        HF_LAUNCH(ctx, K_Z_MUL, fft_z_mul_kernel<N>, dim3(N, tiles, jobs - 1), dim3(yz), 0, st, Jr, L);
        HF_LAUNCH(ctx, K_Z_MUL, fft_z_mul_kernel<N>, dim3(N, tiles, 1), dim3(yz), 0, st, J, L);
    } else {
        HF_LAUNCH(ctx, K_Z_MUL, fft_z_mul_kernel<N>, dim3(N, tiles, jobs), dim3(yz), 0, st, J, L);
    }
    HF_LAUNCH(ctx, K_Y_INV, fft_y_inv_kernel<N>, dim3(tiles, N, jobs), dim3(yz), 0, st, J, L);
    HF_LAUNCH(ctx, K_X_INV, fft_x_inv_kernel<N>, dim3(iblocks, jobs), dim3(XI::T), 0, st, J, L);
    return launch_status();
}
