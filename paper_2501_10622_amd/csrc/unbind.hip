// Steps 9-10 (Sec. 2.3): the self-boundness check of the groups one scale
// keeps.  For each group, repeatedly: the centre of mass of its remaining
// particles (equal masses) and their mean velocity; every particle's radius;
// the spherical shell potential at each particle,
//   Phi_i = -G m [ (members at or inside (r_i, id_i)) / r_i + sum over the
//                  members outside of 1 / r_j ],
// and the particles whose speed relative to the mean exceeds the local escape
// speed sqrt(-2 Phi_i) leave; until none leaves.  A group that lost more than
// 40% of its particles (5 removed > 2 N), or keeps fewer than particle_th, is
// discarded.  Afterwards only the bound particles of the groups that pass keep
// their labels.
//
// Layout of the work: the members of every kept group are gathered into
// contiguous runs (counts, an exclusive scan, then one slot per member by an
// atomic cursor).  A team checks each group: a whole workgroup of 16 wavefronts
// the groups of more than UB_WAVE_CAP members, a single wavefront the others.
// The team sorts its run by particle index, so the member order -- and with it
// every floating-point sum -- does not depend on the order the atomics resolved
// in.  It then iterates the rounds: FP64 reductions for the centre and mean
// velocity, each member's radius and speed, then the remaining members sorted
// by (radius, member position) -- chunks of UB_CHUNK sorted in LDS, then merged
// pairwise in global memory -- so that a member's inner count is its sorted
// position plus one and its outer sum a suffix sum of 1 / r over the sorted
// order, formed block by block from the outermost inward (O(N log N) per
// round).  Member positions follow particle indices, so equal radii are ordered
// by particle index, the order the definition uses.
//
// Nothing here streams: what bounds a group is the chain of its rounds' short
// loops (dependent loads, LDS passes of the sorts), and what bounds the launch is
// the largest groups' chains, since most groups have a few hundred members and
// a few have ten thousand.  So a large group gets a whole CU (16 wavefronts, 153
// KB of LDS) and the largest ones start first, while a small group gets one
// wavefront, whose sorts and sums need no barrier.  Both sorts go by bins (a
// histogram, a scan, and a count of the smaller ones in a member's own bin:
// a few operations per member) instead of a bitonic network's log^2.  The
// members' positions and velocities are put into group order by the gather, where
// they stream by; fetched from the input arrays they cost two lines per member in
// each of a round's two passes.  On a 256^3 phase-space box (373, 2668 and 15,841
// groups on grids of 270, 345 and 470; 1.5, 3.5 and 5.3 million members, the
// largest 15,375) the checks took 4.4, 3.9 and 3.2 ms with 256 threads per group
// and bitonic sorts, and take 0.48, 1.00 and 0.96 ms (1.46, 2.26 and 2.25 ms
// before the bin sorts, 1.49, 1.58 and 1.48 ms before the records).
#include <cmath>
#include <type_traits>

#include "hf_internal.h"
#include "scan.h"

using namespace hf;

namespace {

constexpr int UB_THREADS = 256;          // of the streaming passes
constexpr int UB_WAVES = 16;             // wavefronts of a group workgroup
constexpr int UB_TEAM = 64 * UB_WAVES;
constexpr int UB_PER = 10;               // members per thread that the LDS holds
constexpr int UB_BPER = 8;               // sort bins per thread
constexpr int UB_CHUNK = UB_TEAM * UB_PER;  // members a workgroup sorts by radius in LDS
constexpr int UB_WAVE_CAP = 64 * UB_PER;    // and a wavefront, in its share
constexpr uint32_t UB_WAVE_MOST = 640;   // members of the largest group that one wavefront checks
constexpr uint32_t UB_BIN_MOST = 48;     // fullest bin of a bin sort; else the bitonic one
constexpr uint32_t UB_HUGE = 4096;       // groups above this are checked first
constexpr int UB_BATCH = 4;              // members per thread whose loads are issued together
constexpr int SCAN_GROUPS = 2;           // scan tag of this use

// Counters of the group lists: lengths of the huge, middle and small lists,
// then the takes from the first two together and from the third.
enum { Q_HUGE, Q_MID, Q_SMALL, Q_TAKE_BIG, Q_TAKE_SMALL, Q_COUNT };

struct UnbindLayout {
    size_t slot, cnt, start, cursor, partial, queue, pid, rad, ord, tmp, spd, alive, total;
    size_t perm, rec, full;  // with the members' records, where the workspace has room for them
};

UnbindLayout unbind_layout(int n, int64_t np, int64_t nroots) {
    UnbindLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes);
        return at;
    };
    L.slot = take(sizeof(uint32_t) * size_t(n) * size_t(n) * size_t(n));
    L.cnt = take(sizeof(uint32_t) * size_t(nroots > 0 ? nroots : 1));
    L.start = take(sizeof(uint32_t) * size_t(nroots + 1));
    L.cursor = take(sizeof(uint32_t) * size_t(nroots > 0 ? nroots : 1));
    L.partial = take(sizeof(uint64_t) * SCAN_MAX_GROUPS);
    L.queue = take(Q_COUNT * sizeof(uint32_t));
    L.pid = take(sizeof(int32_t) * size_t(np > 0 ? np : 1));
    L.rad = take(sizeof(double) * size_t(np > 0 ? np : 1));
    L.ord = take(sizeof(uint32_t) * size_t(np > 0 ? np : 1));
    L.tmp = take(sizeof(uint32_t) * size_t(np > 0 ? np : 1));
    L.spd = take(sizeof(double) * size_t(np > 0 ? np : 1));
    L.alive = take(sizeof(uint8_t) * size_t(np > 0 ? np : 1));
    L.total = off;
    L.perm = take(sizeof(uint32_t) * size_t(np > 0 ? np : 1));
    L.rec = take(6 * sizeof(double) * size_t(np > 0 ? np : 1));
    L.full = off;
    return L;
}

// Number of roots: min(*d_count, cap) when the count is on the device, else cap.
__device__ __forceinline__ int64_t ub_roots(const int64_t *d_count, int64_t cap) {
    if (!d_count) return cap;
    const int64_t c = *d_count;
    return c < cap ? c : cap;
}

unsigned ub_grid(const hf_ctx *ctx, int64_t work) {
    const int64_t want = (work + UB_THREADS - 1) / UB_THREADS;
    const int64_t cap = int64_t(ctx->cus) * 32;
    return unsigned(want < 1 ? 1 : (want > cap ? cap : want));
}

// slot[root_i] = i and cursor[i] = 0 for every root; cnt[i] = 0, or, where the
// members have been counted already, the parts of a group whose keep flag is set
// (the counters of the cells, GroupCounters); the group lists' counters to 0.
__global__ void __launch_bounds__(UB_THREADS) ub_slots_kernel(const int32_t *__restrict__ roots,
                                                              const int64_t *d_count, int64_t cap, int64_t ncells,
                                                              const uint32_t *__restrict__ parts,
                                                              const uint32_t *__restrict__ kept,
                                                              uint32_t *__restrict__ slot, uint32_t *__restrict__ cnt,
                                                              uint32_t *__restrict__ cur, uint32_t *__restrict__ queue,
                                                              uint32_t *status) {
    const int64_t nroots = ub_roots(d_count, cap);
    if (blockIdx.x == 0 && threadIdx.x < Q_COUNT) queue[threadIdx.x] = 0u;
    bool bad = false;
    for (int64_t i = blockIdx.x * int64_t(UB_THREADS) + threadIdx.x; i < nroots;
         i += int64_t(gridDim.x) * UB_THREADS) {
        cur[i] = 0u;
        const int32_t r = roots[i];
        if (r < 0 || r >= ncells) {
            cnt[i] = 0u;
            bad = true;
            continue;
        }
        cnt[i] = parts && kept[r] ? parts[r] : 0u;
        slot[r] = uint32_t(i);
    }
    if (bad) atomicOr(status, ST_INPUT);
}

// The group of a label, or -1: a label must be one of the roots (else it is
// reported and dropped), and its group must be kept (else dropped).
__device__ __forceinline__ int64_t group_of(int32_t l, const int32_t *__restrict__ roots, int64_t nroots,
                                            int64_t ncells, const uint32_t *__restrict__ slot,
                                            const uint8_t *__restrict__ keep, bool &bad) {
    if (l < 0) return -1;
    if (l >= ncells) {
        bad = true;
        return -1;
    }
    const uint32_t i = slot[l];
    if (int64_t(i) >= nroots || roots[i] != l) {
        bad = true;
        return -1;
    }
    return keep[i] ? int64_t(i) : -1;
}

// Members per kept group; labels outside a kept group become -1.
__global__ void __launch_bounds__(UB_THREADS) ub_count_kernel(int32_t *__restrict__ label, int64_t np,
                                                              const int32_t *__restrict__ roots,
                                                              const int64_t *d_count, int64_t cap, int64_t ncells,
                                                              const uint32_t *__restrict__ slot,
                                                              const uint8_t *__restrict__ keep,
                                                              uint32_t *__restrict__ cnt, uint32_t *status) {
    const int64_t nroots = ub_roots(d_count, cap);
    bool bad = false;
    for (int64_t p = blockIdx.x * int64_t(UB_THREADS) + threadIdx.x; p < np; p += int64_t(gridDim.x) * UB_THREADS) {
        const int32_t l = label[p];
        if (l < 0) continue;
        const int64_t g = group_of(l, roots, nroots, ncells, slot, keep, bad);
        if (g < 0) label[p] = -1;
        else atomicAdd(cnt + g, 1u);
    }
    if (bad) atomicOr(status, ST_INPUT);
}

// One slot per member in its group's run (in the order the cursors give).  Where
// the members have been counted before (guard), labels come as the loop over scales
// left them: a listed root's only if its group is kept, but also those of roots past
// the end of a list that is too short for its maxima, which have no slot, and are
// reported and dropped, as ub_count_kernel does where it runs (the lookups and the
// run's end: 1.04 -> 1.20 ms for the three scales above).  With rec, the member's
// position and velocity are put into the slot too (6 values): here they stream by in
// input order, while the check would fetch two lines from all over the arrays for
// every member and pass over them.
template <typename T>
__global__ void __launch_bounds__(UB_THREADS) ub_gather_kernel(int32_t *__restrict__ label, int64_t np, bool guard,
                                                               const int32_t *__restrict__ roots,
                                                               const int64_t *d_count, int64_t cap, int64_t ncells,
                                                               const uint32_t *__restrict__ slot,
                                                               const uint32_t *__restrict__ start,
                                                               uint32_t *__restrict__ cur, int32_t *__restrict__ pid,
                                                               const T *__restrict__ pos, const T *__restrict__ vel,
                                                               T *__restrict__ rec, uint32_t *status) {
    const int64_t nroots = ub_roots(d_count, cap);
    bool bad = false;
    for (int64_t p = blockIdx.x * int64_t(UB_THREADS) + threadIdx.x; p < np; p += int64_t(gridDim.x) * UB_THREADS) {
        const int32_t l = label[p];
        if (l < 0) continue;
        const uint32_t g = l < ncells ? slot[l] : 0xffffffffu;
        if (guard && (int64_t(g) >= nroots || roots[g] != l)) {
            label[p] = -1;
            bad = true;
            continue;
        }
        T v[6];
        if (rec) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                v[a] = pos[3 * p + a];
                v[3 + a] = vel[3 * p + a];
            }
        }
        const int64_t k = int64_t(start[g]) + atomicAdd(cur + g, 1u);
        if (guard && k >= int64_t(start[g + 1])) {  // more members than were counted: the run is full
            label[p] = -1;
            bad = true;
            continue;
        }
        pid[k] = int32_t(p);
        if (rec) {
#pragma unroll
            for (int a = 0; a < 6; ++a) rec[6 * k + a] = v[a];
        }
    }
    if (bad) atomicOr(status, ST_INPUT);
}

// The kept groups by size: the huge ones at the front of `big`, the middle ones
// at its back, the small ones in `small` (no order within a list, none is
// needed); bound_keep of the others, and of those without a member, is 0.  A
// workgroup gathers the groups of UB_LIST roots in LDS and reserves their places
// once per list: one counter atomic per group took 158 us for the 15,841 groups of
// 2.5 million roots.
constexpr int UB_LIST = 8 * UB_THREADS;

__global__ void __launch_bounds__(UB_THREADS) ub_list_kernel(const int64_t *d_count, int64_t cap,
                                                             const uint8_t *__restrict__ keep,
                                                             const uint32_t *__restrict__ start,
                                                             uint32_t *__restrict__ big, uint32_t *__restrict__ small,
                                                             uint32_t *__restrict__ queue,
                                                             uint8_t *__restrict__ bound_keep) {
    __shared__ uint32_t n[3], first[3];
    const int64_t nroots = ub_roots(d_count, cap);
    for (int64_t g0 = int64_t(blockIdx.x) * UB_LIST; g0 < nroots; g0 += int64_t(gridDim.x) * UB_LIST) {
        if (threadIdx.x < 3) n[threadIdx.x] = 0u;
        __syncthreads();
        int list[UB_LIST / UB_THREADS];
        uint32_t at[UB_LIST / UB_THREADS];
#pragma unroll
        for (int u = 0; u < UB_LIST / UB_THREADS; ++u) {
            const int64_t g = g0 + u * UB_THREADS + threadIdx.x;
            list[u] = -1;
            if (g >= nroots) continue;
            const uint32_t m = start[g + 1] - start[g];
            if (!keep[g] || m == 0u) {
                bound_keep[g] = 0;
                continue;
            }
            list[u] = m > UB_HUGE ? Q_HUGE : (m > UB_WAVE_MOST ? Q_MID : Q_SMALL);
            at[u] = atomicAdd(&n[list[u]], 1u);
        }
        __syncthreads();
        if (threadIdx.x < 3 && n[threadIdx.x]) first[threadIdx.x] = atomicAdd(queue + threadIdx.x, n[threadIdx.x]);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < UB_LIST / UB_THREADS; ++u) {
            if (list[u] < 0) continue;
            const uint32_t g = uint32_t(g0 + u * UB_THREADS + threadIdx.x), k = first[list[u]] + at[u];
            if (list[u] == Q_HUGE) big[k] = g;
            else if (list[u] == Q_MID) big[cap - 1 - int64_t(k)] = g;
            else small[k] = g;
        }
        __syncthreads();  // n and first are read before the next sweep clears them
    }
}

// A value that every lane of the wavefront holds alike, told to the compiler
// (it then keeps the group's sizes and pointers in scalar registers).
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// A team of W wavefronts: one, or the whole workgroup.  sync() orders the
// team's accesses to LDS and to global memory (one wavefront needs no barrier,
// only its accesses completed and not moved by the compiler); lane_sync() does
// so for LDS within each wavefront.
__device__ __forceinline__ void lane_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int W>
struct Team {
    static constexpr int N = 64 * W;
    static __device__ __forceinline__ int tid() { return W == 1 ? int(threadIdx.x & 63) : int(threadIdx.x); }
    static __device__ __forceinline__ int wave() { return W == 1 ? 0 : int(threadIdx.x >> 6); }
    static __device__ __forceinline__ void sync() {
        if constexpr (W == 1) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        } else {
            __syncthreads();
        }
    }
};

// A team's share of the LDS.
struct TeamLds {
    double *key;      // [64 W UB_PER]
    uint32_t *idx;    // [64 W UB_PER], right after key
    uint32_t *bins;   // [64 W UB_BPER]
    double *red;      // [6 W]
    uint32_t *count;  // [1 + W]
};

// Whether pred holds for any thread of the team (a sync as well).
template <int W>
__device__ __forceinline__ bool team_any(bool pred) {
    if constexpr (W == 1) {
        Team<1>::sync();
        return __any(pred);
    } else {
        return __syncthreads_or(pred);
    }
}

// The team's smallest lo and largest hi.
template <int W>
__device__ __forceinline__ void team_range(uint32_t &lo, uint32_t &hi, const TeamLds &lds) {
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t a = __shfl_xor(lo, off, 64), b = __shfl_xor(hi, off, 64);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    if constexpr (W > 1) {
        uint32_t *r = reinterpret_cast<uint32_t *>(lds.red);
        if ((threadIdx.x & 63) == 0) {
            r[2 * Team<W>::wave()] = lo;
            r[2 * Team<W>::wave() + 1] = hi;
        }
        Team<W>::sync();
        const int w = int(threadIdx.x) % W;
        lo = r[2 * w];
        hi = r[2 * w + 1];
        for (int off = W / 2; off > 0; off >>= 1) {
            const uint32_t a = __shfl_xor(lo, off, 64), b = __shfl_xor(hi, off, 64);
            lo = a < lo ? a : lo;
            hi = b > hi ? b : hi;
        }
        Team<W>::sync();
    }
}

// Bins of equal width over the values lo .. hi, the last taking what lies above.
template <int W>
struct BinMap {
    static constexpr uint32_t BINS = 64 * W * UB_BPER;
    uint32_t lo;
    uint64_t mult;
    __device__ __forceinline__ BinMap(uint32_t l, uint32_t h)
        : lo(l), mult((uint64_t(BINS) << 32) / (uint64_t(h - l) + 1)) {}
    __device__ __forceinline__ uint32_t operator()(uint32_t v) const {
        const uint64_t b = v <= lo ? 0 : (uint64_t(v - lo) * mult) >> 32;
        return b < BINS ? uint32_t(b) : BINS - 1;
    }
};

// Counts in bins[] -> where each bin starts; false (for the whole team) if a
// bin holds more than UB_BIN_MOST.  The counts are complete on entry (synced).
template <int W>
__device__ __forceinline__ bool team_bin_starts(const TeamLds &lds) {
    using Tm = Team<W>;
    const int lane = threadIdx.x & 63;
    uint32_t *mine = lds.bins + Tm::tid() * UB_BPER;
    uint32_t c[UB_BPER], sum = 0, most = 0;
#pragma unroll
    for (int k = 0; k < UB_BPER; ++k) {
        c[k] = mine[k];
        sum += c[k];
        most = c[k] > most ? c[k] : most;
    }
    uint32_t inc = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(inc, off, 64);
        if (lane >= off) inc += y;
    }
    uint32_t at = inc - sum;
    if constexpr (W > 1) {
        if (lane == 63) lds.count[1 + Tm::wave()] = inc;
    }
    const bool full = team_any<W>(most > UB_BIN_MOST);
    if constexpr (W > 1) {
#pragma unroll 4
        for (int w = 0; w < W; ++w) at += w < Tm::wave() ? lds.count[1 + w] : 0u;
    }
#pragma unroll
    for (int k = 0; k < UB_BPER; ++k) {
        mine[k] = at;
        at += c[k];
    }
    Tm::sync();
    return !full;
}

// A bin sort places more members than the LDS holds in segments of whole bins:
// the bins [b0, b1] from `bin` on that start at places [first, first + room).
// The next segment starts with bin b1 + 1, where bin b1 ends.  (A bin holds at most UB_BIN_MOST, so a
// segment's members fit room + UB_BIN_MOST places.)
struct BinSegment {
    uint32_t b0, b1;
};

template <int W>
__device__ __forceinline__ BinSegment team_segment(const TeamLds &lds, uint32_t bin, uint32_t first,
                                                   uint32_t room) {
    BinSegment s{0xffffffffu, 0u};
    for (int k = 0; k < UB_BPER; ++k) {
        const uint32_t b = Team<W>::tid() * UB_BPER + k, at = lds.bins[b];
        if (b < bin || at - first >= room) continue;
        s.b0 = b < s.b0 ? b : s.b0;
        s.b1 = b > s.b1 ? b : s.b1;
    }
    team_range<W>(s.b0, s.b1, lds);
    Team<W>::sync();
    return s;
}

// Bitonic sort of the places [0, m) held in LDS, through cswap(lo, hi), which
// puts the smaller of two places' values at lo (hi >= m stands for +infinity:
// nothing moves): the all-ascending form (each merge first compares an element
// with its mirror in the block, then half-cleaners) over the next power of
// two.  Each wavefront takes a contiguous share of the comparators, so that
// the steps whose blocks lie within one share need no barrier (of the 91 steps
// for 8192 places 81 do not).
template <int W, class Swap>
__device__ __forceinline__ void team_bitonic(int m, Swap &&cswap) {
    using Tm = Team<W>;
    int p2 = 128;
    while (p2 < m) p2 <<= 1;
    const int share = p2 / 2 / W > 64 ? p2 / 2 / W : 64;  // comparators per wavefront
    const int local = 2 * share;                          // places of a share
    const int t0 = Tm::wave() * share + int(threadIdx.x & 63);
    const int t1 = Tm::wave() * share + share < p2 / 2 ? Tm::wave() * share + share : p2 / 2;
    auto step_done = [&](int span, int next) {
        if (W > 1 && (span > local || next > local)) __syncthreads();
        else lane_sync();
    };
    for (int size = 2; size <= p2; size <<= 1) {
        const int half = size >> 1;
        for (int t = t0; t < t1; t += 64) {
            const int q = t & (half - 1), b = (t - q) * 2;
            if (b + size - 1 - q < m) cswap(b + q, b + size - 1 - q);
        }
        step_done(size, half > 1 ? half : 2 * size);
        for (int stride = half >> 1; stride > 0; stride >>= 1) {
            for (int t = t0; t < t1; t += 64) {
                const int lo = 2 * t - (t & (stride - 1));
                if (lo + stride < m) cswap(lo, lo + stride);
            }
            step_done(2 * stride, stride > 1 ? stride : 2 * size);
        }
    }
    Tm::sync();
}

// Sorts the distinct particle indices a[0..m) ascending by bins: the indices
// spread evenly over their range, so a bin of the range's 1 / BINS holds a few,
// and an index's place is its bin's start plus the smaller ones in its bin.
// With a bin above UB_BIN_MOST, by the bitonic network in LDS, or, past its
// room, in place in global memory.  True if perm received where every index
// stood before (by bins only).  tmp: m words of scratch.
template <int W>
__device__ bool sort_members(int32_t *a, int m, uint32_t *perm, uint32_t *tmp, const TeamLds &lds) {
    using Tm = Team<W>;
    constexpr int ROOM = Tm::N * UB_PER;
    const int tid = Tm::tid();
    int32_t *s = reinterpret_cast<int32_t *>(lds.key);
    uint32_t lo = 0xffffffffu, hi = 0u;
    for (int k = 0; k < UB_BPER; ++k) lds.bins[k * Tm::N + tid] = 0u;
    for (int k = tid; k < m; k += Tm::N) {
        const uint32_t v = uint32_t(a[k]);
        lo = v < lo ? v : lo;
        hi = v > hi ? v : hi;
    }
    team_range<W>(lo, hi, lds);
    Tm::sync();
    const BinMap<W> bin(lo, hi);
    for (int k = tid; k < m; k += Tm::N) atomicAdd(&lds.bins[bin(uint32_t(a[k]))], 1u);
    Tm::sync();
    if (team_bin_starts<W>(lds)) {
        const bool one = m <= ROOM;
        int32_t *out = one ? a : reinterpret_cast<int32_t *>(tmp);
        for (uint32_t first = 0, next = 0; first < uint32_t(m);) {
            const BinSegment seg = one ? BinSegment{0u, BinMap<W>::BINS - 1}
                                       : team_segment<W>(lds, next, first, ROOM - UB_BIN_MOST);
            for (int k = tid; k < m; k += Tm::N) {
                const int32_t v = a[k];
                const uint32_t b = bin(uint32_t(v));
                if (b < seg.b0 || b > seg.b1) continue;
                const uint32_t at = atomicAdd(&lds.bins[b], 1u) - first;
                s[at] = v;
                lds.idx[at] = uint32_t(k);
            }
            Tm::sync();
            // the segment's bins[b] is now where bin b ends
            const uint32_t end = lds.bins[seg.b1];
            for (uint32_t t = tid; t < end - first; t += Tm::N) {
                const int32_t v = s[t];
                const uint32_t b = bin(uint32_t(v));
                const uint32_t from = b > seg.b0 ? lds.bins[b - 1] : first, to = lds.bins[b];
                uint32_t rank = from;
                for (uint32_t j = from; j < to; ++j) rank += s[j - first] < v ? 1u : 0u;
                out[rank] = v;
                if (perm) perm[rank] = lds.idx[t];
            }
            Tm::sync();
            first = uniform(end);
            next = uniform(seg.b1) + 1;
        }
        if (!one) {
            for (int k = tid; k < m; k += Tm::N) a[k] = out[k];
            Tm::sync();
        }
        return perm != nullptr;
    }
    constexpr int CAP = Tm::N * UB_PER * 3;  // the key and idx buffers together
    if (m <= CAP) {
        for (int k = Tm::tid(); k < m; k += Tm::N) s[k] = a[k];
        Tm::sync();
        team_bitonic<W>(m, [&](int lo, int hi) {
            const int32_t x = s[lo], y = s[hi];
            if (x > y) {
                s[lo] = y;
                s[hi] = x;
            }
        });
        for (int k = Tm::tid(); k < m; k += Tm::N) a[k] = s[k];
        Tm::sync();
        return false;
    }
    int p2 = 1;
    while (p2 < m) p2 <<= 1;
    auto cswap = [&](int lo, int hi) {
        if (hi >= m) return;
        const int32_t x = a[lo], y = a[hi];
        if (x > y) {
            a[lo] = y;
            a[hi] = x;
        }
    };
    for (int size = 2; size <= p2; size <<= 1) {
        const int half = size >> 1;
        for (int t = Tm::tid(); t < p2 / 2; t += Tm::N) {
            const int q = t % half, b = (t / half) * size;
            cswap(b + q, b + size - 1 - q);
        }
        Tm::sync();
        for (int stride = half >> 1; stride > 0; stride >>= 1) {
            for (int t = Tm::tid(); t < p2 / 2; t += Tm::N) {
                const int lo = 2 * t - (t & (stride - 1));
                cswap(lo, lo + stride);
            }
            Tm::sync();
        }
    }
    return false;
}

// Minimum-image offset of a coordinate from the group's reference point.
__device__ __forceinline__ double unwrap(double d, double box_len) {
    const double half = __dmul_rn(0.5, box_len);
    if (d >= half) return __dsub_rn(d, box_len);
    if (d < -half) return __dadd_rn(d, box_len);
    return d;
}

// (R[x], x) < (R[y], y): radius first, then member position.
__device__ __forceinline__ bool by_radius(const double *R, uint32_t x, uint32_t y) {
    const double a = R[x], b = R[y];
    return a < b || (a == b && x < y);
}

// One merge of sorted runs a[0..na) and b[0..nb) into out by the team: each
// thread finds where its share of the output starts on the merge path
// (a binary search), then merges its share in order.
template <int W>
__device__ void merge_runs(const uint32_t *a, int na, const uint32_t *b, int nb, uint32_t *out, const double *R) {
    const int total = na + nb;
    const int per = (total + Team<W>::N - 1) / Team<W>::N;
    const int o0 = Team<W>::tid() * per;
    if (o0 >= total) return;
    const int o1 = o0 + per < total ? o0 + per : total;
    int lo = o0 - nb > 0 ? o0 - nb : 0, hi = o0 < na ? o0 : na;
    while (lo < hi) {  // how many of the first o0 outputs come from a
        const int i = (lo + hi) >> 1;
        if (by_radius(R, a[i], b[o0 - i - 1])) lo = i + 1;
        else hi = i;
    }
    int i = lo, j = o0 - lo;
    for (int o = o0; o < o1; ++o) {
        const bool from_a = j >= nb || (i < na && by_radius(R, a[i], b[j]));
        out[o] = from_a ? a[i++] : b[j++];
    }
}

// Sorts the member positions ord[0..m) by (R, position) with the team: runs of
// the LDS's room there, then pairwise merges between ord and tmp.  Returns the array that holds the result.
template <int W>
__device__ uint32_t *sort_by_radius(const double *R, uint32_t *ord, uint32_t *tmp, int m, const TeamLds &lds) {
    using Tm = Team<W>;
    constexpr int CAP = W * 64 * UB_PER;
    double *skey = lds.key;
    uint32_t *sidx = lds.idx;
    for (int c0 = 0; c0 < m; c0 += CAP) {
        const int len = m - c0 < CAP ? m - c0 : CAP;
        for (int k = Tm::tid(); k < len; k += Tm::N) {
            const uint32_t x = ord[c0 + k];
            sidx[k] = x;
            skey[k] = R[x];
        }
        Tm::sync();
        team_bitonic<W>(len, [&](int lo, int hi) {
            const double a = skey[lo], b = skey[hi];
            const uint32_t x = sidx[lo], y = sidx[hi];
            if (b < a || (b == a && y < x)) {
                skey[lo] = b;
                skey[hi] = a;
                sidx[lo] = y;
                sidx[hi] = x;
            }
        });
        for (int k = Tm::tid(); k < len; k += Tm::N) ord[c0 + k] = sidx[k];
        Tm::sync();
    }
    uint32_t *src = ord, *dst = tmp;
    for (int w = CAP; w < m; w *= 2) {
        for (int a = 0; a < m; a += 2 * w) {
            const int na = m - a < w ? m - a : w;
            const int nb = m - a - na < w ? m - a - na : w;
            merge_runs<W>(src + a, na, src + a + na, nb, dst + a, R);
        }
        Tm::sync();
        uint32_t *t = src;
        src = dst;
        dst = t;
    }
    return src;
}

// The order of radii as unsigned integers: non-negative doubles order as their
// bits (a NaN counts as larger, so that the order is total).
__device__ __forceinline__ uint64_t radius_bits(double r) { return uint64_t(__double_as_longlong(r)); }

// Sorts the alive members k of [0, m0) by (R[k], k) by bins, as sort_members
// does, into key (radii) and idx (members) in LDS, or, where there are more than
// it holds, the members into ord: the bins are even in the bits of the radius
// as a float (nearly its logarithm) over the 16 octaves below the largest,
// where a halo's members spread over the bins to a few each.  lo and hi: the
// thread's smallest and largest such bits.  False (for the whole team, nothing
// sorted) if a bin is too full.
constexpr uint32_t UB_OCTAVES = 16u << 23;

template <int W>
__device__ bool bin_sort_radii(const double *R, const uint8_t *A, int m0, int m, uint32_t lo, uint32_t hi,
                               uint32_t *ord, const TeamLds &lds) {
    using Tm = Team<W>;
    constexpr int ROOM = Tm::N * UB_PER;
    const int tid = Tm::tid();
    for (int k = 0; k < UB_BPER; ++k) lds.bins[k * Tm::N + tid] = 0u;
    team_range<W>(lo, hi, lds);
    if (hi > UB_OCTAVES && lo < hi - UB_OCTAVES) lo = hi - UB_OCTAVES;
    const BinMap<W> of(lo, hi);
    auto bin = [&](double r) { return of(__float_as_uint(float(r))); };
    Tm::sync();
    // f(k, R[k]) for the alive members, UB_BATCH loads in flight
    auto alive = [&](auto &&f) {
        for (int k0 = tid; k0 < m0; k0 += UB_BATCH * Tm::N) {
            double r[UB_BATCH];
            bool on[UB_BATCH];
#pragma unroll
            for (int u = 0; u < UB_BATCH; ++u) {
                const int k = k0 + u * Tm::N < m0 ? k0 + u * Tm::N : 0;
                r[u] = R[k];
                on[u] = k0 + u * Tm::N < m0 && A[k] != 0;
            }
#pragma unroll
            for (int u = 0; u < UB_BATCH; ++u)
                if (on[u]) f(k0 + u * Tm::N, r[u]);
        }
    };
    alive([&](int, double r) { atomicAdd(&lds.bins[bin(r)], 1u); });
    Tm::sync();
    if (!team_bin_starts<W>(lds)) return false;
    const bool one = m <= ROOM;
    for (uint32_t first = 0, next = 0; first < uint32_t(m);) {
        const BinSegment seg = one ? BinSegment{0u, BinMap<W>::BINS - 1}
                                   : team_segment<W>(lds, next, first, ROOM - UB_BIN_MOST);
        alive([&](int k, double r) {
            const uint32_t b = bin(r);
            if (b < seg.b0 || b > seg.b1) return;
            const uint32_t at = atomicAdd(&lds.bins[b], 1u) - first;
            lds.key[at] = r;
            lds.idx[at] = uint32_t(k);
        });
        Tm::sync();
        // the segment's bins[b] is now where bin b ends; every member's place,
        // then all of them move
        const uint32_t end = lds.bins[seg.b1];
        double r[UB_PER];
        uint32_t x[UB_PER], place[UB_PER];
#pragma unroll
        for (int u = 0; u < UB_PER; ++u) {
            const uint32_t s = u * Tm::N + tid;
            place[u] = 0xffffffffu;
            if (s >= end - first) continue;
            r[u] = lds.key[s];
            x[u] = lds.idx[s];
            const uint32_t b = bin(r[u]);
            const uint32_t from = (b > seg.b0 ? lds.bins[b - 1] : first) - first, to = lds.bins[b] - first;
            const uint64_t q = radius_bits(r[u]);
            uint32_t rank = from;
            for (uint32_t t = from; t < to; ++t) {
                const uint64_t p = radius_bits(lds.key[t]);
                rank += p < q || (p == q && lds.idx[t] < x[u]) ? 1u : 0u;
            }
            place[u] = rank;
        }
        Tm::sync();
#pragma unroll
        for (int u = 0; u < UB_PER; ++u) {
            if (place[u] == 0xffffffffu) continue;
            if (one) {
                lds.key[place[u]] = r[u];
                lds.idx[place[u]] = x[u];
            } else {
                ord[first + place[u]] = x[u];
            }
        }
        Tm::sync();
        first = uniform(end);
        next = uniform(seg.b1) + 1;
    }
    return true;
}

// What the check of a group reads and writes.
template <typename T>
struct UnbindJob {
    const T *pos, *vel;
    int32_t *label;
    const int32_t *roots;
    const uint32_t *start;
    int32_t *pid;
    double *rad;
    uint32_t *ord, *tmp;
    double *spd;
    uint8_t *alive;
    uint32_t *perm;  // [np], and
    const T *rec;    // [np][6] the members' records, or both null
    int n;
    double box_len, gm;
    int64_t particle_th;
    uint8_t *bound_keep;
};

// The check of kept group g (steps 9-10) by one team: its members sorted by
// particle index, then the rounds, the decision and the labels.
template <int W, typename T>
__device__ void check_group(uint32_t g, const UnbindJob<T> &jb, const TeamLds &lds) {
    using Tm = Team<W>;
    constexpr int U = W == 1 ? UB_BATCH : 1;  // a workgroup has 16 wavefronts' loads in flight, and no registers to spare
    const int tid = Tm::tid(), lane = threadIdx.x & 63, wave = Tm::wave();
    g = uniform(g);
    const uint32_t s0 = uniform(jb.start[g]);
    const int m0 = int(uniform(jb.start[g + 1]) - s0);
    int32_t *P = jb.pid + s0;
    double *R = jb.rad + s0, *S = jb.spd + s0;
    uint32_t *ord = jb.ord + s0, *tmp = jb.tmp + s0;
    uint8_t *A = jb.alive + s0;
    const double box_len = jb.box_len;
    // member k's position and velocity: record from[k] of the group's run, or
    // (no records, or their order not kept) those of particle P[k]
    const bool recs = sort_members<W>(P, m0, jb.perm ? jb.perm + s0 : nullptr, ord, lds);
    const uint32_t *from = recs ? jb.perm + s0 : reinterpret_cast<const uint32_t *>(P);
    const T *__restrict__ pos = recs ? jb.rec + 6 * int64_t(s0) : jb.pos;
    const T *__restrict__ vel = recs ? pos + 3 : jb.vel;
    const uint32_t pitch = recs ? 6 : 3;
    const uint32_t un = uint32_t(jb.n), r0 = uniform(uint32_t(jb.roots[g]));
    const double dx = box_len / double(jb.n);
    const double ref[3] = {__dmul_rn(double(r0 % un), dx), __dmul_rn(double((r0 / un) % un), dx),
                           __dmul_rn(double(r0 / (un * un)), dx)};
    for (int k = tid; k < m0; k += Tm::N) A[k] = 1;
    Tm::sync();
    // positions and velocities of the members k0 + u N, and whether they are
    // still there; all loads issued before any is used
    struct Member {
        T p[3], v[3];
        bool on;
    };
    auto load_members = [&](int k0, Member (&mb)[U]) {
        int64_t at[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * Tm::N < m0 ? k0 + u * Tm::N : 0;
            mb[u].on = k0 + u * Tm::N < m0 && A[k] != 0;
            at[u] = int64_t(pitch) * from[k];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                mb[u].p[a] = pos[at[u] + a];
                mb[u].v[a] = vel[at[u] + a];
            }
        }
    };
    int m = m0;
    while (m > 0) {
        // centre of mass and mean velocity of the remaining members
        double sum[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int k0 = tid; k0 < m0; k0 += U * Tm::N) {
            Member mb[U];
            load_members(k0, mb);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!mb[u].on) continue;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    sum[a] = __dadd_rn(sum[a], unwrap(__dsub_rn(double(mb[u].p[a]), ref[a]), box_len));
                    sum[3 + a] = __dadd_rn(sum[3 + a], double(mb[u].v[a]));
                }
            }
        }
        double mean[6];
#pragma unroll
        for (int a = 0; a < 6; ++a)
            for (int off = 32; off > 0; off >>= 1) sum[a] = __dadd_rn(sum[a], __shfl_down(sum[a], off, 64));
        if constexpr (W == 1) {
#pragma unroll
            for (int a = 0; a < 6; ++a) mean[a] = __ddiv_rn(__shfl(sum[a], 0, 64), double(m));
        } else {
            if (lane == 0) {
#pragma unroll
                for (int a = 0; a < 6; ++a) lds.red[6 * wave + a] = sum[a];
            }
            Tm::sync();
#pragma unroll
            for (int a = 0; a < 6; ++a) mean[a] = 0.0;
#pragma unroll 1  // unrolled, the 6 W partial sums would all be live (and spill)
            for (int w = 0; w < W; ++w) {
#pragma unroll
                for (int a = 0; a < 6; ++a) mean[a] = __dadd_rn(mean[a], lds.red[6 * w + a]);
            }
#pragma unroll
            for (int a = 0; a < 6; ++a) mean[a] = __ddiv_rn(mean[a], double(m));
            Tm::sync();
        }
        // radius and speed^2 of every remaining member
        uint32_t lo = 0xffffffffu, hi = 0u;  // of the radii's float bits
        for (int k0 = tid; k0 < m0; k0 += U * Tm::N) {
            Member mb[U];
            load_members(k0, mb);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!mb[u].on) continue;
                double r2 = 0.0, s2 = 0.0;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const double e = __dsub_rn(unwrap(__dsub_rn(double(mb[u].p[a]), ref[a]), box_len), mean[a]);
                    const double w = __dsub_rn(double(mb[u].v[a]), mean[3 + a]);
                    r2 = __dadd_rn(r2, __dmul_rn(e, e));
                    s2 = __dadd_rn(s2, __dmul_rn(w, w));
                }
                const double r = __dsqrt_rn(r2);
                R[k0 + u * Tm::N] = r;
                S[k0 + u * Tm::N] = s2;
                const uint32_t f = __float_as_uint(float(r));
                lo = f < lo ? f : lo;
                hi = f > hi ? f : hi;
            }
        }
        Tm::sync();
        // the remaining members sorted by radius: in key and idx, or, where they
        // do not fit there or the bins do not do, as positions in srt
        const uint32_t *srt = m > Tm::N * UB_PER ? ord : nullptr;
        if (!bin_sort_radii<W>(R, A, m0, m, lo, hi, ord, lds)) {
            uint32_t base = 0;
            for (int k0 = 0; k0 < m0; k0 += Tm::N) {  // their positions, in order
                const bool on = k0 + tid < m0 && A[k0 + tid] != 0;
                const unsigned long long bits = __ballot(on);
                uint32_t before = base + uint32_t(__popcll(bits & ((1ull << lane) - 1ull)));
                if constexpr (W == 1) {
                    base += uint32_t(__popcll(bits));
                } else {
                    if (lane == 0) lds.count[1 + wave] = uint32_t(__popcll(bits));
                    Tm::sync();
#pragma unroll 4
                    for (int w = 0; w < W; ++w) {
                        const uint32_t c = lds.count[1 + w];
                        before += w < wave ? c : 0u;
                        base += c;
                    }
                    Tm::sync();
                }
                if (on) ord[before] = uint32_t(k0 + tid);
            }
            Tm::sync();
            srt = sort_by_radius<W>(R, ord, tmp, m, lds);
        }
        if (W > 1 && tid == 0) lds.count[0] = 0u;
        // the shell potential at each remaining member from its sorted position
        // p: (p + 1) / r inside, plus the suffix sum of 1 / r of the members
        // after it, formed block by block from the outermost inward; a leaver
        // is marked 2 (still counted this round)
        uint32_t leaving = 0;
        {
            double carry = 0.0;
            // member, radius and speed^2 at place p; the next block's are fetched
            // while a block is summed
            auto fetch = [&](int p, uint32_t &x, double &r, double &s) {
                const bool in = p >= 0 && p < m;
                x = in ? (srt ? srt[p] : lds.idx[p]) : 0u;
                r = in ? (srt ? R[x] : lds.key[p]) : 0.0;
                s = in ? S[x] : 0.0;
            };
            int b = ((m - 1) / Tm::N) * Tm::N;
            uint32_t xn;
            double rn, sn;
            fetch(b + tid, xn, rn, sn);
            for (; b >= 0; b -= Tm::N) {
                const int p = b + tid;
                const uint32_t x = xn;
                const double r = rn, s = sn;
                fetch(p - Tm::N, xn, rn, sn);
                const double v = p < m ? __ddiv_rn(1.0, r) : 0.0;  // inf at r = 0
                double incl = v;  // sum over this lane and the later lanes of the wavefront
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const double y = __shfl_down(incl, off, 64);
                    if (lane + off < 64) incl = __dadd_rn(incl, y);
                }
                const double after = __shfl_down(incl, 1, 64);
                double later = lane < 63 ? after : 0.0;
                double outer;
                if constexpr (W == 1) {
                    outer = __dadd_rn(later, carry);
                    carry = __dadd_rn(carry, __shfl(incl, 0, 64));
                } else {
                    if (lane == 0) lds.red[wave] = incl;
                    Tm::sync();
#pragma unroll 1
                    for (int w = wave + 1; w < W; ++w) later = __dadd_rn(later, lds.red[w]);
                    outer = __dadd_rn(later, carry);
#pragma unroll 4
                    for (int w = 0; w < W; ++w) carry = __dadd_rn(carry, lds.red[w]);
                    Tm::sync();
                }
                if (p < m) {
                    const double phi = -__dmul_rn(jb.gm, __dadd_rn(__ddiv_rn(double(p + 1), r), outer));
                    if (s > __dmul_rn(-2.0, phi)) {
                        A[x] = 2;
                        ++leaving;
                    }
                }
            }
        }
        uint32_t left;
        if constexpr (W == 1) {
            for (int off = 32; off > 0; off >>= 1) leaving += __shfl_xor(leaving, off, 64);
            left = leaving;
            Tm::sync();
        } else {
            if (leaving) atomicAdd(&lds.count[0], leaving);
            Tm::sync();
            left = lds.count[0];
        }
        if (left == 0) break;
        for (int k = tid; k < m0; k += Tm::N)
            if (A[k] == 2) A[k] = 0;
        m -= int(uniform(left));
        Tm::sync();
    }
    const int removed = m0 - m;
    const bool ok = m > 0 && 5LL * removed <= 2LL * m0 && int64_t(m) >= jb.particle_th;
    if (tid == 0) jb.bound_keep[g] = ok ? 1 : 0;
    for (int k = tid; k < m0; k += Tm::N)
        if (!ok || !A[k]) jb.label[P[k]] = -1;
    Tm::sync();  // the team's LDS is free for the next group
}

// Persistent, one workgroup per CU: first the workgroups take the huge and then
// the middle groups from their list, one at a time; when it is empty, each
// wavefront takes small groups for itself.  No more of either take than there may be
// groups for (a wavefront per small group beside those of the workgroups that big
// ones keep busy), and small groups go several to a take where there are many (eight
// takes per wavefront, then): a take from the one counter is 12 ns, 50 us for 4096
// wavefronts, which a launch with a few groups, or none, would last, and 7.6 ms for
// 650,000 groups of a member or two.
template <typename T>
__global__ void __launch_bounds__(UB_TEAM) ub_group_kernel(UnbindJob<T> jb, const uint32_t *__restrict__ big,
                                                           int64_t cap, const uint32_t *__restrict__ small,
                                                           uint32_t *queue) {
    __shared__ double sort_lds[UB_CHUNK * 3 / 2];  // radii (8 B), then member positions (4 B)
    __shared__ uint32_t bins[UB_TEAM * UB_BPER];
    __shared__ double red[6 * UB_WAVES];
    __shared__ uint32_t count[1 + UB_WAVES];
    __shared__ uint32_t s_next;
    static_assert(sizeof(sort_lds) + sizeof(bins) + sizeof(red) + sizeof(count) + sizeof(s_next) <= 160 * 1024,
                  "a CU's LDS");
    const uint32_t nhuge = queue[Q_HUGE], nbig = nhuge + queue[Q_MID], nsmall = queue[Q_SMALL];
    const TeamLds whole{sort_lds, reinterpret_cast<uint32_t *>(sort_lds + UB_CHUNK), bins, red, count};
    while (blockIdx.x < nbig) {
        if (threadIdx.x == 0) s_next = atomicAdd(queue + Q_TAKE_BIG, 1u);
        __syncthreads();
        const uint32_t k = s_next;
        __syncthreads();  // s_next is read before the next take
        if (k >= nbig) break;
        check_group<UB_WAVES>(k < nhuge ? big[k] : big[cap - 1 - int64_t(k - nhuge)], jb, whole);
    }
    const int wave = threadIdx.x >> 6;
    const uint32_t busy = nbig < gridDim.x ? nbig : gridDim.x;
    if (uint32_t(wave) * gridDim.x + blockIdx.x >= nsmall + UB_WAVES * busy) return;
    double *mine = sort_lds + wave * (UB_WAVE_CAP * 3 / 2);
    const TeamLds own{mine, reinterpret_cast<uint32_t *>(mine + UB_WAVE_CAP), bins + wave * 64 * UB_BPER, nullptr,
                      nullptr};
    const uint32_t share = nsmall / (8u * UB_WAVES * gridDim.x), batch = share < 1u ? 1u : (share < 64u ? share : 64u);
    for (;;) {
        uint32_t k = 0;
        if ((threadIdx.x & 63) == 0) k = atomicAdd(queue + Q_TAKE_SMALL, batch);
        k = uniform(__shfl(k, 0, 64));
        if (k >= nsmall) break;
        const uint32_t end = nsmall - k < batch ? nsmall : k + batch;
        for (; k < end; ++k) check_group<1>(small[k], jb, own);
    }
}

// The identification loop: particles this scale claimed whose label the check
// removed are free again.
__global__ void __launch_bounds__(UB_THREADS) ub_unclaim_kernel(const int32_t *__restrict__ label, int64_t np,
                                                                int32_t scale, int32_t *__restrict__ halo_scale,
                                                                int32_t *__restrict__ halo_root) {
    for (int64_t p = blockIdx.x * int64_t(UB_THREADS) + threadIdx.x; p < np; p += int64_t(gridDim.x) * UB_THREADS) {
        if (halo_scale[p] == scale && label[p] < 0) {
            halo_scale[p] = -1;
            halo_root[p] = -1;
        }
    }
}

__global__ void __launch_bounds__(UB_THREADS) ub_clear_kernel(int32_t *__restrict__ label, int64_t np) {
    for (int64_t p = blockIdx.x * int64_t(UB_THREADS) + threadIdx.x; p < np; p += int64_t(gridDim.x) * UB_THREADS)
        label[p] = -1;
}

}  // namespace

size_t hf::unbind_ws_bytes(const hf_box &box, int64_t np, int64_t nroots, bool records) {
    const UnbindLayout L = unbind_layout(box.n, np, nroots);
    return records ? L.full : L.total;
}

hf_status hf::unbind_dev(hf_ctx *ctx, const hf_box &box, const void *pos, const void *vel, hf_dtype dtype,
                         int64_t np, const int32_t *roots, int64_t nroots, const uint8_t *keep, int32_t *label,
                         double grav_mass, int64_t particle_th, uint8_t *bound_keep, void *ws, size_t ws_bytes,
                         const int64_t *d_count, const GroupCounters *counted) {
    if (nroots <= 0) return HF_OK;
    const UnbindLayout L = unbind_layout(box.n, np, nroots);
    char *w = static_cast<char *>(ws);
    auto *slot = reinterpret_cast<uint32_t *>(w + L.slot);
    auto *cnt = reinterpret_cast<uint32_t *>(w + L.cnt);
    auto *start = reinterpret_cast<uint32_t *>(w + L.start);
    auto *cur = reinterpret_cast<uint32_t *>(w + L.cursor);
    auto *partial = reinterpret_cast<uint64_t *>(w + L.partial);
    auto *queue = reinterpret_cast<uint32_t *>(w + L.queue);
    auto *pid = reinterpret_cast<int32_t *>(w + L.pid);
    const int64_t ncells = int64_t(box.n) * box.n * box.n;
    hipStream_t st = ctx->stream;
    HF_LAUNCH(ctx, K_UNBIND, ub_slots_kernel, dim3(ub_grid(ctx, nroots)), dim3(UB_THREADS), 0, st, roots, d_count,
              nroots, ncells, counted ? counted->parts : nullptr, counted ? counted->cells : nullptr, slot, cnt, cur,
              queue, ctx->d_status);
    if (np > 0 && !counted)
        HF_LAUNCH(ctx, K_UNBIND, ub_count_kernel, dim3(ub_grid(ctx, np)), dim3(UB_THREADS), 0, st, label, np, roots,
                  d_count, nroots, ncells, slot, keep, cnt, ctx->d_status);
    ScanJob sj = scan_job(cnt, nroots, partial, start);
    sj.d_n = d_count;
    launch_scan<SCAN_GROUPS>(ctx, K_UNBIND, sj);
    const bool records = ws_bytes >= L.full;
    auto gather = [&](auto *p, auto *v) {
        using T = std::remove_const_t<std::remove_pointer_t<decltype(p)>>;
        HF_LAUNCH(ctx, K_UNBIND, ub_gather_kernel<T>, dim3(ub_grid(ctx, np)), dim3(UB_THREADS), 0, st, label, np,
                  counted != nullptr, roots, d_count, nroots, ncells, slot, start, cur, pid, p, v,
                  records ? reinterpret_cast<T *>(w + L.rec) : nullptr, ctx->d_status);
    };
    if (np > 0 && dtype == HF_F32) gather(static_cast<const float *>(pos), static_cast<const float *>(vel));
    else if (np > 0) gather(static_cast<const double *>(pos), static_cast<const double *>(vel));
    // counts and cursors have served: the group lists take their place
    HF_LAUNCH(ctx, K_UNBIND, ub_list_kernel, dim3(ub_grid(ctx, (nroots + 7) / 8)), dim3(UB_THREADS), 0, st, d_count, nroots,
              keep, start, cnt, cur, queue, bound_keep);
    auto check = [&](auto *p, auto *v) {
        using T = std::remove_const_t<std::remove_pointer_t<decltype(p)>>;
        const UnbindJob<T> jb{p, v, label, roots, start, pid, reinterpret_cast<double *>(w + L.rad),
                              reinterpret_cast<uint32_t *>(w + L.ord), reinterpret_cast<uint32_t *>(w + L.tmp),
                              reinterpret_cast<double *>(w + L.spd), reinterpret_cast<uint8_t *>(w + L.alive),
                              records ? reinterpret_cast<uint32_t *>(w + L.perm) : nullptr,
                              records ? reinterpret_cast<const T *>(w + L.rec) : nullptr, box.n, box.box_len, grav_mass, particle_th, bound_keep};
        HF_LAUNCH(ctx, K_UNBIND, ub_group_kernel<T>, dim3(unsigned(ctx->cus)), dim3(UB_TEAM), 0, st, jb, cnt, nroots,
                  cur, queue);
    };
    if (dtype == HF_F32) check(static_cast<const float *>(pos), static_cast<const float *>(vel));
    else check(static_cast<const double *>(pos), static_cast<const double *>(vel));
    return launch_status();
}

hf_status hf::unclaim(hf_ctx *ctx, const int32_t *label, int64_t np, int32_t scale, int32_t *halo_scale,
                      int32_t *halo_root) {
    if (np <= 0) return HF_OK;
    HF_LAUNCH(ctx, K_UNBIND, ub_unclaim_kernel, dim3(ub_grid(ctx, np)), dim3(UB_THREADS), 0, ctx->stream, label,
              np, scale, halo_scale, halo_root);
    return launch_status();
}

extern "C" hf_status hf_unbind_ws_size(const hf_box *box, int64_t np, int64_t nroots, size_t *bytes) {
    if (!bytes || np < 0 || nroots < 0) return HF_ERR_ARG;
    hf_status s = check_box_grid(box);
    if (s != HF_OK) return s;
    *bytes = unbind_ws_bytes(*box, np, nroots, true);
    return HF_OK;
}

extern "C" hf_status hf_unbind_ws_size_least(const hf_box *box, int64_t np, int64_t nroots, size_t *bytes) {
    if (!bytes || np < 0 || nroots < 0) return HF_ERR_ARG;
    hf_status s = check_box_grid(box);
    if (s != HF_OK) return s;
    *bytes = unbind_ws_bytes(*box, np, nroots, false);
    return HF_OK;
}

extern "C" hf_status hf_unbind(hf_ctx *ctx, const hf_box *box, const void *pos, const void *vel, hf_dtype dtype,
                               int64_t np, const int32_t *roots, int64_t nroots, const uint8_t *group_keep,
                               int32_t *particle_label, double grav_mass, int64_t particle_th,
                               uint8_t *bound_keep, void *ws, size_t ws_bytes) {
    if (!ctx) return HF_ERR_ARG;
    hf_status s = check_box_grid(box);
    if (s != HF_OK) return s;
    const int64_t ncells = int64_t(box->n) * box->n * box->n;
    if (np < 0 || np > int64_t(INT32_MAX) || nroots < 0 || nroots > ncells) return HF_ERR_ARG;
    if (dtype != HF_F32 && dtype != HF_F64) return HF_ERR_ARG;
    if (!(grav_mass > 0.0) || !(grav_mass < 1e300) || particle_th < 0) return HF_ERR_ARG;
    if (np > 0 && (!pos || !vel || !particle_label)) return HF_ERR_ARG;
    if (nroots > 0 && (!roots || !group_keep || !bound_keep)) return HF_ERR_ARG;
    s = check_ws(ws, ws_bytes, unbind_ws_bytes(*box, np, nroots, false));
    if (s != HF_OK) return s;
    if (hipSetDevice(ctx->device) != hipSuccess) return HF_ERR_DEVICE;
    if (nroots == 0) {  // no group: every label goes
        if (np > 0)
            HF_LAUNCH(ctx, K_UNBIND, ub_clear_kernel, dim3(ub_grid(ctx, np)), dim3(UB_THREADS), 0, ctx->stream,
                      particle_label, np);
        return launch_status();
    }
    return unbind_dev(ctx, *box, pos, vel, dtype, np, roots, nroots, group_keep, particle_label, grav_mass,
                      particle_th, bound_keep, ws, ws_bytes, nullptr, nullptr);
}
