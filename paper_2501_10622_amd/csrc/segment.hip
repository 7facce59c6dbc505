// Step 4 (local maxima of the grid CWT) and step 5 (segmentation of the grid
// by its maxima, Sec. 2.3) on the FP32 CWT field.
//
// Order on cells: (value, linear index), larger value first, equal values by
// larger index, -0 equal to +0.  It is encoded as a 64-bit key whose integer
// order is that order: high word = order-preserving bits of the float, low
// word = index.  A cell's parent is the largest key of its 3x3x3 periodic
// neighbourhood (itself included); a cell is a maximum iff it is its own
// parent and its value exceeds tau.
//
// One workgroup per 32x16x16 tile holds the tile and a one-cell halo of the
// field in LDS, forms every cell's parent (the largest key of its 3x3x3
// neighbourhood) and the maxima mask, and follows the parent chains inside the
// tile, so the parents never go to memory.
//  - maxima: a wavefront covers two 32-cell rows, so its ballot is two aligned
//    32-bit words of a linear-order bit mask; count / scan / write passes turn
//    the mask into the sorted index list.
//  - segmentation: every cell ends at a root or at the first cell its chain
//    reaches outside the tile.  Such exit targets are always on a tile boundary,
//    so only the 2312 boundary cells of each tile (kept in a compact array) have
//    their chains followed across tiles.  A root at or below tau is no root to
//    its own tile, so the chains carry the threshold along and no later pass
//    reads the field again.  A last pass, one workgroup per tile, loads the
//    resolved entries of the one-cell shell around the tile (every exit target
//    lies in it) into LDS and maps each cell of the tile through them.
// Any n: where n is not a multiple of a tile's extent, the last tile along
// that axis is short (its cells past n are absent); a short tile's far-edge
// cells take the boundary ranks of a full tile's far edge, and the maxima are set
// bit by bit (rows straddle mask words).
#include "hf_internal.h"
#include "scan.h"

using namespace hf;

namespace {

// ------------------------------------------------------------------ keys
__device__ __forceinline__ uint32_t ordered_bits(float c, bool &nan) {
    uint32_t u = __float_as_uint(c);
    if ((u & 0x7fffffffu) > 0x7f800000u) nan = true;
    if (u == 0x80000000u) u = 0u;  // -0 -> +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ uint32_t wrap(int v, int n) { return uint32_t(v < 0 ? v + n : (v >= n ? v - n : v)); }

uint32_t host_ordered_bits(float c) {
    uint32_t u;
    static_assert(sizeof(u) == sizeof(c), "float is 32-bit");
    __builtin_memcpy(&u, &c, sizeof(u));
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// ------------------------------------------------------------------ tile geometry
// Resolve tiles: chains are followed inside RX x RY x RZ tiles.
constexpr int RX = 32, RY = 16, RZ = 16;
constexpr int RCELLS = RX * RY * RZ;                          // 8192
constexpr int RHX = RX + 2, RHY = RY + 2, RHZ = RZ + 2;
constexpr int RHCELLS = RHX * RHY * RHZ;                      // 11016 (tile plus one-cell shell)
static_assert(2 * RHX * RHY + (RHZ - 2) * (2 * RHX + 2 * (RHY - 2)) == RHCELLS - RCELLS, "shell enumeration");
constexpr int RING = 2 * RX + 2 * (RY - 2);                   // boundary cells of an inner z plane
constexpr int NBND = 2 * RX * RY + (RZ - 2) * RING;           // 2312 boundary cells per tile

struct TileGrid {
    int n;
    int ntx, nty, ntz;  // tiles per axis
    FastDiv dn;         // division by n
};

__device__ __forceinline__ void cell_coords(const TileGrid &tg, uint32_t g, uint32_t &x, uint32_t &y, uint32_t &z) {
    const uint32_t q = tg.dn.div(g);
    x = g - q * uint32_t(tg.n);
    z = tg.dn.div(q);
    y = q - z * uint32_t(tg.n);
}

// Rank of local cell (x, y, z) among its resolve tile's boundary cells, or -1.
// Order: plane z = 0, planes 1..RZ-2 (row y = 0, then x = 0 / x = RX-1 of rows
// 1..RY-2, then row y = RY-1), plane z = RZ-1.
__device__ __forceinline__ int bnd_rank(int x, int y, int z) {
    if (z == 0) return y * RX + x;
    if (z == RZ - 1) return RX * RY + (RZ - 2) * RING + y * RX + x;
    const int base = RX * RY + (z - 1) * RING;
    if (y == 0) return base + x;
    if (y == RY - 1) return base + RX + 2 * (RY - 2) + x;
    if (x == 0) return base + RX + 2 * (y - 1);
    if (x == RX - 1) return base + RX + 2 * (y - 1) + 1;
    return -1;
}

// Extent along one axis of the resolve tile starting at `origin`: R, or less
// for the last tile where n is not a multiple of R.
__device__ __forceinline__ int tile_extent(int origin, int R, int n) { return n - origin < R ? n - origin : R; }

// Rank among its tile's boundary cells of local cell (x, y, z) of a tile of
// extents (wx, wy, wz), or -1: a coordinate on a short tile's far edge counts
// as the full tile's far edge, which keeps the ranks distinct.
__device__ __forceinline__ int bnd_rank_in(int x, int y, int z, int wx, int wy, int wz) {
    return bnd_rank(x == wx - 1 ? RX - 1 : x, y == wy - 1 ? RY - 1 : y, z == wz - 1 ? RZ - 1 : z);
}

// Where the compact boundary array keeps cell (x, y, z) (rg: the resolve-tile
// grid), or -1 if it is interior to its tile.  FULL: n is a multiple of every
// tile extent, so no tile is short.
template <bool FULL>
__device__ __forceinline__ int64_t bnd_slot_at(const TileGrid &rg, uint32_t x, uint32_t y, uint32_t z) {
    const int tx = int(x / RX), ty = int(y / RY), tz = int(z / RZ);
    const int lx = int(x) - tx * RX, ly = int(y) - ty * RY, lz = int(z) - tz * RZ;
    const int r = FULL ? bnd_rank(lx, ly, lz)
                       : bnd_rank_in(lx, ly, lz, tile_extent(tx * RX, RX, rg.n), tile_extent(ty * RY, RY, rg.n),
                                     tile_extent(tz * RZ, RZ, rg.n));
    if (r < 0) return -1;
    const int64_t tile = (int64_t(tz) * rg.nty + ty) * rg.ntx + tx;
    return tile * NBND + r;
}

template <bool FULL>
__device__ __forceinline__ int64_t bnd_slot(const TileGrid &rg, int32_t g) {
    uint32_t x, y, z;
    cell_coords(rg, uint32_t(g), x, y, z);
    return bnd_slot_at<FULL>(rg, x, y, z);
}

__device__ __forceinline__ void rtile_origin(const TileGrid &rg, int t, int &x0, int &y0, int &z0) {
    x0 = (t % rg.ntx) * RX;
    y0 = ((t / rg.ntx) % rg.nty) * RY;
    z0 = (t / (rg.ntx * rg.nty)) * RZ;
}

// Parents and the chains inside a resolve tile in one pass, one workgroup per
// RX x RY x RZ tile.  A cell's parent is the largest key of its 3x3x3
// neighbourhood, and a root (its own parent) at or below tau is no root; with a
// mask the tile's maxima bits are written as well (the maxima are exactly the
// cells that are their own parent, above tau); without CHAINS they are all that is
// wanted.
//
// The tile and a one-cell shell of the field sit in LDS as 32-bit
// order-preserving bits, a row of RHX of them per (hy, hz).  A thread walks one
// z column.  Its nine columns' addresses are kept in the order of their cells'
// linear indices (rotated where the column or row lies at the end of the
// periodic box), so the largest key of a halo plane is the last largest value
// met in that order: a 32-bit compare and two selects per neighbour, the
// neighbour's address itself being what is selected.  A cell's parent is the
// largest of the three plane maxima around it, planes in index order too.
//
// The field's array then becomes the pointer array, with byte addresses as
// pointers: a cell points at its parent, a root and every cell of the shell at
// itself, a root at or below tau at the extra place NONE, which points at
// itself.  Following a pointer is one LDS read, done when it leads to itself.
// Wavefronts go on for themselves: what one reads while another writes lies
// further along the same chain.  The addresses reached go to ptr (16 bits per
// cell, a column of RZ per thread), and for the tile's boundary cells the index
// of the cell reached to bnd.
//
// Bound by the vector ALUs, busy 78% of the time with 108 instructions per cell
// (half of them the parents, a quarter the pointers).  With an index decoded per
// parent, a bounds check per axis, and workgroup-wide rounds over 32-bit indices it
// was 181 per cell and all of the time: 88 -> 67 us at 256^3, 4.76 -> 3.71 ms at
// 1024^3, 22 -> 15 us at 96^3.  For the maxima alone it took the place of
// a pass over 32x8x8 tiles
// with 64-bit keys and, where n is no multiple of 32, of one that read 27 values per
// cell from memory (235^3: 157 -> 37 us).
constexpr int PR_THREADS = RX * RY;           // one z column each
constexpr int PLANE_BYTES = 4 * RHX * RHY;
constexpr uint32_t NONE = 4 * RHCELLS;        // address of the place past the halo tile
static_assert(NONE <= 0xffffu, "addresses fit 16 bits");
static_assert(RZ % 8 == 0, "a column of addresses is whole 16-byte words");
constexpr int CHASE_FLAGS = 8;  // one per round of the boundary chase, at most 3 at n = 1024

// The words of a column's 16-bit addresses, RZ / 8 of 16 bytes.
constexpr int COLUMN_WORDS = RZ / 8;

template <bool FULL, bool CHAINS>
struct ParentResolve {
    static __device__ __forceinline__ void run(TileGrid rg, const float *__restrict__ c, uint32_t tau_ord,
                                               uint4 *__restrict__ ptr, int32_t *__restrict__ bnd,
                                               uint32_t *__restrict__ mask, uint32_t *__restrict__ flags,
                                               uint32_t *status) {
        __shared__ uint32_t V[RHCELLS + 1];
        __shared__ uint32_t rowbase[RHY * RHZ];  // index of the first cell of each halo row's grid row
        if (CHAINS && blockIdx.x == 0 && threadIdx.x < CHASE_FLAGS) flags[threadIdx.x] = 0u;  // of the chase that follows
        int x0, y0, z0;
        const uint32_t tile = xcd_remap(blockIdx.x, gridDim.x);
        rtile_origin(rg, int(tile), x0, y0, z0);
        const int n = rg.n;
        const uint32_t un = uint32_t(n);
        // a tile at the far end of an axis is short where n is not a multiple of
        // the tile: its cells past n are absent (never pointed to, never written)
        const int wx = FULL ? RX : tile_extent(x0, RX, n), wy = FULL ? RY : tile_extent(y0, RY, n),
                  wz = FULL ? RZ : tile_extent(z0, RZ, n);
        const int tid = threadIdx.x, x = tid % RX, y = tid / RX;
        if (tid < RHY * RHZ) {
            const int hy = tid % RHY, hz = tid / RHY;
            const bool there = FULL || (hy <= wy + 1 && hz <= wz + 1);
            rowbase[tid] = there ? (wrap(z0 + hz - 1, n) * un + wrap(y0 + hy - 1, n)) * un : 0u;
        }
        __syncthreads();
        bool nan = false;
        {
            // all loads of the halo tile are issued before any is used: the rows'
            // inner columns, 32 lanes to a row, then their two ends
            constexpr int ROWS = RHY * RHZ, STEP = PR_THREADS / RX, LOADS = (ROWS + STEP - 1) / STEP;
            constexpr int ENDS = (2 * ROWS + PR_THREADS - 1) / PR_THREADS;
            float v[LOADS], w[ENDS];
            // (past a short tile's shell any cell will do: nothing looks there)
            const uint32_t gx = FULL ? uint32_t(x0 + x) : (x <= wx ? wrap(x0 + x, n) : 0u);
            const uint32_t ends[2] = {wrap(x0 - 1, n), FULL || wx == RX ? wrap(x0 + RX, n) : 0u};
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const int r = y + i * STEP;
                if (r < ROWS) v[i] = c[rowbase[r] + gx];
            }
#pragma unroll
            for (int i = 0; i < ENDS; ++i) {
                const int e = tid + i * PR_THREADS;
                if (e < 2 * ROWS) w[i] = c[rowbase[e >> 1] + ends[e & 1]];
            }
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const int r = y + i * STEP;
                if (r < ROWS) V[r * RHX + x + 1] = ordered_bits(v[i], nan);
            }
#pragma unroll
            for (int i = 0; i < ENDS; ++i) {
                const int e = tid + i * PR_THREADS;
                if (e < 2 * ROWS) V[(e >> 1) * RHX + (e & 1) * (RHX - 1)] = ordered_bits(w[i], nan);
            }
        }
        __syncthreads();
        char *const lds = reinterpret_cast<char *>(V);
        auto at = [lds](uint32_t a) { return reinterpret_cast<uint32_t *>(lds + a); };
        // addresses in halo plane 0 of the columns around (x, y), in the order of
        // their linear indices: of rows y - 1, y, y + 1 and columns x - 1, x, x + 1 the
        // one beyond the end of the box comes last or first
        const uint32_t own = 4u * uint32_t((y + 1) * RHX + x + 1);
        uint32_t a[9];
        {
            const int xr = x0 + x == 0 ? 1 : (x0 + x == n - 1 ? 2 : 0), yr = y0 + y == 0 ? 1 : (y0 + y == n - 1 ? 2 : 0);
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const int dy = (k / 3 + yr) % 3 - 1, dx = (k % 3 + xr) % 3 - 1;
                a[k] = own + uint32_t(4 * (dy * RHX + dx));
            }
        }
        // value and address of the largest key of halo plane hz around the column
        auto plane_arg = [&](int hz, uint32_t &bv, uint32_t &ba) {
            bv = *at(a[0] + uint32_t(hz * PLANE_BYTES));
            ba = a[0];
#pragma unroll
            for (int k = 1; k < 9; ++k) {
                const uint32_t v = *at(a[k] + uint32_t(hz * PLANE_BYTES));
                const bool up = v >= bv;
                bv = up ? v : bv;
                ba = up ? a[k] : ba;
            }
            ba += uint32_t(hz * PLANE_BYTES);
        };
        auto larger = [](uint32_t &bv, uint32_t &ba, uint32_t v, uint32_t va) {
            const bool up = v >= bv;
            bv = up ? v : bv;
            ba = up ? va : ba;
        };
        const bool column = FULL || (x < wx && y < wy);
        uint32_t l[RZ];
        uint32_t maxima = 0;  // of the column
        {
            uint32_t v0, p0, v1, p1;
            plane_arg(0, v0, p0);
            plane_arg(1, v1, p1);
#pragma unroll
            for (int z = 0; z < RZ; ++z) {
                uint32_t v2, p2, bv, ba;
                plane_arg(z + 2, v2, p2);
                if (z0 + z == 0) {  // plane z - 1 is the last of the box
                    bv = v1;
                    ba = p1;
                    larger(bv, ba, v2, p2);
                    larger(bv, ba, v0, p0);
                } else if (z0 + z == n - 1) {  // plane z + 1 is the first
                    bv = v2;
                    ba = p2;
                    larger(bv, ba, v0, p0);
                    larger(bv, ba, v1, p1);
                } else {
                    bv = v0;
                    ba = p0;
                    larger(bv, ba, v1, p1);
                    larger(bv, ba, v2, p2);
                }
                const bool self = ba == own + uint32_t((z + 1) * PLANE_BYTES);
                const bool high = bv > tau_ord;
                if (FULL && mask) {  // a wavefront covers rows y and y + 1: two aligned mask words
                    const unsigned long long bits = __ballot(self && high);
                    if ((tid & 63) == 0) {
                        const uint32_t g = (uint32_t(z0 + z) * un + uint32_t(y0 + y)) * un + uint32_t(x0 + x);
                        mask[g >> 5] = uint32_t(bits);
                        mask[(g + un) >> 5] = uint32_t(bits >> 32);
                    }
                }
                maxima |= self && high ? 1u << z : 0u;
                l[z] = self && !high ? NONE : ba;
                v0 = v1;
                p0 = p1;
                v1 = v2;
                p1 = p2;
            }
        }
        if (nan) atomicOr(status, ST_INPUT);
        if (!FULL && mask && column) {  // rows straddle words: the mask was cleared first
            const uint32_t g = (uint32_t(z0) * un + uint32_t(y0 + y)) * un + uint32_t(x0 + x);
            for (int z = 0; z < wz; ++z) {
                const uint32_t gz = g + uint32_t(z) * un * un;
                if (maxima >> z & 1u) atomicOr(&mask[gz >> 5], 1u << (gz & 31u));
            }
        }
        if (!CHAINS) return;
        __syncthreads();  // every read of the field is done
        for (uint32_t e = tid; e <= uint32_t(RHCELLS); e += PR_THREADS) V[e] = 4u * e;
        __syncthreads();
        // where the column's pointers are; an absent cell's goes to NONE, which it holds
        auto slot = [=](int z) {
            return FULL || (column && z < wz) ? own + uint32_t((z + 1) * PLANE_BYTES) : NONE;
        };
#pragma unroll
        for (int z = 0; z < RZ; ++z) {
            if (!FULL && slot(z) == NONE) l[z] = NONE;
            *at(slot(z)) = l[z];
        }
        __syncthreads();
        // (relaxed atomic accesses: other wavefronts write while this one reads)
        bool open = true;
        while (open) {
            uint32_t w[RZ];
            uint32_t moved = 0;
#pragma unroll
            for (int z = 0; z < RZ; ++z) w[z] = __hip_atomic_load(at(l[z]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
            for (int z = 0; z < RZ; ++z) {
                moved |= w[z] ^ l[z];
                l[z] = w[z];
            }
#pragma unroll
            for (int z = 0; z < RZ; ++z)
                __hip_atomic_store(at(slot(z)), w[z], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            open = __any(moved != 0u);
        }
        uint4 *out = ptr + (size_t(tile) * PR_THREADS + uint32_t(tid)) * COLUMN_WORDS;
#pragma unroll
        for (int q = 0; q < COLUMN_WORDS; ++q)
            out[q] = make_uint4(l[8 * q] | (l[8 * q + 1] << 16), l[8 * q + 2] | (l[8 * q + 3] << 16),
                                l[8 * q + 4] | (l[8 * q + 5] << 16), l[8 * q + 6] | (l[8 * q + 7] << 16));
        if (!FULL && !(wx == RX && wy == RY && wz == RZ)) {
            // a short tile leaves some of its boundary slots unused: they hold -1
            // (final), so that the chase, which visits every slot, reads no
            // stale entry
            for (int k = tid; k < NBND; k += PR_THREADS) bnd[int64_t(tile) * NBND + k] = -1;
            __syncthreads();
        }
        if (!column) return;
        // index of the cell at address p
        auto cell_at = [&](uint32_t p) {
            if (p == NONE) return -1;
            const uint32_t r = p / (4u * RHX), hx = p / 4u - r * RHX;
            return int32_t(rowbase[r] + wrap(x0 + int(hx) - 1, n));
        };
        const int bx = x == wx - 1 ? RX - 1 : x, by = y == wy - 1 ? RY - 1 : y;  // a short tile's far edge: bnd_rank_in
        int32_t *mine = bnd + int64_t(tile) * NBND;
        const int ring = bnd_rank(bx, by, 1);  // of plane 1; later inner planes' ranks follow at equal distances
#pragma unroll
        for (int z = 0; z < RZ; ++z) {
            if (!FULL && z >= wz) continue;
            if (z == wz - 1)
                mine[bnd_rank(bx, by, RZ - 1)] = cell_at(l[z]);
            else if (z == 0)
                mine[bnd_rank(bx, by, 0)] = cell_at(l[z]);
            else if (ring >= 0)
                mine[ring + (z - 1) * RING] = cell_at(l[z]);
        }
    }
};

template <bool FULL, bool CHAINS>
__global__ void __launch_bounds__(PR_THREADS) parent_resolve_kernel(const float *__restrict__ c, TileGrid rg,
                    uint32_t tau_ord, uint4 *__restrict__ ptr, int32_t *__restrict__ bnd, uint32_t *__restrict__ mask,
                    uint32_t *__restrict__ flags, uint32_t *status) {
    ParentResolve<FULL, CHAINS>::run(rg, c, tau_ord, ptr, bnd, mask, flags, status);
}

__global__ void zero_words_kernel(uint32_t *w, int64_t count) {
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < count; i += int64_t(gridDim.x) * blockDim.x)
        w[i] = 0u;
}

// Follows the pointer chains of the boundary entries to their ends, in place:
// an entry is final when it is -1, points at an interior cell (a root, since a
// chain leaves a tile through its boundary) or at a boundary cell that points
// at itself (a root).  Entries of other tiles may be advanced while they are
// read; whatever a read returns lies further along the same chain, so the ends
// do not depend on the order.
//
// One launch takes at most CHASE_HOPS hops per entry: after it every pointer
// is final or has come CHASE_HOPS boundary cells along its chain, so each hop of
// the next launch covers as many, and ceil(log_CHASE_HOPS(entries)) rounds
// reach the end of any chain.  A launch runs only if the one before left an
// entry open, and the last round is the final pass's, on the entries it reads
// (follow).  Chains cross few tiles (one to three at scales of 1 to 4 cells),
// so the first launch ends them all, and a hop is two dependent loads: the
// latency of BATCH chains per thread is what bounds it.  Rounds of pointer
// doubling with lists of the entries still open (one hop per launch,
// ceil(log2(entries)) + 1 launches, 18 at 64^3 to 30 at 1024^3, 2.2 us each when
// nothing is left to do) took 48 us at 64^3, 123 us at 256^3 and 2.0 ms at
// 1024^3 where the chase takes 17 us, 47 us and 1.47 ms.
constexpr int BATCH = 8;  // independent chains per thread, so their loads overlap
constexpr int CHASE_HOPS = 1024;

template <bool FULL>
__device__ int32_t follow(const int32_t *__restrict__ bnd, const TileGrid &tg, int32_t p) {
    while (p >= 0) {
        const int64_t s = bnd_slot<FULL>(tg, p);
        const int32_t q = s >= 0 ? bnd[s] : p;
        if (q == p) break;
        p = q;
    }
    return p;
}

template <bool FULL>
struct BndChase {
    static __device__ __forceinline__ void run(TileGrid tg, int32_t *bnd, int64_t count, uint32_t *flags, int round) {
        if (round > 0 && flags[round] == 0u) return;
        bool open = false;
        const int64_t step = int64_t(gridDim.x) * blockDim.x * BATCH;
        for (int64_t k0 = blockIdx.x * int64_t(blockDim.x) * BATCH + threadIdx.x; k0 < count; k0 += step) {
            int32_t p0[BATCH], p[BATCH];
            bool on[BATCH];
            bool any = false;
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int64_t k = k0 + int64_t(i) * blockDim.x;
                p0[i] = k < count ? bnd[k] : -1;
            }
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                p[i] = p0[i];
                on[i] = p[i] >= 0;
                any |= on[i];
            }
            for (int hop = 0; any && hop < CHASE_HOPS; ++hop) {
                int32_t q[BATCH];
#pragma unroll
                for (int i = 0; i < BATCH; ++i) {
                    const int64_t s = on[i] ? bnd_slot<FULL>(tg, p[i]) : -1;
                    q[i] = s >= 0 ? bnd[s] : p[i];
                }
                any = false;
#pragma unroll
                for (int i = 0; i < BATCH; ++i) {
                    on[i] = q[i] != p[i] && q[i] >= 0;
                    p[i] = q[i];
                    any |= on[i];
                }
            }
            open |= any;
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int64_t k = k0 + int64_t(i) * blockDim.x;
                if (p[i] != p0[i]) bnd[k] = p[i];
            }
        }
        if (__ballot(open) && (threadIdx.x & 63) == 0) flags[round + 1] = 1u;
    }
};

template <bool FULL>
__global__ void __launch_bounds__(256) bnd_chase_kernel(int32_t *bnd, int64_t count, TileGrid tg, uint32_t *flags,
                    int round) {
    BndChase<FULL>::run(tg, bnd, count, flags, round);
}

// One workgroup per resolve tile.  A table in LDS holds, at each place of the
// halo tile, the root that a pointer to it stands for: the resolved boundary
// entries of the one-cell shell around the tile (they belong to the neighbouring
// tiles; every exit target of the tile lies in the shell), each cell of the tile
// its own index (only roots above tau are pointed at), and -1 at NONE.  A cell's
// label is then the table's entry at its address.  Bound by HBM: 2 bytes read and
// 4 written per cell (1024^3: 1.57 ms, 4.1 TB/s).  With 32-bit indices in ptr, taken
// apart into coordinates for every cell, 2.38 ms; 256^3 40 -> 22 us.
template <bool FULL>
struct SegFinalize {
    static __device__ __forceinline__ void run(TileGrid rg, const uint4 *__restrict__ ptr,
                                               const int32_t *__restrict__ bnd, const uint32_t *__restrict__ open,
                                               int32_t *__restrict__ label) {
        __shared__ int32_t table[RHCELLS + 1];
        int x0, y0, z0;
        const uint32_t tile = xcd_remap(blockIdx.x, gridDim.x);
        rtile_origin(rg, int(tile), x0, y0, z0);
        const int n = rg.n;
        const uint32_t un = uint32_t(n);
        const int wx = FULL ? RX : tile_extent(x0, RX, n), wy = FULL ? RY : tile_extent(y0, RY, n),
                  wz = FULL ? RZ : tile_extent(z0, RZ, n);
        // this column's addresses and the shell's entries, all loads issued before any is used
        const int tid = threadIdx.x, x = tid % RX, y = tid / RX;
        uint4 t[COLUMN_WORDS];
        const uint4 *in = ptr + (size_t(tile) * PR_THREADS + uint32_t(tid)) * COLUMN_WORDS;
#pragma unroll
        for (int q = 0; q < COLUMN_WORDS; ++q) t[q] = in[q];
        // the one-cell shell around the tile's (wx, wy, wz) cells, enumerated: the
        // two z planes, then per inner plane the two y rows and the two x ends of
        // the rows between them; shell cell (hx, hy, hz) sits at LDS place
        // (hz RHY + hy) RHX + hx, with the tile's cells at 1..wx, 1..wy, 1..wz
        const int ex = wx + 2, ey = wy + 2, ez = wz + 2;
        const int zplane = ex * ey, ring = 2 * ex + 2 * (ey - 2);
        const int nshell = 2 * zplane + (ez - 2) * ring;
        constexpr int LOADS = (RHCELLS - RCELLS + PR_THREADS - 1) / PR_THREADS;
        int32_t v[LOADS];
        int at[LOADS];
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int k = tid + i * PR_THREADS;
            at[i] = -1;
            if (k >= nshell) continue;
            int hx, hy, hz;
            if (k < 2 * zplane) {
                hz = k < zplane ? 0 : ez - 1;
                const int j = k % zplane;
                hy = j / ex;
                hx = j % ex;
            } else {
                const int j = k - 2 * zplane;
                hz = 1 + j / ring;
                const int r = j % ring;
                if (r < 2 * ex) {
                    hy = r < ex ? 0 : ey - 1;
                    hx = r % ex;
                } else {
                    const int q = r - 2 * ex;
                    hy = 1 + q / 2;
                    hx = (q & 1) ? ex - 1 : 0;
                }
            }
            const uint32_t gx = wrap(x0 + hx - 1, n), gy = wrap(y0 + hy - 1, n), gz = wrap(z0 + hz - 1, n);
            v[i] = bnd[bnd_slot_at<FULL>(rg, gx, gy, gz)];  // on its tile's boundary
            at[i] = (hz * RHY + hy) * RHX + hx;
        }
#pragma unroll
        for (int i = 0; i < LOADS; ++i)
            if (at[i] >= 0) table[at[i]] = v[i];
        __syncthreads();
        if (*open != 0u) {  // the chase left entries open: the rest of the way, at most CHASE_HOPS steps
#pragma unroll 1
            for (int k = tid; k < RHCELLS; k += PR_THREADS) {
                const int hx = k % RHX, hy = (k / RHX) % RHY, hz = k / (RHX * RHY);
                if (hx >= ex || hy >= ey || hz >= ez) continue;
                if (hx == 0 || hx == ex - 1 || hy == 0 || hy == ey - 1 || hz == 0 || hz == ez - 1)
                    table[k] = follow<FULL>(bnd, rg, bnd[bnd_slot_at<FULL>(rg, wrap(x0 + hx - 1, n), wrap(y0 + hy - 1, n),
                                                                           wrap(z0 + hz - 1, n))]);
            }
        }
        if (tid == 0) table[RHCELLS] = -1;
        const bool column = x < wx && y < wy;
        const uint32_t g0 = ((uint32_t(z0) * un) + uint32_t(y0 + y)) * un + uint32_t(x0 + x);
        const int own = (RHY + y + 1) * RHX + x + 1;
#pragma unroll
        for (int z = 0; z < RZ; ++z)
            if (FULL || (column && z < wz)) table[own + z * RHX * RHY] = int32_t(g0 + uint32_t(z) * un * un);
        __syncthreads();
        if (!column) return;
        const char *lds = reinterpret_cast<const char *>(table);
#pragma unroll
        for (int z = 0; z < RZ; ++z) {
            if (!FULL && z >= wz) continue;
            const uint32_t word = (&t[z / 8].x)[(z % 8) / 2], a = z & 1 ? word >> 16 : word & 0xffffu;
            label[g0 + uint32_t(z) * un * un] = *reinterpret_cast<const int32_t *>(lds + a);
        }
    }
};

template <bool FULL>
__global__ void __launch_bounds__(PR_THREADS) seg_finalize_kernel(const uint4 *__restrict__ ptr,
                    const int32_t *__restrict__ bnd, TileGrid rg, const uint32_t *__restrict__ open,
                    int32_t *__restrict__ label) {
    SegFinalize<FULL>::run(rg, ptr, bnd, open, label);
}

// ------------------------------------------------------------------ mask -> sorted list
constexpr int LIST_CHUNK_WORDS = 128;  // 4096 cells per chunk

__global__ void __launch_bounds__(LIST_CHUNK_WORDS) mask_count_kernel(const uint32_t *__restrict__ mask,
                                                                      int64_t words, uint32_t *__restrict__ counts) {
    const int64_t w = int64_t(blockIdx.x) * LIST_CHUNK_WORDS + threadIdx.x;
    uint32_t v = w < words ? uint32_t(__popc(mask[w])) : 0u;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    __shared__ uint32_t red[LIST_CHUNK_WORDS / 64];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = red[0] + red[1];
}

// Writes the cells of this thread's mask word (word w, value bits) of a chunk
// whose first cell goes to place `base` of the list; returns the place after the
// thread's last.
__device__ __forceinline__ uint32_t write_cells(int64_t w, uint32_t bits, uint32_t base, int64_t cap,
                                                int32_t *__restrict__ out) {
    static_assert(LIST_CHUNK_WORDS == 128, "two wavefronts");
    __shared__ uint32_t first;  // maxima of the first wavefront's words
    const uint32_t count = uint32_t(__popc(bits));
    uint32_t upto = count;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t v = __shfl_up(upto, off, 64);
        if (int(threadIdx.x & 63u) >= off) upto += v;
    }
    if (threadIdx.x == 63) first = upto;
    __syncthreads();
    uint32_t r = base + upto - count + (threadIdx.x >= 64 ? first : 0u);
    while (bits) {
        const int b = __ffs(bits) - 1;
        bits &= bits - 1;
        if (int64_t(r) < cap) out[r] = int32_t(w * 32 + b);
        ++r;
    }
    return r;
}

__global__ void __launch_bounds__(LIST_CHUNK_WORDS) list_write_kernel(const uint32_t *__restrict__ mask,
                                                                      int64_t words,
                                                                      const uint32_t *__restrict__ offsets,
                                                                      int64_t cap, int32_t *__restrict__ out) {
    const int64_t w = int64_t(blockIdx.x) * LIST_CHUNK_WORDS + threadIdx.x;
    write_cells(w, w < words ? mask[w] : 0u, offsets[blockIdx.x], cap, out);
}

// A short mask (up to LIST_SHORT chunks, n = 128) in one launch: a workgroup counts
// the words before its chunk itself, and the last one has the total.  Three
// launches of 3 to 5 us each are what the short lists took (12.2 us at 64^3, 13.4 at
// 128^3, where this takes 4.4 and 11); at 256^3 the words would be read 2048 times.
constexpr int LIST_SHORT = 512;

struct ListShort {
    static __device__ __forceinline__ void run(int64_t words, const uint32_t *__restrict__ mask, int64_t cap,
                                               int32_t *__restrict__ out, int64_t *__restrict__ d_count,
                                               uint32_t *status) {
        __shared__ uint32_t red[LIST_CHUNK_WORDS / 64];
        const uint4 *before = reinterpret_cast<const uint4 *>(mask);  // whole chunks lie before this one
        uint32_t sum = 0;
#pragma unroll 8
        for (uint32_t k = threadIdx.x; k < blockIdx.x * (LIST_CHUNK_WORDS / 4); k += LIST_CHUNK_WORDS) {
            const uint4 m = before[k];
            sum += uint32_t(__popc(m.x) + __popc(m.y) + __popc(m.z) + __popc(m.w));
        }
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
        __syncthreads();
        const int64_t w = int64_t(blockIdx.x) * LIST_CHUNK_WORDS + threadIdx.x;
        const uint32_t end = write_cells(w, w < words ? mask[w] : 0u, red[0] + red[1], cap, out);
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == LIST_CHUNK_WORDS - 1) {
            *d_count = int64_t(end);
            if (int64_t(end) > cap) atomicOr(status, ST_CAPACITY);
        }
    }
};

__global__ void __launch_bounds__(LIST_CHUNK_WORDS) list_short_kernel(const uint32_t *__restrict__ mask,
                    int64_t words, int64_t cap, int32_t *__restrict__ out, int64_t *__restrict__ d_count,
                    uint32_t *status) {
    ListShort::run(words, mask, cap, out, d_count, status);
}

// ------------------------------------------------------------------ host side
// True where every resolve tile is whole (n a multiple of 32, hence of 16).
bool all_full(int n) { return n % RX == 0 && n % RY == 0 && n % RZ == 0; }

// Resolve tiles over any n: the last tile along an axis is short where n is
// not a multiple of the tile.
TileGrid resolve_grid(int n) {
    return TileGrid{n, (n + RX - 1) / RX, (n + RY - 1) / RY, (n + RZ - 1) / RZ, FastDiv(uint32_t(n))};
}

// Rounds that end every chain of at most `count` boundary cells (a launch at least, and the final pass's).
int chase_rounds(uint64_t count) {
    int k = 2;
    for (uint64_t reach = uint64_t(CHASE_HOPS) * CHASE_HOPS; reach < count; reach *= CHASE_HOPS) ++k;
    return k;
}

struct MaximaLayout {
    size_t mask, counts, offsets, partial, total;
    int64_t words;
    int nchunks;
};

MaximaLayout maxima_layout(int n) {
    MaximaLayout L{};
    const size_t cells = size_t(n) * n * n;
    L.words = int64_t((cells + 31) / 32);
    L.nchunks = int((L.words + LIST_CHUNK_WORDS - 1) / LIST_CHUNK_WORDS);
    size_t off = 0;
    L.mask = off;
    off = align_up(off + sizeof(uint32_t) * size_t(L.words + 2));
    L.counts = off;
    off = align_up(off + sizeof(uint32_t) * L.nchunks);
    L.offsets = off;
    off = align_up(off + sizeof(uint32_t) * (L.nchunks + 1));
    L.partial = off;
    off = align_up(off + sizeof(uint64_t) * SCAN_MAX_GROUPS);
    L.total = off;
    return L;
}

int stride_grid(int64_t work) {
    int64_t g = (work + 255) / 256;
    return int(g > 4096 ? 4096 : (g < 1 ? 1 : g));
}

struct SegmentLayout {
    size_t flags, ptr, bnd, total;
    int rounds;  // of the boundary chase, the last one the final pass's
    int64_t nbnd;
};

SegmentLayout segment_layout(int n) {
    SegmentLayout L{};
    const TileGrid rg = resolve_grid(n);
    const uint64_t tiles = uint64_t(rg.ntx) * rg.nty * rg.ntz;
    L.nbnd = int64_t(tiles) * NBND;
    L.rounds = chase_rounds(uint64_t(L.nbnd));
    size_t off = 0;
    L.flags = off;
    off = align_up(off + sizeof(uint32_t) * CHASE_FLAGS);
    L.ptr = off;
    off = align_up(off + sizeof(uint16_t) * RCELLS * tiles);
    L.bnd = off;
    off = align_up(off + sizeof(int32_t) * size_t(L.nbnd));
    L.total = off;
    return L;
}

}  // namespace

size_t hf::maxima_ws_bytes(const hf_box &box) { return maxima_layout(box.n).total; }

size_t hf::segment_ws_bytes(const hf_box &box) { return segment_layout(box.n).total; }

namespace {

// Count / scan / write passes: maxima bit mask (in the maxima workspace at w8)
// -> sorted index list and its length.
hf_status mask_to_list(hf_ctx *ctx, const MaximaLayout &L, char *w8, int32_t *max_idx, int64_t max_cap,
                       int64_t *d_count) {
    auto *mask = reinterpret_cast<uint32_t *>(w8 + L.mask);
    auto *counts = reinterpret_cast<uint32_t *>(w8 + L.counts);
    auto *offsets = reinterpret_cast<uint32_t *>(w8 + L.offsets);
    if (L.nchunks <= LIST_SHORT) {
        HF_LAUNCH(ctx, K_MAX_WRITE, list_short_kernel, dim3(L.nchunks), dim3(LIST_CHUNK_WORDS), 0, ctx->stream, mask,
                  L.words, max_cap, max_idx, d_count, ctx->d_status);
        return launch_status();
    }
    HF_LAUNCH(ctx, K_MAX_COUNT, mask_count_kernel, dim3(L.nchunks), dim3(LIST_CHUNK_WORDS), 0, ctx->stream, mask,
              L.words, counts);
    const ScanJob sj = scan_job(counts, L.nchunks, reinterpret_cast<uint64_t *>(w8 + L.partial), offsets, nullptr,
                                d_count, max_cap, ctx->d_status);
    launch_scan<SCAN_MAXIMA>(ctx, K_MAX_SCAN, sj);
    HF_LAUNCH(ctx, K_MAX_WRITE, list_write_kernel, dim3(L.nchunks), dim3(LIST_CHUNK_WORDS), 0, ctx->stream, mask,
              L.words, offsets, max_cap, max_idx);
    return launch_status();
}

// Parents (and the maxima mask when given), with the chains inside each resolve
// tile followed: ptr and bnd of the segmentation workspace.
hf_status launch_parent_resolve(hf_ctx *ctx, const SegmentLayout &L, char *w8, int n, const float *cwt, float tau,
                                uint32_t *mask) {
    const TileGrid tg = resolve_grid(n);
    const dim3 grid(tg.ntx * tg.nty * tg.ntz);
    auto *ptr = reinterpret_cast<uint4 *>(w8 + L.ptr);
    auto *bnd = reinterpret_cast<int32_t *>(w8 + L.bnd);
    auto *flags = reinterpret_cast<uint32_t *>(w8 + L.flags);
    if (all_full(n))
        HF_LAUNCH(ctx, K_PARENT, (parent_resolve_kernel<true, true>), grid, dim3(PR_THREADS), 0, ctx->stream, cwt, tg,
                  host_ordered_bits(tau), ptr, bnd, mask, flags, ctx->d_status);
    else
        HF_LAUNCH(ctx, K_PARENT, (parent_resolve_kernel<false, true>), grid, dim3(PR_THREADS), 0, ctx->stream, cwt, tg,
                  host_ordered_bits(tau), ptr, bnd, mask, flags, ctx->d_status);
    return launch_status();
}

// Where rows straddle mask words the maxima are set bit by bit into a cleared mask.
void clear_mask(hf_ctx *ctx, const MaximaLayout &L, int n, uint32_t *mask) {
    if (!all_full(n))
        HF_LAUNCH(ctx, K_FLAGS, zero_words_kernel, dim3(stride_grid(L.words)), dim3(256), 0, ctx->stream, mask, L.words);
}

// After launch_parent_resolve: the chains of the boundary entries, and the
// final mapping through them.
hf_status segment_finish(hf_ctx *ctx, const SegmentLayout &L, char *w8, int n, int32_t *cell_label) {
    const TileGrid tg = resolve_grid(n);
    auto *flags = reinterpret_cast<uint32_t *>(w8 + L.flags);
    auto *ptr = reinterpret_cast<uint4 *>(w8 + L.ptr);
    auto *bnd = reinterpret_cast<int32_t *>(w8 + L.bnd);
    const bool full = all_full(n);
    const dim3 chase(stride_grid((L.nbnd + BATCH - 1) / BATCH));
    for (int r = 0; r + 1 < L.rounds; ++r) {
        if (full)
            HF_LAUNCH(ctx, K_JUMP, bnd_chase_kernel<true>, chase, dim3(256), 0, ctx->stream, bnd, L.nbnd, tg, flags,
                      r);
        else
            HF_LAUNCH(ctx, K_JUMP, bnd_chase_kernel<false>, chase, dim3(256), 0, ctx->stream, bnd, L.nbnd, tg, flags,
                      r);
    }
    const dim3 grid(tg.ntx * tg.nty * tg.ntz);
    if (full)
        HF_LAUNCH(ctx, K_FINALIZE, seg_finalize_kernel<true>, grid, dim3(PR_THREADS), 0, ctx->stream, ptr, bnd, tg,
                  flags + L.rounds - 1, cell_label);
    else
        HF_LAUNCH(ctx, K_FINALIZE, seg_finalize_kernel<false>, grid, dim3(PR_THREADS), 0, ctx->stream, ptr, bnd, tg,
                  flags + L.rounds - 1, cell_label);
    return launch_status();
}

}  // namespace

bool hf::segment_group_supported(int n) { return all_full(n) && maxima_layout(n).nchunks <= LIST_SHORT; }

hf_status hf::segment_group(hf_ctx *ctx, int n, int count, const GroupBox *b) {
    const SegmentLayout L = segment_layout(n);
    const MaximaLayout ML = maxima_layout(n);
    const TileGrid tg = resolve_grid(n);
    const unsigned tiles = unsigned(tg.ntx * tg.nty * tg.ntz);
    Boxes<const float *, uint32_t, uint4 *, int32_t *, uint32_t *, uint32_t *, uint32_t *> parent{};
    Boxes<const uint32_t *, int64_t, int32_t *, int64_t *, uint32_t *> list{};
    Boxes<int32_t *, int64_t, uint32_t *, int> chase{};
    Boxes<const uint4 *, const int32_t *, const uint32_t *, int32_t *> last{};
    for (int j = 0; j < count; ++j) {
        auto *ptr = reinterpret_cast<uint4 *>(b[j].ws + L.ptr);
        auto *bnd = reinterpret_cast<int32_t *>(b[j].ws + L.bnd);
        auto *flags = reinterpret_cast<uint32_t *>(b[j].ws + L.flags);
        auto *mask = reinterpret_cast<uint32_t *>(b[j].ws + L.total + ML.mask);
        pack(parent.a[j], b[j].cwt, host_ordered_bits(b[j].tau), ptr, bnd, mask, flags, ctx->d_status);
        pack(list.a[j], static_cast<const uint32_t *>(mask), b[j].max_cap, b[j].max_idx, b[j].d_count, ctx->d_status);
        pack(chase.a[j], bnd, L.nbnd, flags, 0);
        pack(last.a[j], static_cast<const uint4 *>(ptr), static_cast<const int32_t *>(bnd),
             static_cast<const uint32_t *>(flags + L.rounds - 1), b[j].cell_label);
    }
    launch_group<ParentResolve<true, true>, PR_THREADS>(ctx, K_PARENT, tiles, count, parent, tg);
    launch_group<ListShort, LIST_CHUNK_WORDS>(ctx, K_MAX_WRITE, unsigned(ML.nchunks), count, list, ML.words);
    for (int r = 0; r + 1 < L.rounds; ++r) {
        for (int j = 0; j < count; ++j) pack(chase.a[j], chase.a[j].head, L.nbnd, chase.a[j].tail.tail.head, r);
        launch_group<BndChase<true>, 256>(ctx, K_JUMP, unsigned(stride_grid((L.nbnd + BATCH - 1) / BATCH)), count, chase,
                                          tg);
    }
    launch_group<SegFinalize<true>, PR_THREADS>(ctx, K_FINALIZE, tiles, count, last, tg);
    return launch_status();
}

size_t hf::maxima_segment_ws_bytes(const hf_box &box) {
    return segment_layout(box.n).total + maxima_layout(box.n).total;
}

// Steps 4 and 5 together: on tiled grids one pass over the field yields both
// the parents and the maxima mask.  Same results as hf_maxima then hf_segment.
hf_status hf::maxima_segment(hf_ctx *ctx, const hf_box &box, const float *cwt, float tau, int32_t *max_idx,
                             int64_t max_cap, int64_t *d_count, int32_t *cell_label, void *ws, size_t ws_bytes) {
    const int n = box.n;
    if (!ctx || !cwt || !d_count || !cell_label || max_cap < 0 || (max_cap > 0 && !max_idx) || tau != tau)
        return HF_ERR_ARG;
    const SegmentLayout SL = segment_layout(n);
    const MaximaLayout ML = maxima_layout(n);
    hf_status s = check_ws(ws, ws_bytes, SL.total + ML.total);
    if (s != HF_OK) return s;
    if (hipSetDevice(ctx->device) != hipSuccess) return HF_ERR_DEVICE;
    char *w8 = static_cast<char *>(ws);
    char *wm = w8 + SL.total;
    auto *mask = reinterpret_cast<uint32_t *>(wm + ML.mask);
    clear_mask(ctx, ML, n, mask);
    s = launch_parent_resolve(ctx, SL, w8, n, cwt, tau, mask);
    if (s != HF_OK) return s;
    s = mask_to_list(ctx, ML, wm, max_idx, max_cap, d_count);
    if (s != HF_OK) return s;
    return segment_finish(ctx, SL, w8, n, cell_label);
}

extern "C" hf_status hf_maxima(hf_ctx *ctx, const hf_box *box, const float *cwt, float tau, int32_t *max_idx,
                               int64_t max_cap, int64_t *d_count, void *ws, size_t ws_bytes) {
    if (!ctx || !cwt || !d_count || max_cap < 0 || (max_cap > 0 && !max_idx)) return HF_ERR_ARG;
    if (tau != tau) return HF_ERR_ARG;
    hf_status s = check_box_grid(box);
    if (s != HF_OK) return s;
    const MaximaLayout L = maxima_layout(box->n);
    s = check_ws(ws, ws_bytes, L.total);
    if (s != HF_OK) return s;
    if (hipSetDevice(ctx->device) != hipSuccess) return HF_ERR_DEVICE;
    char *w8 = static_cast<char *>(ws);
    auto *mask = reinterpret_cast<uint32_t *>(w8 + L.mask);
    const int n = box->n;
    const TileGrid tg = resolve_grid(n);
    const dim3 grid(tg.ntx * tg.nty * tg.ntz);
    clear_mask(ctx, L, n, mask);
    if (all_full(n))
        HF_LAUNCH(ctx, K_MAX_MARK, (parent_resolve_kernel<true, false>), grid, dim3(PR_THREADS), 0, ctx->stream, cwt,
                  tg, host_ordered_bits(tau), nullptr, nullptr, mask, nullptr, ctx->d_status);
    else
        HF_LAUNCH(ctx, K_MAX_MARK, (parent_resolve_kernel<false, false>), grid, dim3(PR_THREADS), 0, ctx->stream, cwt,
                  tg, host_ordered_bits(tau), nullptr, nullptr, mask, nullptr, ctx->d_status);
    return mask_to_list(ctx, L, w8, max_idx, max_cap, d_count);
}

extern "C" hf_status hf_segment(hf_ctx *ctx, const hf_box *box, const float *cwt, float tau, int32_t *cell_label,
                                void *ws, size_t ws_bytes) {
    if (!ctx || !cwt || !cell_label) return HF_ERR_ARG;
    if (tau != tau) return HF_ERR_ARG;
    hf_status s = check_box_grid(box);
    if (s != HF_OK) return s;
    const SegmentLayout L = segment_layout(box->n);
    s = check_ws(ws, ws_bytes, L.total);
    if (s != HF_OK) return s;
    if (hipSetDevice(ctx->device) != hipSuccess) return HF_ERR_DEVICE;
    char *w8 = static_cast<char *>(ws);
    const int n = box->n;
    s = launch_parent_resolve(ctx, L, w8, n, cwt, tau, nullptr);
    if (s != HF_OK) return s;
    return segment_finish(ctx, L, w8, n, cell_label);
}
