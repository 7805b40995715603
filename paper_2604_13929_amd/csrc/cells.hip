// cells.hip -- the cell walk of large runs.
//
// k_walk deposits every voxel visit at the memory side: 0.34 requests of 64 bytes per
// photon-step at best, at 26.8e9 requests/s (the chip's rate for atomics), 7.8e10 steps/s.
// Here the tally a photon deposits into is in LDS instead.  The volume is cut into cells of at
// most 32^3 voxels; a workgroup holds one cell's mask and tally (34^3 words with a halo of one
// voxel, 157 KB: one workgroup of 16 wavefronts per compute unit) and advances photons that
// stand in that cell until they leave it, some 30 steps later.  A photon waits between two visits
// in a slot of device memory (64 bytes, one line).  A run is a sequence of rounds:
//   k_cells_count    launches photons into free slots, counts the slots' photons per cell
//   k_cells_columns  turns the blocks' counts into ranks
//   k_cells_scatter  lists the slots cell by cell and cuts the list into items for the walk
//   k_cells_walk     every workgroup takes items (a cell and a stretch of its list) until none is left
// Once too few photons are alive to fill the chip this way, the rounds end and k_cells_tail
// walks the rest to their ends with the deposit log.  The number of rounds enqueued is an
// estimate made on the host, so that nothing waits for the device and the sequence can be
// captured: rounds after the end return at once, and what a short estimate (or one of more than
// kMaxRounds, 1.3e9 photons at 256^3) leaves undone the tail does.  A photon's own history, the
// integer tallies and so every result are those of k_walk, bit for bit.
// Measured on the 256^3 workload of 1e8 photons: 491 ms (1.98e11 steps/s) against 1259 ms.  Within
// a round the walk is bound by its VALU (busy 91 % of the cycles its wavefronts are resident, which
// is 84 % of the round): 86 wave-instructions per iteration, about 48 of 64 lanes stepping.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>

#include "cells.hpp"
#include "score.hpp"
#include "stage.hpp"

using namespace pmc;
using namespace pmc::host;

static_assert(sizeof(Job) % 8 == 0, "jobs are written in 8-byte words");

namespace {

constexpr int kCell = 32;                  // largest cell extent per axis
constexpr int kSide = kCell + 2;           // with one halo voxel on each side
constexpr int kRow = kSide, kLayer = kSide * kSide, kWords = kSide * kSide * kSide;
constexpr uint32_t kDead = 0xFFFFFFFFu;
constexpr size_t kLds = 160 * 1024;         // LDS of a compute unit
constexpr int kSortBlocks = 256;
constexpr int kSortThreads = 1024;
constexpr int32_t kMaxCells = 32768;
constexpr uint32_t kMinItem = 2048, kMaxItem = 65536;   // photons of an item
// When the rounds end: a round has a fixed cost (launches, and a cell's mask in and tally out for each cell
// taken), the tail runs at the deposit log's rate.  Ending at less than kStopPerCu photons per compute unit and
// kStopPerCell per cell measured lowest or within 2 % of it for 256^3 (512 cells, 1e7 photons: 75 ms; 80 at
// 0.33e6 photons whatever the cells), 512 x 512 x 256 (2048 cells, 2e7 photons: 118 ms; 147) and a batch of 12
// volumes (69 ms; 104).  A cell with fewer than kLeastPerCell photons is not taken: they wait for more to
// come (the batch: 77 ms with every cell taken, 75 from 256 photons on, 70 from 512, 69 from 1024; 256^3 loses
// 6 % at 4096).
constexpr uint32_t kStopPerCu = 2560;
constexpr uint32_t kStopPerCell = 640, kLeastPerCell = 1024;
// The least photons of a run in rounds: below, the end takes them all (faster_in_cells has what decides above it).
constexpr uint64_t kMinPhotons = 2000000;
// The rounds of a run are no more than this (16 000 launches, 45 ms if all are empty).
constexpr double kMaxRounds = 4000.0;

struct Grid {                              // device copy of CellDims
    int32_t ncx, ncy, ncz, ex, ey, ez, zlo;
    uint32_t base;                         // first cell key of the job
    uint32_t qx, qy, qz;                   // ceil(2^32 / e): v / e = umulhi(v, q) for v < 2^17, e <= kCell (q = 0: e = 1)
};

struct Ctrl {
    unsigned long long next_id;            // next queue position to launch
    unsigned long long total;              // queue positions
    uint32_t n_items, item_cursor;
    uint32_t alive, done;
    uint32_t stop_at;                      // rounds end once no more photons than this (and kStopPerCell a cell) are worth one
    unsigned long long tail_next;
    uint32_t n_jobs, n_cells, slots, walkers;   // walkers: workgroups of the walk
};

struct Item { uint32_t cell, begin, end, pad; };

// ---------------------------------------------------------------------------
// Photon in a lane and in a slot
// ---------------------------------------------------------------------------
template <typename R>
struct CellPhoton {
    using Real = R;
    R fx, fy, fz, ux, uy, uz, iux, iuy, iuz;
    R bx, by, bz;              // far face per axis: 1 where u > 0, else 0
    R nx, ny, nz;              // near face per axis (offset on entering the next voxel): 1 - b
    int32_t sx, sy, sz;        // byte step in the cell per axis
    double s_rem, l_void, l_tot, score_g, l_opt;
    uint32_t w, k, steps, pid, nf;
    R wq;                      // weight in quanta per voxel length
    U4 fr;
};

template <typename R>
__device__ __forceinline__ void set_faces(CellPhoton<R> &p)
{
    const bool px = p.ux > (R)0, py = p.uy > (R)0, pz = p.uz > (R)0;
    p.bx = px ? (R)1 : (R)0; p.nx = px ? (R)0 : (R)1; p.sx = px ? 4 : -4;
    p.by = py ? (R)1 : (R)0; p.ny = py ? (R)0 : (R)1; p.sy = py ? 4 * kRow : -4 * kRow;
    p.bz = pz ? (R)1 : (R)0; p.nz = pz ? (R)0 : (R)1; p.sz = pz ? 4 * kLayer : -4 * kLayer;
}

template <typename R> __device__ __forceinline__ void set_direction(CellPhoton<R> &p, R ux, R uy, R uz)
{
    p.ux = ux;
    p.uy = uy;
    p.uz = uz;
    // 1/0 = +inf: the distance along an axis the photon does not move on is then +inf, or NaN (0 x inf)
    // on a face, which the minimum over the axes passes over
    p.iux = r_rcp(fabs(ux));
    p.iuy = r_rcp(fabs(uy));
    p.iuz = r_rcp(fabs(uz));
    set_faces(p);
}

template <typename R> __device__ __forceinline__ void set_weight(CellPhoton<R> &p, uint32_t w)
{
    p.w = w;
    p.wq = (R)w * (R)(1.0 / (1 << kDepositShift));
}

// Words of a slot, in 16-byte units.
template <typename R, bool GENERAL, bool GRAD> constexpr int slot_quads()
{
    return (std::is_same<R, float>::value ? 4 : 6) + (GENERAL ? 1 : 0) + (GRAD ? 1 : 0);
}

__device__ __forceinline__ uint32_t lo32(double x) { return (uint32_t)__double_as_longlong(x); }
__device__ __forceinline__ uint32_t hi32(double x) { return (uint32_t)((uint64_t)__double_as_longlong(x) >> 32); }
__device__ __forceinline__ double mk64(uint32_t lo, uint32_t hi)
{
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

template <typename R, bool GENERAL, bool GRAD, class P>
__device__ __forceinline__ void store_slot(uint4 *s, const P &p, int32_t ix, int32_t iy, int32_t iz)
{
    int q = 0;
    const uint32_t xy = (uint32_t)ix | ((uint32_t)iy << 16);
    if constexpr (std::is_same<R, float>::value) {
        s[q++] = make_uint4(xy, (uint32_t)iz, __float_as_uint(p.fx), __float_as_uint(p.fy));
        s[q++] = make_uint4(__float_as_uint(p.fz), __float_as_uint(p.ux), __float_as_uint(p.uy), __float_as_uint(p.uz));
        s[q++] = make_uint4(lo32(p.s_rem), hi32(p.s_rem), lo32(p.l_void), hi32(p.l_void));
        s[q++] = make_uint4(p.w, p.k, p.steps, p.pid);
    } else {
        s[q++] = make_uint4(xy, (uint32_t)iz, p.w, p.k);
        s[q++] = make_uint4(p.steps, p.pid, lo32(p.fx), hi32(p.fx));
        s[q++] = make_uint4(lo32(p.fy), hi32(p.fy), lo32(p.fz), hi32(p.fz));
        s[q++] = make_uint4(lo32(p.ux), hi32(p.ux), lo32(p.uy), hi32(p.uy));
        s[q++] = make_uint4(lo32(p.uz), hi32(p.uz), lo32(p.s_rem), hi32(p.s_rem));
        s[q++] = make_uint4(lo32(p.l_void), hi32(p.l_void), 0u, 0u);
    }
    if constexpr (GENERAL) s[q++] = make_uint4(lo32(p.l_opt), hi32(p.l_opt), p.nf, 0u);
    if constexpr (GRAD) s[q++] = make_uint4(lo32(p.l_tot), hi32(p.l_tot), lo32(p.score_g), hi32(p.score_g));
}

// Everything but the direction's derived terms; the direction comes back in u.
template <typename R, bool GENERAL, bool GRAD, class P>
__device__ __forceinline__ void load_slot(const uint4 *s, P &p, int32_t &ix, int32_t &iy, int32_t &iz, const Job &J)
{
    R ux, uy, uz;
    int q = 0;
    if constexpr (std::is_same<R, float>::value) {
        const uint4 a = s[0], b = s[1], c = s[2], d = s[3];
        q = 4;
        ix = (int32_t)(a.x & 0xFFFFu);
        iy = (int32_t)(a.x >> 16);
        iz = (int32_t)a.y;
        p.fx = __uint_as_float(a.z);
        p.fy = __uint_as_float(a.w);
        p.fz = __uint_as_float(b.x);
        ux = __uint_as_float(b.y);
        uy = __uint_as_float(b.z);
        uz = __uint_as_float(b.w);
        p.s_rem = mk64(c.x, c.y);
        p.l_void = mk64(c.z, c.w);
        p.w = d.x;
        p.k = d.y;
        p.steps = d.z;
        p.pid = d.w;
    } else {
        const uint4 a = s[0], b = s[1], c = s[2], d = s[3], e = s[4], f = s[5];
        q = 6;
        ix = (int32_t)(a.x & 0xFFFFu);
        iy = (int32_t)(a.x >> 16);
        iz = (int32_t)a.y;
        p.w = a.z;
        p.k = a.w;
        p.steps = b.x;
        p.pid = b.y;
        p.fx = mk64(b.z, b.w);
        p.fy = mk64(c.x, c.y);
        p.fz = mk64(c.z, c.w);
        ux = mk64(d.x, d.y);
        uy = mk64(d.z, d.w);
        uz = mk64(e.x, e.y);
        p.s_rem = mk64(e.z, e.w);
        p.l_void = mk64(f.x, f.y);
    }
    p.l_opt = 0.0;
    p.l_tot = 0.0;
    p.score_g = 0.0;
    p.nf = 0u;
    if constexpr (GENERAL) {
        const uint4 g = s[q++];
        p.l_opt = mk64(g.x, g.y);
        p.nf = g.z;
        // the Fresnel words not drawn yet, as fresnel_uniform leaves them
        const uint32_t drawn = p.nf & 3u;
        if (J.fresnel && drawn != 0u) {
            p.fr = philox4x32_10(U4{p.nf >> 2, p.pid, J.stream_id, 4u}, J.key0, J.key1);
            p.fr.x = drawn == 1u ? p.fr.y : (drawn == 2u ? p.fr.z : p.fr.w);
            p.fr.y = drawn == 1u ? p.fr.z : p.fr.w;
            p.fr.z = p.fr.w;
        }
    }
    if constexpr (GRAD) {
        const uint4 g = s[q++];
        p.l_tot = mk64(g.x, g.y);
        p.score_g = mk64(g.z, g.w);
    }
    set_direction(p, ux, uy, uz);
}

__device__ __forceinline__ uint32_t cell_quotient(uint32_t v, uint32_t q) { return q ? __umulhi(v, q) : v; }

__device__ __forceinline__ uint32_t cell_key(const Grid &G, int32_t ix, int32_t iy, int32_t iz)
{
    const uint32_t cx = cell_quotient((uint32_t)ix, G.qx), cy = cell_quotient((uint32_t)iy, G.qy);
    const uint32_t cz = cell_quotient((uint32_t)(iz - G.zlo), G.qz);
    return G.base + (cz * (uint32_t)G.ncy + cy) * (uint32_t)G.ncx + cx;
}

// A struct every lane of the wavefront reads alike, into scalar registers: the loops that use
// its fields would otherwise reload them after each store and atomic.
template <class S> __device__ __forceinline__ void load_uniform(S &dst, const S *src)
{
    constexpr int n = sizeof(S) / 4;
    uint32_t w[n];
#pragma unroll
    for (int i = 0; i < n; ++i) w[i] = __builtin_amdgcn_readfirstlane(((const uint32_t *)src)[i]);
    __builtin_memcpy(&dst, w, sizeof(S));
}

__device__ __forceinline__ uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }
__device__ __forceinline__ bool lanes(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
__device__ __forceinline__ int32_t popcount(uint64_t m) { return (int32_t)__builtin_popcountll(m); }

// Zero, in a vector register the compiler cannot see through: an LDS address that holds it
// counts as different in each lane, so that an add by a few lanes stays one instruction instead
// of a loop that first sums the lanes.
__device__ __forceinline__ int32_t opaque_zero()
{
    int32_t z = 0;
    asm volatile("" : "+v"(z));
    return z;
}

// ---------------------------------------------------------------------------
// Between two rounds: launch photons into free slots, sort the slots by cell
// ---------------------------------------------------------------------------
struct Tables {
    const Job *jobs;
    const Grid *grids;
    Ctrl *ctrl;
    uint32_t *count;       // [cells] photons per cell
    uint32_t *block_base;  // [kSortBlocks][cells] a block's photons per cell, then those of the blocks before it
    Item *items;
    uint32_t *keys;        // [slots] cell of the slot's photon, kDead: free
    uint32_t *list;        // [slots] slots ordered by cell
    uint4 *slots;
};

__device__ __forceinline__ int32_t job_of_queue(const Job *jobs, int32_t n, uint64_t q)
{
    int32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (jobs[mid].queue_begin <= q) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ int32_t job_of_cell(const Grid *grids, int32_t n, uint32_t cell)
{
    int32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (grids[mid].base <= cell) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Inclusive scan over the block (1024 threads) of one value per thread.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *part)
{
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(v, o);
        if (lane >= (uint32_t)o) v += u;
    }
    if (lane == 63u) part[wave] = v;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t i = 0; i < wave; ++i) before += part[i];
    __syncthreads();
    return v + before;
}

// Keys in flight per thread, in uint4.
constexpr int kKeyLoads = 4;

// The keys of a block's slots, kKeyLoads uint4 at a time; f(key, slot) for each.
template <class F>
__device__ __forceinline__ void for_keys(const uint32_t *keys, uint32_t begin, uint32_t end, F f)
{
    const uint4 none = make_uint4(kDead, kDead, kDead, kDead);
    for (uint32_t t = begin + 4u * threadIdx.x; t < end; t += 4u * kSortThreads * kKeyLoads) {
        uint4 k4[kKeyLoads];
#pragma unroll
        for (int l = 0; l < kKeyLoads; ++l) {
            const uint32_t i = t + 4u * kSortThreads * (uint32_t)l;
            k4[l] = i < end ? *(const uint4 *)(keys + i) : none;
        }
#pragma unroll
        for (int l = 0; l < kKeyLoads; ++l) {
            const uint32_t i = t + 4u * kSortThreads * (uint32_t)l;
            if (i < end) {
                f(k4[l].x, i);
                f(k4[l].y, i + 1u);
                f(k4[l].z, i + 2u);
                f(k4[l].w, i + 3u);
            }
        }
    }
}

template <typename R, bool GENERAL, bool GRAD>
__global__ __launch_bounds__(kSortThreads) void k_cells_count(Tables T, uint32_t room)
{
    extern __shared__ uint32_t s_hist[];                   // [cells], then room for the free slots: uint16 offsets
    __shared__ uint32_t s_nd;
    __shared__ unsigned long long s_base;
    Ctrl *c = T.ctrl;
    if (c->done != 0u) {
        if (blockIdx.x == 0 && threadIdx.x == 0) c->done = 2u;
        return;
    }
    const uint32_t cells = c->n_cells, slots = c->slots;
    const uint32_t per = (slots / kSortBlocks + 4u) & ~3u;   // whole uint4 of keys
    const uint32_t begin = min(slots, blockIdx.x * per), end = min(slots, begin + per);
    const uint64_t total = c->total;
    uint16_t *s_free = (uint16_t *)(s_hist + cells);
    for (uint32_t i = threadIdx.x; i < cells; i += kSortThreads) s_hist[i] = 0u;
    if (threadIdx.x == 0) s_nd = 0u;
    __syncthreads();
    const bool feed = __hip_atomic_load(&c->next_id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < total;
    for_keys(T.keys, begin, end, [&](uint32_t key, uint32_t i) {
        if (key != kDead) {
            atomicAdd(&s_hist[key], 1u);
        } else if (feed) {
            // free slots beyond the room wait for the next pass
            const uint32_t n = atomicAdd(&s_nd, 1u);
            if (n < room) s_free[n] = (uint16_t)(i - begin);
        }
    });
    __syncthreads();
    const uint32_t nd = min(s_nd, room);
    if (threadIdx.x == 0) {
        s_base = ~0ull;
        if (nd != 0u && __hip_atomic_load(&c->next_id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < total)
            s_base = atomicAdd(&c->next_id, (unsigned long long)nd);
    }
    __syncthreads();
    const uint64_t base = s_base;
    if (base < total) {
        const int32_t n_jobs = (int32_t)c->n_jobs;
        Job J;
        Grid G;
        load_uniform(J, T.jobs);
        load_uniform(G, T.grids);
        for (uint32_t i = threadIdx.x; i < nd; i += kSortThreads) {
            const uint64_t q = base + i;
            if (q >= total) continue;
            if (n_jobs > 1) {
                const int32_t j = job_of_queue(T.jobs, n_jobs, q);
                J = T.jobs[j];
                G = T.grids[j];
            }
            Photon<R> p;
            launch_state<GENERAL>(p, J, (uint32_t)(J.photon_begin + (q - J.queue_begin)));
            const uint32_t slot = begin + s_free[i];
            store_slot<R, GENERAL, GRAD>(T.slots + (size_t)slot * slot_quads<R, GENERAL, GRAD>(), p, p.ix, p.iy, p.iz);
            const uint32_t key = cell_key(G, p.ix, p.iy, p.iz);
            T.keys[slot] = key;
            atomicAdd(&s_hist[key], 1u);
        }
    }
    __syncthreads();
    uint32_t *row = T.block_base + (size_t)blockIdx.x * cells;
    for (uint32_t i = threadIdx.x; i < cells; i += kSortThreads) row[i] = s_hist[i];
}

// Per cell, the exclusive sums of its blocks' counts down the blocks, in place, and their total.  A
// workgroup takes 64 cells, each wavefront kSortBlocks / 16 rows of them.
__global__ __launch_bounds__(kSortThreads) void k_cells_columns(Tables T)
{
    constexpr int kRows = kSortBlocks / (kSortThreads / 64);
    __shared__ uint32_t s_sum[kSortThreads / 64][64];
    const Ctrl *c = T.ctrl;
    if (c->done == 2u) return;
    const uint32_t cells = c->n_cells;
    const uint32_t cell = blockIdx.x * 64u + (threadIdx.x & 63u), wave = threadIdx.x >> 6;
    uint32_t *col = T.block_base + (size_t)wave * kRows * cells + cell;
    uint32_t v[kRows], sum = 0u;
#pragma unroll
    for (int r = 0; r < kRows; ++r) v[r] = cell < cells ? col[(size_t)r * cells] : 0u;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const uint32_t x = v[r];
        v[r] = sum;
        sum += x;
    }
    s_sum[wave][threadIdx.x & 63u] = sum;
    __syncthreads();
    uint32_t before = 0u;
    for (uint32_t w = 0; w < wave; ++w) before += s_sum[w][threadIdx.x & 63u];
    if (cell < cells) {
#pragma unroll
        for (int r = 0; r < kRows; ++r) col[(size_t)r * cells] = v[r] + before;
        if (wave == kSortThreads / 64 - 1) T.count[cell] = before + sum;
    }
}

// Size class of an item of n <= W photons, 0 the largest.
constexpr uint32_t kClasses = 32;
__device__ __forceinline__ uint32_t item_class(uint32_t n, uint32_t W) { return (uint32_t)((uint64_t)(W - n) * kClasses / W); }

// Each block orders the cells for itself (a scan of their totals), then writes its slots' numbers
// into the list; block 0 also cuts the list into the walk's items.
__global__ __launch_bounds__(kSortThreads) void k_cells_scatter(Tables T, int32_t force)
{
    extern __shared__ uint32_t s_hist[];
    __shared__ uint32_t s_part[kSortThreads / 64], s_alive, s_class[kClasses], s_used, s_cells;
    Ctrl *c = T.ctrl;
    if (c->done == 2u) return;
    const uint32_t cells = c->n_cells, slots = c->slots;
    const uint32_t per = (slots / kSortBlocks + 4u) & ~3u;   // whole uint4 of keys
    const uint32_t begin = min(slots, blockIdx.x * per), end = min(slots, begin + per);
    const uint32_t cpt = (cells + kSortThreads - 1) / kSortThreads;
    const uint32_t c0 = min(cells, threadIdx.x * cpt), c1 = min(cells, c0 + cpt);
    uint32_t mine = 0u;
    for (uint32_t i = c0; i < c1; ++i) mine += T.count[i];
    const uint32_t first = block_scan(mine, s_part) - mine;
    if (threadIdx.x == kSortThreads - 1) s_alive = first + mine;
    uint32_t off = first;
    for (uint32_t i = c0; i < c1; ++i) {
        s_hist[i] = off;
        off += T.count[i];
    }
    __syncthreads();
    const uint32_t alive = s_alive;
    if (blockIdx.x == 0) {
        // photons per item: a workgroup's even share, so about one full item each, and what is left of each cell
        const uint32_t W = min(max(alive / c->walkers, kMinItem), kMaxItem);
        // the items by size, largest first: each workgroup of the walk takes the next one when it is
        // done with its last, and the short ones even out the end
        // a cell with few photons lets them wait until there are more: taking it costs a workgroup as much
        // time as some 1000 visits.  At least half of the photons are in cells that are taken.
        const uint32_t least = min(kLeastPerCell, alive / (2u * cells));
        uint32_t mine_used = 0u, mine_cells = 0u;
        if (threadIdx.x < kClasses) s_class[threadIdx.x] = 0u;
        if (threadIdx.x == 0) s_used = s_cells = 0u;
        __syncthreads();
        for (uint32_t i = c0; i < c1; ++i) {
            const uint32_t k = T.count[i];
            if (k < least) continue;
            mine_used += k;
            ++mine_cells;
            if (k >= W) atomicAdd(&s_class[0], k / W);
            if (k % W) atomicAdd(&s_class[item_class(k % W, W)], 1u);
        }
        if (mine_cells) {
            atomicAdd(&s_used, mine_used);
            atomicAdd(&s_cells, mine_cells);
        }
        __syncthreads();
        uint32_t n_items = 0u;
        if (threadIdx.x == 0)
            for (uint32_t j = 0; j < kClasses; ++j) {
                const uint32_t k = s_class[j];
                s_class[j] = n_items;
                n_items += k;
            }
        __syncthreads();
        off = first;
        for (uint32_t i = c0; i < c1; ++i) {
            uint32_t k = T.count[i];
            if (k < least) {
                off += k;
                continue;
            }
            while (k != 0u) {
                const uint32_t n = min(k, W);
                T.items[atomicAdd(&s_class[item_class(n, W)], 1u)] = Item{i, off, off + n, 0u};
                off += n;
                k -= n;
            }
        }
        if (threadIdx.x == 0) {
            const bool stop = force || (c->next_id >= c->total && s_used <= c->stop_at + kStopPerCell * s_cells);
            c->alive = alive;
            c->n_items = stop ? 0u : n_items;
            c->item_cursor = 0u;
            if (stop) c->done = 1u;
        }
    }
    const uint32_t *row = T.block_base + (size_t)blockIdx.x * cells;
    for (uint32_t i = threadIdx.x; i < cells; i += kSortThreads) s_hist[i] += row[i];
    __syncthreads();
    for_keys(T.keys, begin, end, [&](uint32_t key, uint32_t i) {
        if (key != kDead) T.list[atomicAdd(&s_hist[key], 1u)] = i;
    });
}

// ---------------------------------------------------------------------------
// The walk inside a cell
// ---------------------------------------------------------------------------
// Score bins of a cell, int32 words in LDS moved to the global pair before they can overflow
// (see score.hpp): with 1024 threads to a workgroup the direct path starts at 2^20, so
// |word| < 2^28 + 1024 * 2^20.
constexpr long long kCellGradDirect = 1ll << 20;

__device__ __forceinline__ void cell_grad_add(int *bin, unsigned long long *grad, int32_t i, long long v)
{
    if (v == 0) return;
    if (v >= kCellGradDirect || v <= -kCellGradDirect) {
        grad_global_add(grad, i, v);
        return;
    }
    const long long nv = (long long)atomicAdd(bin, (int)v) + v;
    if (nv >= kGradSpill || nv <= -kGradSpill) grad_global_add(grad, i, (long long)atomicExch(bin, 0));
}

// Lanes parked before an exchange; once an item's list is used up, iterations a wavefront still
// takes, and the lanes it needs busy to go on after that.
constexpr int32_t kRefill = 16, kCutAfter = 16, kCutLanes = 32;

// Lanes that wait before their interactions run: the wait takes half of them from the steps
// and an interaction's code then runs for that many, so the best number goes with the root of
// the rate of interactions.  256^3, a fixed 20 against 28 sqrt(mu_t) (20 at mu_t = 0.51): mu_t
// 0.037 (paper's model) 108.5 -> 104.6 ms, 0.21 61.8 -> 60.7, 1.03 51.2 -> 50.3.
constexpr float kDeferScale = 28.0f;

// bits below the quanta in a tally word
constexpr uint32_t kSolid = 1u, kOutside = 2u, kSpecial = 4u;  // special: outside -> mirror, inside -> air pad

// A photon's terminal outcome into the workgroup's channels (LDS).  The weight absorbed
// and the roulette balance are counted as they happen.
template <class P>
__device__ __forceinline__ void cell_account(unsigned long long *acc, const P &p, int32_t ev, int32_t nz)
{
    acc += opaque_zero();
    if (ev == EV_ESC_R || ev == EV_ESC_T) {
        atomicAdd(&acc[ev == EV_ESC_R ? MC_S_R : MC_S_T], (unsigned long long)p.w);
        atomicAdd(&acc[MC_S_ESC_W], (unsigned long long)p.w);
        atomicAdd(&acc[MC_S_ESC_N], 1ull);
        if (p.l_void > (double)nz) {
            atomicAdd(&acc[MC_S_ESC_W_GTL], (unsigned long long)p.w);
            atomicAdd(&acc[MC_S_ESC_N_GTL], 1ull);
        }
        const unsigned long long vp = __double2ull_rn((double)p.w * p.l_void);
        atomicAdd(&acc[MC_S_ESC_W_VOID_PATH], vp & 0xFFFFFFFFull);
        if (vp >> 32) atomicAdd(&acc[MC_S_ESC_W_VOID_PATH_HI], vp >> 32);
    } else if (ev == EV_LOST) {
        atomicAdd(&acc[MC_S_LOST], (unsigned long long)p.w);
    } else if (ev == EV_GATED) {
        atomicAdd(&acc[MC_S_GATED], (unsigned long long)p.w);
    }
    atomicAdd(&acc[MC_S_STEPS], (unsigned long long)p.steps);
    atomicAdd(&acc[MC_S_INTERACTIONS], (unsigned long long)p.k);
    atomicAdd(&acc[MC_S_LAUNCHED], 1ull);
}

__device__ __forceinline__ void esc_add(const BatchEsc *esc, int32_t job, double l_void, uint32_t w)
{
    const BatchEsc &e = esc[job];
    if (e.w == nullptr) return;
    const size_t b = (size_t)(blockIdx.x % kEscReplicas) * kEscMaxBins + (size_t)escape_path_bin(l_void, e.width, e.nbins);
    __hip_atomic_fetch_add(e.rw + b, (unsigned long long)w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(e.rn + b, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The escape histogram of a run of one job (HIST), a workgroup's in LDS: where most photons leave by a few bins the adds to
// their copies in memory take longer than the walk (512 x 512 x 8, 2e6 photons, bins of 8 voxels: 2.35 ms; 1.06).
// A batch, whose workgroups go from job to job, adds to the copies.
template <bool HIST> struct EscBins {
    unsigned long long w[HIST ? kEscMaxBins : 1];
    unsigned int n[HIST ? kEscMaxBins : 1];          // a workgroup's photons, fewer than 2^32
};

template <bool HIST> __device__ __forceinline__ void esc_clear(EscBins<HIST> &s)
{
    if (HIST)
        for (int32_t i = threadIdx.x; i < kEscMaxBins; i += blockDim.x) {
            s.w[i] = 0ull;
            s.n[i] = 0u;
        }
}

template <bool HIST>
__device__ __forceinline__ void esc_count(EscBins<HIST> &s, const BatchEsc *esc, int32_t job, double l_void, uint32_t w)
{
    if (HIST) {
        const int32_t b = escape_path_bin(l_void, esc->width, esc->nbins);
        atomicAdd(&s.w[b], (unsigned long long)w);
        atomicAdd(&s.n[b], 1u);
    } else if (esc != nullptr) {
        esc_add(esc, job, l_void, w);
    }
}

// The workgroup's bins into one of the copies; every thread's counts are in.
template <bool HIST> __device__ __forceinline__ void esc_flush(const EscBins<HIST> &s, const BatchEsc *esc)
{
    if (HIST)
        for (int32_t i = threadIdx.x; i < esc->nbins; i += blockDim.x)
            if (s.n[i]) {
                const size_t b = (size_t)(blockIdx.x % kEscReplicas) * kEscMaxBins + (size_t)i;
                __hip_atomic_fetch_add(esc->rw + b, s.w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_add(esc->rn + b, (unsigned long long)s.n[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
}

// Threads of a workgroup, the one its compute unit holds: the FP64 transport's state needs more than
// the 128 registers 16 wavefronts leave each lane.
template <typename R> constexpr int walk_block() { return std::is_same<R, float>::value ? 1024 : 512; }

template <typename R, bool GENERAL, bool GRAD, bool HIST>
__global__ __launch_bounds__(walk_block<R>()) void k_cells_walk(Tables T, unsigned long long *__restrict__ grad,
                                                       const BatchEsc *__restrict__ esc)
{
    constexpr int SH = GENERAL ? 3 : 2;                      // flag bits of a tally word
    constexpr int NQ = slot_quads<R, GENERAL, GRAD>();
    constexpr int kBlock = walk_block<R>();
    __shared__ __align__(16) uint32_t tally[kWords];
    __shared__ unsigned long long acc[MC_NSCALARS];
    __shared__ uint32_t s_item, s_cursor;
    __shared__ int s_grad[GRAD ? 6 * kCell : 1];
    __shared__ EscBins<HIST> s_esc;
    const uint32_t lane = __lane_id();
    Ctrl *c = T.ctrl;
    const uint32_t n_items = c->n_items;
    int32_t cur_job = -1;
    if (threadIdx.x < MC_NSCALARS) acc[threadIdx.x] = 0ull;
    esc_clear(s_esc);
    uint64_t absorbed = 0ull;

    auto cell_word = [&](uint32_t lb) -> uint32_t { return *(const uint32_t *)__builtin_assume_aligned((const char *)tally + lb, 4); };

    for (;;) {
        __syncthreads();                                     // the last item's flush has read the tally
        if (threadIdx.x == 0) {
            s_item = atomicAdd(&c->item_cursor, 1u);
            s_cursor = 0u;
        }
        __syncthreads();
        const uint32_t item = __builtin_amdgcn_readfirstlane(s_item);
        if (item >= n_items) break;
        const Item it = T.items[item];
        const uint32_t cell = __builtin_amdgcn_readfirstlane(it.cell);
        const uint32_t n_ph = __builtin_amdgcn_readfirstlane(it.end - it.begin);
        const uint32_t *list = T.list + __builtin_amdgcn_readfirstlane(it.begin);
        const int32_t job = __builtin_amdgcn_readfirstlane(job_of_cell(T.grids, (int32_t)c->n_jobs, cell));
        Job J;
        Grid G;
        load_uniform(J, T.jobs + job);
        load_uniform(G, T.grids + job);
        if (job != cur_job) {
            // the channels so far belong to the job before
            if (cur_job >= 0) {
                const unsigned long long a = absorbed;
                if (a) atomicAdd(&acc[MC_S_A], a);
                absorbed = 0ull;
                __syncthreads();
                if (threadIdx.x < MC_NSCALARS) {
                    const unsigned long long v = acc[threadIdx.x];
                    if (v) atomicAdd((unsigned long long *)&T.jobs[cur_job].scalars[threadIdx.x], v);
                    acc[threadIdx.x] = 0ull;
                }
            }
            cur_job = job;
        }
        const uint32_t lc = cell - G.base;
        const int32_t cx = (int32_t)(lc % (uint32_t)G.ncx);
        const int32_t cy = (int32_t)((lc / (uint32_t)G.ncx) % (uint32_t)G.ncy);
        const int32_t cz = (int32_t)(lc / ((uint32_t)G.ncx * (uint32_t)G.ncy));
        const int32_t x0 = cx * G.ex, y0 = cy * G.ey, z0 = cz * G.ez + G.zlo;
        const int32_t zend = J.nz - G.zlo;                   // one past the last layer walked in
        const int32_t ex = min(G.ex, J.nx - x0), ey = min(G.ey, J.ny - y0), ez = min(G.ez, zend - z0);

        // the cell's mask and flags, the tally zero: 17 pairs of columns per row of voxels, kPairs of
        // them per thread at a time with their loads issued together
        constexpr int kPairs = GENERAL || GRAD ? 3 : 5;
        for (uint32_t i0 = threadIdx.x; i0 < (uint32_t)(kWords / 2); i0 += kPairs * kBlock) {
            uint64_t b[kPairs][2];
            uint32_t at[kPairs][2], code[kPairs][2];
#pragma unroll
            for (int j = 0; j < kPairs; ++j) {
                const uint32_t i = i0 + (uint32_t)(j * kBlock);
                const uint32_t row = i / (uint32_t)(kSide / 2);
                const int32_t hx = 2 * (int32_t)(i - row * (uint32_t)(kSide / 2));
                const int32_t hz = (int32_t)(row / (uint32_t)kSide), hy = (int32_t)(row - (uint32_t)hz * (uint32_t)kSide);
                const int32_t gy0 = y0 + hy - 1, gz = z0 + hz - 1;
                const bool row_in = hy >= 1 && hy <= ey && hz >= 1 && hz <= ez;
                // rows past the halo are never entered; their words read some voxel of the volume
                const int32_t gy = gy0 < 0 ? J.ny - 1 : (gy0 >= J.ny ? 0 : gy0);
                const bool mask_row = gz >= 0 && gz < J.nz;
                const int32_t gzc = mask_row ? gz : 0;
                const uint32_t row_brick = brick_of(J, 0, gy, gzc);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int32_t h = hx + k, gx0 = x0 + h - 1;
                    const bool inside = row_in && h >= 1 && h <= ex;
                    uint32_t f = inside ? 0u : kOutside;
                    if (GENERAL) {
                        if (J.lateral && (gy0 < 0 || gy0 >= J.ny || gx0 < 0 || gx0 >= J.nx)) f |= kSpecial;
                        else if (inside && !mask_row) f |= kSpecial;
                    }
                    const int32_t gx = gx0 < 0 ? J.nx - 1 : (gx0 >= J.nx ? 0 : gx0);
                    b[j][k] = J.bricks[row_brick + (uint32_t)(gx >> 2)];
                    at[j][k] = bit_of(gx, gy, gzc);
                    code[j][k] = mask_row ? f | kSolid : f;    // cleared below where the mask has a pore
                }
            }
#pragma unroll
            for (int j = 0; j < kPairs; ++j) {
                const uint32_t i = i0 + (uint32_t)(j * kBlock);
                uint2 w;
                w.x = ((b[j][0] >> at[j][0]) & 1ull) ? code[j][0] & ~kSolid : code[j][0];
                w.y = ((b[j][1] >> at[j][1]) & 1ull) ? code[j][1] & ~kSolid : code[j][1];
                if (i < (uint32_t)(kWords / 2)) ((uint2 *)tally)[i] = w;
            }
        }
        if (GRAD)
            for (int32_t i = threadIdx.x; i < 6 * kCell; i += kBlock) s_grad[i] = 0;
        __syncthreads();

        CellPhoton<R> p;
        uint32_t lb = 0u, cw = 0u, slot = 0u;                // byte offset and word of the photon's voxel, its slot
        int32_t end = 0;                                     // the event of a photon that ended
        // lanes that hold a photon, that run, that wait at an interaction point; a photon that does neither
        // is parked until the next exchange: ended, at its step cap, or outside the cell
        uint64_t have = 0ull, run = 0ull, wait = 0ull;
        bool drained = false;                                // the item's list is used up
        int32_t since = 0;                                   // iterations since then
        const int32_t defer = min(max((int32_t)(kDeferScale * sqrtf((float)J.mu_t)), 2), 32);
        // lanes of each wavefront in use: few photons are spread over all wavefronts
        const int32_t cap = (int32_t)min(64u, (n_ph + (kBlock / 64) - 1) / (kBlock / 64));

        for (;;) {
            run &= ballot((cw & kOutside) == 0u && p.steps < J.max_steps);
            int32_t step = 0;                                // to the next voxel's word; 0: none is entered
            if (lanes(run)) {
                const R dx = fabs(p.bx - p.fx) * p.iux, dy = fabs(p.by - p.fy) * p.iuy, dz = fabs(p.bz - p.fz) * p.iuz;
                const R d_face = fmin(fmin(dx, dy), dz);
                // the face axis is the first minimum in x, y, z order
                const uint64_t m0 = ballot(dx == d_face), m1 = ballot(dy == d_face) & ~m0, m2 = ~(m0 | m1);
                const uint64_t in_solid = ballot((cw & kSolid) != 0u);
                const bool solid = lanes(in_solid);
                uint64_t hit = ballot(p.s_rem <= (double)d_face) & in_solid;
                R d = lanes(hit) ? (R)p.s_rem : d_face;
                uint64_t stay = hit;
                bool in_slab = true;
                double n_here = 1.0;
                if constexpr (GENERAL) {
                    in_slab = (cw & kSpecial) == 0u;
                    n_here = solid ? (double)J.n_solid : 1.0;
                    // the optical path may reach the gate, not pass it
                    const bool gated = p.l_opt + n_here * (double)d > J.gate;
                    if (gated) {
                        d = (R)fmax((J.gate - p.l_opt) / n_here, 0.0);
                        end = EV_GATED;
                    }
                    stay |= ballot(gated);
                }
                if constexpr (GRAD) {
                    if (in_slab) {
                        const int32_t lz = (int32_t)((lb / 4u) / (uint32_t)kLayer) - 1;
                        long long vs, va, vg;
                        grad_values(p, J.mu_s > 0.0 ? 1.0 / J.mu_s : 0.0, (double)d, solid, vs, va, vg);
                        const int32_t lbase = (solid ? 0 : kCell) + lz, gbase = (solid ? 0 : J.nz) + z0 + lz;
                        cell_grad_add(s_grad + lbase, grad, gbase, vs);
                        cell_grad_add(s_grad + 2 * kCell + lbase, grad, 2 * J.nz + gbase, va);
                        cell_grad_add(s_grad + 4 * kCell + lbase, grad, 4 * J.nz + gbase, vg);
                    }
                }
                uint32_t old = 0u, inc = 0u;
                const uint32_t here = lb;
                if (!GENERAL || in_slab) {
                    // a segment inside one voxel is shorter than 2 voxel lengths: its quanta fit 25 bits
                    inc = (uint32_t)rint(p.wq * d) << SH;
                    old = __hip_atomic_fetch_add((uint32_t *)__builtin_assume_aligned((char *)tally + lb, 4), inc,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    // s_rem -= d in the solid, l_void += d in a pore: the products are exact
                    p.s_rem = fma((double)d, solid ? -1.0 : 0.0, p.s_rem);
                    p.l_void = fma((double)d, solid ? 0.0 : 1.0, p.l_void);
                    if constexpr (GRAD) p.l_tot += (double)d;
                }
                if constexpr (GENERAL) p.l_opt += n_here * (double)d;
                p.steps += 1u;
                const R ax = clamp01(p.fx + p.ux * d), ay = clamp01(p.fy + p.uy * d), az = clamp01(p.fz + p.uz * d);
                step = lanes(stay) ? 0 : (lanes(m0) ? p.sx : (lanes(m1) ? p.sy : p.sz));
                if constexpr (!GENERAL) {
                    lb += (uint32_t)step;
                    cw = cell_word(lb);
                    p.fx = lanes(m0 & ~stay) ? p.nx : ax;
                    p.fy = lanes(m1 & ~stay) ? p.ny : ay;
                    p.fz = lanes(m2 & ~stay) ? p.nz : az;
                } else {
                    const uint32_t next = cell_word(lb + (uint32_t)step);
                    const bool next_solid = (next & kSolid) != 0u;
                    p.fx = ax;
                    p.fy = ay;
                    p.fz = az;
                    if (step != 0) {
                        const bool a0 = lanes(m0), a1 = lanes(m1), a2 = lanes(m2), up = step > 0;
                        bool reflect = (next & (kOutside | kSpecial)) == (kOutside | kSpecial);
                        if (!reflect && J.fresnel && next_solid != solid) {
                            const R ua = a0 ? p.ux : (a1 ? p.uy : p.uz);
                            const R n1 = solid ? (R)J.n_solid : (R)1, n2 = next_solid ? (R)J.n_solid : (R)1;
                            R ct;
                            const R rf = fresnel(n1, n2, fabs(ua), &ct);
                            if (rf >= (R)1 || fresnel_uniform(p, J) < rf) {
                                reflect = true;
                            } else {
                                const R eta = r_div(n1, n2), ctn = up ? ct : -ct;
                                set_direction(p, a0 ? ctn : eta * p.ux, a1 ? ctn : eta * p.uy, a2 ? ctn : eta * p.uz);
                            }
                        }
                        // on the far face of this voxel if reflected, on the near face of the next one else
                        const R face = reflect == up ? (R)1 : (R)0;
                        p.fx = a0 ? face : p.fx;
                        p.fy = a1 ? face : p.fy;
                        p.fz = a2 ? face : p.fz;
                        if (reflect) {
                            p.ux = a0 ? -p.ux : p.ux;
                            p.uy = a1 ? -p.uy : p.uy;
                            p.uz = a2 ? -p.uz : p.uz;
                            set_faces(p);
                        } else {
                            lb += (uint32_t)step;
                            cw = next;
                        }
                    }
                }
                // the step's results first: what the add returned is looked at last, when it has come back
                asm volatile("" : "+v"(p.fx), "+v"(p.fy), "+v"(p.fz), "+v"(p.s_rem), "+v"(p.l_void), "+v"(p.steps), "+v"(lb));
                if (__builtin_expect(old + inc < inc, 0)) {
                    // this add wrapped the word's quanta: they go to the voxel's int64 word
                    const uint32_t wi = here / 4u;
                    const int32_t hz = (int32_t)(wi / (uint32_t)kLayer), r = (int32_t)wi - hz * kLayer;
                    const int32_t hy = r / kRow, hx = r - hy * kRow;
                    const uint64_t v = ((uint64_t)(z0 + hz - 1) * (uint64_t)J.ny + (uint64_t)(y0 + hy - 1)) * (uint64_t)J.nx +
                                       (uint64_t)(x0 + hx - 1);
                    __hip_atomic_fetch_add((unsigned long long *)(J.fluence + v), 1ull << (32 - SH + kDepositShift),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            uint64_t stopped = ballot(step == 0) & run;
            run &= ~stopped;
            if (GENERAL) stopped &= ~ballot(end != 0);       // the gated ones
            wait |= stopped;

            const bool cut = drained && since >= kCutAfter && popcount(run | wait) < kCutLanes;
            if (wait != 0ull && (popcount(wait) >= defer || run == 0ull || cut)) {
                if (lanes(wait)) {
                    p.k += 1u;
                    // the round keys are added up here: kept ready, they would fill the scalar registers
                    uint32_t key0 = J.key0, key1 = J.key1;
                    asm volatile("" : "+s"(key0), "+s"(key1));
                    const U4 r = philox4x32_10(U4{p.k, p.pid, J.stream_id, 0u}, key0, key1);
                    uint32_t w_new = (uint32_t)(((uint64_t)p.w * J.s_q + 0x80000000ull) >> 32);
                    asm("" : "+v"(w_new));                   // converted to R as the 32-bit word it is
                    absorbed += (uint64_t)(p.w - w_new);
                    set_weight(p, w_new);
                    if (w_new == 0u) {
                        end = EV_DEAD_ABSORB;
                    } else {
                        const R ct = scatter(p, J, r.x, r.y);
                        if constexpr (GRAD) p.score_g += hg_score((double)ct, (double)J.g);
                        if (w_new < J.w_th) {
                            if ((r.w >> 8) < J.t_m) {
                                atomicAdd(&acc[MC_S_RR + opaque_zero()],
                                          (unsigned long long)(-((int64_t)(J.m - 1u) * (int64_t)w_new)));
                                set_weight(p, w_new * J.m);
                            } else {
                                atomicAdd(&acc[MC_S_RR + opaque_zero()], (unsigned long long)w_new);
                                end = EV_DEAD_ROULETTE;
                            }
                        }
                        p.s_rem = free_path<R>(J, r.z);
                    }
                }
                run |= wait & ballot(end == 0);
                wait = 0ull;
            }
            if (drained) ++since;
            const int32_t free_lanes = cap - popcount(run | wait);
            if (!((run | wait) == 0ull || cut || (!drained && free_lanes >= kRefill))) continue;

            // exchange: the parked photons go (at a cut, all), others come
            const uint64_t going = cut ? have : have & ~(run | wait);
            bool kept = false;
            if (lanes(going)) {
                if (end == 0 && (cw & kOutside) == 0u && p.steps >= J.max_steps) end = EV_LOST;
                if (end != 0) {
                    cell_account(acc, p, end, J.nz);
                    T.keys[slot] = kDead;
                } else {
                    const uint32_t wi = lb / 4u;
                    const int32_t hz = (int32_t)(wi / (uint32_t)kLayer), r = (int32_t)wi - hz * kLayer;
                    const int32_t hy = r / kRow, hx = r - hy * kRow;
                    int32_t ix = x0 + hx - 1, iy = y0 + hy - 1;
                    const int32_t iz = z0 + hz - 1;
                    int32_t kx = cx + (hx > ex ? 1 : (hx < 1 ? -1 : 0));
                    int32_t ky = cy + (hy > ey ? 1 : (hy < 1 ? -1 : 0));
                    const int32_t kz = cz + (hz > ez ? 1 : (hz < 1 ? -1 : 0));
                    // lateral faces are periodic where a photon gets this far
                    if (ix < 0) { ix = J.nx - 1; kx = G.ncx - 1; }
                    if (ix >= J.nx) { ix = 0; kx = 0; }
                    if (iy < 0) { iy = J.ny - 1; ky = G.ncy - 1; }
                    if (iy >= J.ny) { iy = 0; ky = 0; }
                    if (iz < G.zlo || iz >= zend) {
                        cell_account(acc, p, iz < G.zlo ? EV_ESC_R : EV_ESC_T, J.nz);
                        esc_count(s_esc, esc, job, p.l_void, p.w);
                        T.keys[slot] = kDead;
                    } else if ((cw & kOutside) != 0u && kx == cx && ky == cy && kz == cz) {
                        // a lateral wrap onto the cell itself
                        lb = 4u * (uint32_t)((hz * kSide + (iy - y0 + 1)) * kSide + (ix - x0 + 1));
                        cw = cell_word(lb);
                        kept = true;
                    } else {
                        store_slot<R, GENERAL, GRAD>(T.slots + (size_t)slot * NQ, p, ix, iy, iz);
                        T.keys[slot] = G.base + ((uint32_t)kz * (uint32_t)G.ncy + (uint32_t)ky) * (uint32_t)G.ncx + (uint32_t)kx;
                    }
                }
            }
            const uint64_t again = ballot(kept) & going;
            have = (have & ~going) | again;
            run = (run & ~going) | again;
            if (!drained) {
                const uint32_t want = (uint32_t)(cap - popcount(have));
                uint32_t base = 0u;
                if (lane == 0) base = atomicAdd(&s_cursor, want);
                base = __builtin_amdgcn_readfirstlane(base);
                const uint32_t rank = (uint32_t)popcount(~have & __lanemask_lt());
                const bool take = !lanes(have) && rank < want && base + rank < n_ph;
                if (take) {
                    slot = list[base + rank];
                    int32_t ix, iy, iz;
                    load_slot<R, GENERAL, GRAD>(T.slots + (size_t)slot * NQ, p, ix, iy, iz, J);
                    set_weight(p, p.w);
                    lb = 4u * (uint32_t)(((iz - z0 + 1) * kSide + (iy - y0 + 1)) * kSide + (ix - x0 + 1));
                    cw = cell_word(lb);
                    end = 0;
                }
                const uint64_t got = ballot(take);
                have |= got;
                run |= got;
                drained = base + want >= n_ph;
            }
            if (drained && have == 0ull) break;
        }

        __syncthreads();
        // the cell's tally into the caller's
        const uint32_t tx = threadIdx.x & 31u;
        if (tx < (uint32_t)ex) {
            for (uint32_t row = threadIdx.x >> 5; row < (uint32_t)(ey * ez); row += kBlock / 32) {
                const uint32_t hz = row / (uint32_t)ey, hy = row - hz * (uint32_t)ey;
                const int32_t gz = z0 + (int32_t)hz;
                const uint32_t v = tally[(hz + 1u) * kLayer + (hy + 1u) * kRow + tx + 1u] >> SH;
                if (v != 0u && gz >= 0 && gz < J.nz) {
                    const uint64_t i = ((uint64_t)gz * (uint64_t)J.ny + (uint64_t)(y0 + (int32_t)hy)) * (uint64_t)J.nx +
                                       (uint64_t)(x0 + (int32_t)tx);
                    __hip_atomic_fetch_add((unsigned long long *)(J.fluence + i), (unsigned long long)v << kDepositShift,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        if (GRAD)
            for (int32_t i = threadIdx.x; i < 6 * kCell; i += kBlock) {
                const long long v = (long long)s_grad[i];
                if (v) grad_global_add(grad, (i / kCell) * J.nz + z0 + i % kCell, v);
            }
    }
    if (cur_job >= 0) {
        if (absorbed) atomicAdd(&acc[MC_S_A], (unsigned long long)absorbed);
        __syncthreads();
        if (threadIdx.x < MC_NSCALARS) {
            const unsigned long long v = acc[threadIdx.x];
            if (v) atomicAdd((unsigned long long *)&T.jobs[cur_job].scalars[threadIdx.x], v);
        }
        esc_flush(s_esc, esc);
    }
}

// ---------------------------------------------------------------------------
// What the rounds leave: the photons still alive, and any not launched yet
// ---------------------------------------------------------------------------
template <bool GRAD>
struct TailSink : BatchLoggedSink {
    int *bins;
    unsigned long long *grad;
    template <typename R> __device__ __forceinline__ void segment(const Photon<R> &p, const Job &J, R d, bool solid)
    {
        if constexpr (GRAD) {
            if (p.iz < 0 || p.iz >= J.nz) return;
            long long vs, va, vg;
            grad_values(p, J.mu_s > 0.0 ? 1.0 / J.mu_s : 0.0, (double)d, solid, vs, va, vg);
            const int32_t base = (solid ? 0 : J.nz) + p.iz;
            grad_bin_add(bins, grad, base, vs);
            grad_bin_add(bins, grad, 2 * J.nz + base, va);
            grad_bin_add(bins, grad, 4 * J.nz + base, vg);
        }
    }
    template <typename R> __device__ __forceinline__ void deflect(Photon<R> &p, const Job &J, R ct)
    {
        if constexpr (GRAD) p.score_g += hg_score((double)ct, (double)J.g);
    }
};

constexpr int kTailBlock = 256;
constexpr int32_t kTailRefill = 16, kTailDefer = 4;

// JOBS: several jobs, whose staging tallies the log's entries index with 26 bits (log_words)
template <typename R, bool GENERAL, bool GRAD, bool JOBS, bool HIST>
__global__ __launch_bounds__(kTailBlock) void k_cells_tail(Tables T, unsigned long long *__restrict__ grad,
                                                           const BatchEsc *__restrict__ esc)
{
    constexpr int NQ = slot_quads<R, GENERAL, GRAD>();
    constexpr int kWaves = kTailBlock / 64;
    constexpr bool kFP32 = std::is_same<R, float>::value;
    extern __shared__ unsigned long long s_dyn[];   // the jobs, their channels, the score bins
    __shared__ uint32_t s_lidx[kWaves * kBLogK * kBLogStride];
    __shared__ uint32_t s_lval[kWaves * kBLogK * kBLogStride];
    __shared__ EscBins<HIST> s_esc;
    Ctrl *c = T.ctrl;
    const int32_t n_jobs = (int32_t)c->n_jobs;
    Job *s_jobs = (Job *)s_dyn;
    unsigned long long *acc = s_dyn + (size_t)n_jobs * (sizeof(Job) / 8);
    int *s_bins = (int *)(acc + (size_t)n_jobs * MC_NSCALARS);
    for (int32_t i = threadIdx.x; i < n_jobs * (int32_t)(sizeof(Job) / 8); i += kTailBlock)
        s_dyn[i] = ((const unsigned long long *)T.jobs)[i];
    for (int32_t i = threadIdx.x; i < n_jobs * MC_NSCALARS; i += kTailBlock) acc[i] = 0ull;
    const uint32_t lane = __lane_id();
    uint32_t *lidx = s_lidx + (threadIdx.x >> 6) * kBLogK * kBLogStride;
    uint32_t *lval = s_lval + (threadIdx.x >> 6) * kBLogK * kBLogStride;
    for (int i = 0; i < kBLogK; ++i) lval[i * kBLogStride + lane] = 0u;
    esc_clear(s_esc);
    TailSink<GRAD> sink;
    sink.lidx = lidx;
    sink.lval = lval;
    sink.lane = lane;
    sink.head = 0u;
    sink.count = 0u;
    sink.bins = s_bins;
    sink.grad = grad;
    if (GRAD)
        for (int32_t i = threadIdx.x; i < 6 * T.jobs[0].nz; i += kTailBlock) s_bins[i] = 0;
    __syncthreads();
    const uint64_t alive = c->alive, launched = c->next_id < c->total ? c->next_id : c->total;
    const uint64_t total = alive + (c->total - launched);
    // lanes of each wavefront in use: few photons are spread over the chip
    const uint64_t waves = (uint64_t)gridDim.x * kWaves, share = (total + waves - 1) / waves;
    const int32_t cap = (int32_t)(share < 64 ? share : 64);
    const int32_t refill = min(cap, kTailRefill), defer = min(kTailDefer, max(1, cap / 8));
    Photon<R> p;
    int32_t job = 0;
    bool live = false, waiting = false, empty = total == 0;
    for (;;) {
        const uint64_t idle = ballot(!live);
        const int32_t busy = 64 - popcount(idle);
        if (!empty && (busy == 0 || cap - busy >= refill)) {
            const uint32_t want = (uint32_t)(cap - busy);
            unsigned long long base = 0ull;
            if (lane == 0) base = atomicAdd(&c->tail_next, (unsigned long long)want);
            base = __shfl(base, 0);
            const uint32_t rank = (uint32_t)popcount(idle & __lanemask_lt());
            const uint64_t q = base + rank;
            if (!live && rank < want && q < total) {
                if (q < alive) {
                    const uint32_t slot = T.list[q];
                    job = job_of_cell(T.grids, n_jobs, T.keys[slot]);
                    const Job &J = s_jobs[job];
                    load_slot<R, GENERAL, GRAD>(T.slots + (size_t)slot * NQ, p, p.ix, p.iy, p.iz, J);
                    p.absorbed = 0ull;
                    p.rr = 0;
                    p.acc = 0ull;
                    p.brick = 0xFFFFFFFFu;
                    lookup<GENERAL>(p, J);
                } else {
                    const uint64_t qq = launched + (q - alive);
                    job = job_of_queue(T.jobs, n_jobs, qq);
                    const Job &J = s_jobs[job];
                    launch<GENERAL>(p, J, (uint32_t)(J.photon_begin + (qq - J.queue_begin)));
                }
                live = true;
            }
            empty = base + want >= total;
        }
        if (empty && ballot(live) == 0ull) break;
        sink.tag = log_tag<JOBS>(job);
        auto retire = [&](int32_t ev) {
            unsigned long long *a = acc + (size_t)job * MC_NSCALARS;
            cell_account(a, p, ev, s_jobs[job].nz);
            if (p.absorbed) atomicAdd(&a[MC_S_A], (unsigned long long)p.absorbed);
            if (p.rr) atomicAdd(&a[MC_S_RR], (unsigned long long)p.rr);
            if (ev == EV_ESC_R || ev == EV_ESC_T) esc_count(s_esc, esc, job, p.l_void, p.w);
            live = false;
        };
        if (live && !waiting) {
            const Job &J = s_jobs[job];
            // a photon at its step cap when its slot was stored ends here, before another step
            int32_t fin = p.steps >= J.max_steps ? (int32_t)EV_LOST : -1;
            if (fin < 0) {
                const int32_t ev = advance<GENERAL>(p, J, sink);
                if (ev == EV_AT_INTERACTION) waiting = true;
                else fin = finish(p, J, sink, ev);
            }
            if (fin >= 0 && is_terminal(fin)) retire(fin);
        }
        const uint64_t wm = ballot(waiting);
        if (wm != 0ull && ((kFP32 && empty) || popcount(wm) >= defer || ballot(live && !waiting) == 0ull)) {
            if (waiting) {
                const Job &J = s_jobs[job];
                const int32_t fin = finish(p, J, sink, interact(p, J, sink));
                waiting = false;
                if (is_terminal(fin)) retire(fin);
            }
        }
        // a lane logs at most one deposit per iteration
        if (ballot(sink.count >= (uint32_t)kBLogK) != 0ull)
            flush_batch_log<kFP32, JOBS>(lidx, lval, s_jobs, lane,
                                         live ? (stage_word(s_jobs[job], p) | sink.tag) >> 4 : kBNoLine, sink.head,
                                         sink.count);
    }
    flush_batch_log<kFP32, JOBS>(lidx, lval, s_jobs, lane, kBNoLine, sink.head, sink.count);
    __syncthreads();
    esc_flush(s_esc, esc);
    for (int32_t i = threadIdx.x; i < n_jobs * MC_NSCALARS; i += kTailBlock) {
        const unsigned long long v = acc[i];
        if (v) atomicAdd((unsigned long long *)&s_jobs[i / MC_NSCALARS].scalars[i % MC_NSCALARS], v);
    }
    if (GRAD)
        for (int32_t i = threadIdx.x; i < 6 * T.jobs[0].nz; i += kTailBlock) {
            const long long v = (long long)s_bins[i];
            if (v) grad_global_add(grad, i, v);
        }
}

// ---------------------------------------------------------------------------
// Setup
// ---------------------------------------------------------------------------
struct JobPack { Job j[8]; Grid g[8]; };

__global__ void k_cells_jobs(JobPack pack, Job *__restrict__ dst, Grid *__restrict__ grids, int32_t count)
{
    const int32_t w = (int32_t)(sizeof(Job) / 8);
    const uint64_t *src = (const uint64_t *)pack.j;
    uint64_t *d = (uint64_t *)dst;
    for (int32_t i = threadIdx.x; i < count * w; i += blockDim.x) d[i] = src[i];
    if ((int32_t)threadIdx.x < count) grids[threadIdx.x] = pack.g[threadIdx.x];
}

__global__ void k_cells_setup(Tables T, uint64_t total, uint32_t n_jobs, uint32_t n_cells, uint32_t slots, uint32_t stop_at, uint32_t walkers)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x, n = gridDim.x * blockDim.x;
    for (uint32_t k = i; k < slots; k += n) T.keys[k] = kDead;
    if (i == 0u) {
        Ctrl c;
        memset(&c, 0, sizeof c);
        c.total = total;
        c.n_jobs = n_jobs;
        c.n_cells = n_cells;
        c.slots = slots;
        c.stop_at = stop_at;
        c.walkers = walkers;
        *T.ctrl = c;
    }
}

uint32_t quotient_factor(int32_t e) { return e == 1 ? 0u : (uint32_t)((0x100000000ull + (uint64_t)e - 1) / (uint64_t)e); }

size_t up256(size_t x) { return (x + 255) / 256 * 256; }

size_t quads_of(const CellRun &r) { return (r.fp64 ? 6 : 4) + (r.general ? 1 : 0) + (r.grad ? 1 : 0); }
size_t slot_bytes(const CellRun &r) { return quads_of(r) * 16 + 8; }   // with its key and its place in the list

// The slots a walk of so many cells takes at most: enough for items of some 24 000 photons per cell.
constexpr uint64_t kMaxSlots = 12ull << 20, kMinSlots = 1ull << 20;
uint64_t wanted_slots(uint64_t cells) { return std::min(kMaxSlots, std::max(kMinSlots, (uint64_t)(cells * 24576))); }

// Full items hold at least kMinItem photons, and a cell has at most one item that is not full.
size_t item_count(uint64_t cells) { return (size_t)(cells + kMaxSlots / kMinItem + 64); }

struct Plan {
    Tables T;
    CellDims d[MC_MAX_BATCH_JOBS];
    BatchEsc *esc;              // a single run's own table and copies
    unsigned long long *esc_copies;
    uint64_t cells;
    uint32_t slots;
};

constexpr size_t kEscCopyBytes = 2ull * kEscReplicas * kEscMaxBins * sizeof(uint64_t);

// Lays the tables out from `base` (NULL: only their sizes); returns the bytes in front of the slots' arrays.
size_t lay_tables(char *base, uint64_t cells, int32_t n_jobs, Plan *P)
{
    size_t off = 0;
    auto take = [&](size_t bytes) { char *p = base + off; off += up256(bytes); return p; };
    Tables &T = P->T;
    T.ctrl = (Ctrl *)take(sizeof(Ctrl));
    T.jobs = (const Job *)take(sizeof(Job) * (size_t)n_jobs);
    T.grids = (const Grid *)take(sizeof(Grid) * (size_t)n_jobs);
    P->esc = (BatchEsc *)take(sizeof(BatchEsc));
    P->esc_copies = (unsigned long long *)take(kEscCopyBytes);
    T.count = (uint32_t *)take(cells * 4);
    T.block_base = (uint32_t *)take(cells * 4 * kSortBlocks);
    T.items = (Item *)take(item_count(cells) * sizeof(Item));
    return off;
}

constexpr size_t kSlack = 1024;   // the start and the arrays rounded up to 256 bytes

bool plan_of(const CellRun &r, Plan *P)
{
    uint64_t cells = 0;
    for (int32_t i = 0; i < r.n_jobs; ++i) {
        mc_volume v;
        v.nx = r.table[i].nx;
        v.ny = r.table[i].ny;
        v.nz = r.table[i].nz;
        P->d[i] = cell_dims(&v, r.table[i].paper);
        cells += P->d[i].cells;
    }
    P->cells = cells;
    if (cells > (uint64_t)kMaxCells) return false;
    // a caller's workspace may start at any 8 bytes; a slot is one 64-byte line
    char *const ws = (char *)up256((size_t)r.ws);
    const size_t off = lay_tables(ws, cells, r.n_jobs, P), lost = (size_t)(ws - r.ws) + off + kSlack;
    if (r.ws_bytes <= lost) return false;
    const size_t per = slot_bytes(r);
    uint64_t slots = std::min<uint64_t>((r.ws_bytes - lost) / per, wanted_slots(cells));
    slots = std::min<uint64_t>(slots, r.photons + 3) / 4 * 4;   // the keys are read four at a time
    P->slots = (uint32_t)slots;
    char *p = ws + off;
    P->T.keys = (uint32_t *)p;
    P->T.list = (uint32_t *)(p + up256(slots * 4));
    P->T.slots = (uint4 *)(p + 2 * up256(slots * 4));
    return true;
}

template <typename R, bool GENERAL, bool GRAD, bool JOBS, bool HIST>
int enqueue_cells(const CellRun &r, const Plan &P, int rounds, int cus, const BatchEsc *esc, hipStream_t s)
{
    const Tables &T = P.T;
    const size_t hist = P.cells * 4;
    // free slots a block of the count can list at once, at most its share of the slots
    const uint32_t room = (uint32_t)std::min<size_t>((kLds - 1024 - hist) / 2 / 64 * 64, 65536);
    const size_t lds_count = hist + 2 * (size_t)room;
    for (int k = 0; k <= rounds; ++k) {
        hipLaunchKernelGGL((k_cells_count<R, GENERAL, GRAD>), dim3(kSortBlocks), dim3(kSortThreads), lds_count, s, T, room);
        hipLaunchKernelGGL(k_cells_columns, dim3((unsigned)((P.cells + 63) / 64)), dim3(kSortThreads), 0, s, T);
        hipLaunchKernelGGL(k_cells_scatter, dim3(kSortBlocks), dim3(kSortThreads), hist, s, T, (int32_t)(k == rounds));
        if (k < rounds)
            hipLaunchKernelGGL((k_cells_walk<R, GENERAL, GRAD, HIST>), dim3(cus), dim3(walk_block<R>()), 0, s, T, r.grad, esc);
    }
    const size_t lds = (size_t)r.n_jobs * (sizeof(Job) + MC_NSCALARS * 8) + (GRAD ? (size_t)6 * r.table[0].nz * sizeof(int) : 0);
    hipLaunchKernelGGL((k_cells_tail<R, GENERAL, GRAD, JOBS, HIST>), dim3(cus * 4), dim3(kTailBlock), lds, s, T, r.grad, esc);
    HIP_TRY(hipGetLastError());
    return MC_OK;
}

template <typename R, bool GENERAL>
int enqueue_kind(const CellRun &r, const Plan &P, int rounds, int cus, const BatchEsc *esc, hipStream_t s)
{
    // gradients and a histogram of its own are those of a run of one job
    if (r.grad) return enqueue_cells<R, GENERAL, true, false, false>(r, P, rounds, cus, esc, s);
    if (r.hist) return enqueue_cells<R, GENERAL, false, false, true>(r, P, rounds, cus, esc, s);
    if (r.n_jobs > 1) return enqueue_cells<R, GENERAL, false, true, false>(r, P, rounds, cus, esc, s);
    return enqueue_cells<R, GENERAL, false, false, false>(r, P, rounds, cus, esc, s);
}

template <typename R>
int enqueue_general(const CellRun &r, const Plan &P, int rounds, int cus, const BatchEsc *esc, hipStream_t s)
{
    return r.general ? enqueue_kind<R, true>(r, P, rounds, cus, esc, s) : enqueue_kind<R, false>(r, P, rounds, cus, esc, s);
}

// The path, in voxels, on which a photon's weight ends (the interactions from 1 down to the roulette's threshold, or to the
// last bit, 10 / mu_t apart in a mask nine tenths open) or the gate does.
double longest_path(const Job &J)
{
    double path = J.gate;
    const double keep = (double)J.s_q / 4294967296.0;        // weight kept at an interaction
    if (J.mu_t > 0.0 && keep < 1.0) {
        const double last = J.w_th ? J.w_th / 2147483648.0 : 1.0 / 2147483648.0;
        const double interactions = 1.0 + (keep > 0.0 ? log(last) / log(keep) : 0.0);
        path = std::min(path, 10.0 * interactions / J.mu_t);
    }
    return path;
}

// Visits per voxel of path: one over the mean chord 4V/S of a cell, of whose faces those count that lie between two cells (on an
// axis of one cell a periodic photon comes back into it).
double chord_faces(const CellDims &d)
{
    return 0.5 * ((d.ncx > 1 ? 1.0 / d.ex : 0.0) + (d.ncy > 1 ? 1.0 / d.ey : 0.0) + (d.ncz > 1 ? 1.0 / d.ez : 0.0));
}

// Whether a run is faster in cells than by the log (k_walk, k_walk_batch).  What the cells save is the deposits at the memory
// side; what they cost is a round's fixed time and a cell's (its mask in, its tally out), paid by the photons of a workgroup's
// share and of a cell and by the steps of a visit, and the end of the run, which both walk the same way.  They save less where a
// step does more arithmetic: interactions (mu_s), the FP64 transport, interfaces, scores.  Times of the log over those in
// cells, at phi 0.7, mu_s 0.5, mu_a 0.01, g 0.7 but for what is said:
//   256^3                2e6 photons 1.07, 5e6 1.45, 1e7 1.88; FP64 0.99, 1.19; paper's model 1.00, 1.23, 1.36
//   128^3, 64^3          5e6 1.25, 1.08; FP64 128^3 1.12; paper's model 128^3 1.07
//   512 x 512 x 8        2e6 0.94, 5e6 1.01, 1e7 1.11; FP64 0.77, 0.97, 1.04; paper's model 5e6 0.90, 2e7 1.04
//   512 x 512 x 64       mu_s 0.036 2e6 0.90, 5e6 1.14;  64^3 0.86, 1.03;  512 x 512 x 8 1e7 0.90, 5e7 1.17
//   40 x 256 x 40        reach 56e3: mu_s 0.5 2e6 0.96, 5e6 1.04, 2e7 1.11; mu_s 0.036 0.87, 0.89, 1.07; mu_a 0.5 0.93, 0.96, 0.94
//   mu_s 1               2e6 0.85 to 1.0, 5e6 1.04 to 1.25
//   mu_s 2 to 5          256^3 5e6 0.81 to 1.04, 1e7 1.03 to 1.22; 512 x 512 x 64 1.16 to 1.31; 100 x 90 x 110 0.62 to 0.97;
//                        128^3 0.89 to 1.1; 32^3, one cell, 2e6 1.22, 5e6 1.32 to 1.48
//   gradients            256^3 2e6 0.95, 5e6 1.13, 5e7 1.53; FP64 0.94, 1.03, 1.08; paper's model 0.88, 1.07, 1.25; 128^3 (reach
//                        124e3) at most 0.90, FP64 0.80, paper's model 0.72; 512 x 512 x 8 5e6 0.88, 2e7 1.03, paper's model 0.91
//   1024 x 1024 x 384    5e7 plain 1.36 (800 to 1000 photons a cell); paper's model 0.90, mu_s 0.036 2e7 1.10; gradients 0.86
//   1 x 300 x 300        1.2 to 1.9; paper's model 0.78 to 0.94 (each step leaves the cell and comes back)
// The log of a batch, which finds a photon's job in LDS, is slower:
//   64 x 32^3            2e6 1.22, 2e7 1.9; FP64 1.16, 1.35; paper's model 1.20, 1.6
//   3 x 200^3 to 256^3   2e6 1.2, 2e7 1.9; FP64 1.17, 1.6; paper's model 1.24, 1.9; mu_s 4 2e6 0.89, 6e6 1.27, 2e7 1.57
//   64 x 64^3 to 160^3   2e6 1.08, 6e6 1.11, 2e7 1.4; FP64 0.96, 1.08, 1.27 (450, 1000, 2100 photons a cell); with the paper's
//                        model 0.91, 1.07, 1.00;  12 x 64^3 to 128^3, mu_s 0.05 2e6 0.88, 6e6 1.37; mu_s 4 6e6 0.91, 2e7 1.35
bool faster_in_cells(const CellRun &r, const Plan &P, int cus)
{
    double path = 0.0, visits = 0.0, work = 0.0, mu_s = 0.0, depth = 0.0;
    int32_t narrow = kCell;
    bool one_cell = true;
    for (int32_t i = 0; i < r.n_jobs; ++i) {
        const Job &J = r.table[i];
        const double n = (double)J.n_photons, p = std::min(3.0 * J.nz, longest_path(J)), per = chord_faces(P.d[i]);
        path += n * p;
        visits += n * (1.0 + p * per);
        work += n * J.nz;
        mu_s += n * J.mu_s;
        narrow = std::min(narrow, std::min(P.d[i].ex, P.d[i].ey));
        one_cell = one_cell && per == 0.0;
    }
    const double photons = (double)r.photons;
    mu_s /= photons;
    depth = work / photons;
    // photons of a workgroup at once, times the voxels of a visit
    const double reach = (double)P.slots / cus * path / visits, per_cell = (double)P.slots / (double)P.cells;
    if (r.batch) return photons >= (mu_s > 1.5 ? 4e6 : (mu_s * depth < 5.0 ? 3e6 : 0.0)) && (!r.fp64 || per_cell >= 600.0);
    if (!one_cell && photons < (mu_s > 1.5 ? 8e6 : (mu_s > 0.75 ? 4e6 : 0.0))) return false;
    if (mu_s > 1.5 && reach < 250e3) return false;
    if (r.grad) {
        const double bytes = reach * (double)slot_bytes(r) / 72.0;   // a wider photon has fewer slots and takes as much longer
        return photons >= 3e6 && per_cell >= 2000.0 && (r.general ? depth >= 32.0 && bytes >= 360e3 : bytes >= 350e3);
    }
    if (r.fp64 || r.general)
        return per_cell >= (!r.fp64 && mu_s < 0.25 ? 600.0 : 1000.0) && work >= 1.2e8 && reach >= 80e3 && narrow >= (r.general ? 4 : 8);
    return reach >= 50e3 && work >= (mu_s * depth < 3.0 ? 2.3e8 : 5e7);
}

// The rounds to enqueue: those in which the photons are launched, each of which takes a path of three slab thicknesses, and
// those until no more than the end are left, who fall by a factor e on 4.2 thicknesses (1075 voxels; 1075 observed).  A photon
// visits its path over the mean chord 4V/S of a cell (chord_faces): 36 cells for 256^3, 32 observed.  A round that finds nothing
// left costs 11 us; what a short estimate leaves the tail takes (where light diffuses slower, mu_s (1 - g) = 2 at 256^3, 1e7
// photons, the rounds are a tenth of those it would take to the end, and all of them would be slower: 222 ms against 198).
int rounds_of(const CellRun &r, const Plan &P, uint32_t stop_at)
{
    double after = 0.0, launches = 0.0;
    const double folds = log((double)P.slots / (stop_at + 0.5 * kStopPerCell * P.cells));
    for (int32_t i = 0; i < r.n_jobs; ++i) {
        const Job &J = r.table[i];
        const CellDims &d = P.d[i];
        const double per = chord_faces(d);
        launches += (1.0 + per * std::min(3.0 * J.nz, longest_path(J))) * (double)J.n_photons / P.slots;
        after = std::max(after, per * std::min(4.2 * J.nz * folds, longest_path(J)));
    }
    return (int)std::min(kMaxRounds, 8.0 + launches + after);
}

}  // namespace

namespace pmc {
namespace host {

CellDims cell_dims(const mc_volume *vol, bool paper)
{
    CellDims d;
    const int32_t layers = vol->nz + (paper ? 2 : 0);
    d.ncx = (vol->nx + kCell - 1) / kCell;
    d.ncy = (vol->ny + kCell - 1) / kCell;
    d.ncz = (layers + kCell - 1) / kCell;
    d.ex = (vol->nx + d.ncx - 1) / d.ncx;
    d.ey = (vol->ny + d.ncy - 1) / d.ncy;
    d.ez = (layers + d.ncz - 1) / d.ncz;
    // the last cell of an axis is not empty
    d.ncx = (vol->nx + d.ex - 1) / d.ex;
    d.ncy = (vol->ny + d.ey - 1) / d.ey;
    d.ncz = (layers + d.ez - 1) / d.ez;
    d.zlo = paper ? -1 : 0;
    d.cells = (uint64_t)d.ncx * d.ncy * d.ncz;
    return d;
}

size_t cell_workspace_bytes(const CellDims *dims, int32_t n_jobs, uint64_t photons)
{
    uint64_t cells = 0;
    for (int32_t i = 0; i < n_jobs; ++i) cells += dims[i].cells;
    if (cells > (uint64_t)kMaxCells || photons < kMinPhotons) return 0;
    Plan P;
    return up256(lay_tables(nullptr, cells, n_jobs, &P) + kSlack + std::min(photons + 4, wanted_slots(cells)) * (4 * 16 + 8));
}

bool cell_walk_fits(const CellRun &r)
{
    DeviceInfo di;
    if (device_info(&di) != MC_OK) return false;
    for (int32_t i = 0; i < r.n_jobs; ++i) {
        const Job &J = r.table[i];
        // the walk in cells keeps no total path to compare with a cap; the tail logs its deposits
        if (J.path_cap != (float)kInf || J.stage == nullptr || stage_words(J) > log_words(r.n_jobs)) return false;
    }
    Plan P;
    if (!plan_of(r, &P)) return false;
    if (r.always) return P.slots != 0;
    const uint64_t least = std::max<uint64_t>(kMinPhotons, 2ull * di.cus * kStopPerCu);
    return r.photons >= least && P.slots >= least / 2 && faster_in_cells(r, P, di.cus);
}

int cell_walk(const CellRun &r, hipStream_t s)
{
    Plan P;
    if (!plan_of(r, &P)) return fail(MC_ENOSPACE, "cell walk: scratch too small");
    DeviceInfo di;
    int rc = device_info(&di);
    if (rc) return rc;
    uint32_t base = 0;
    for (int32_t i = 0; i < r.n_jobs; i += 8) {
        JobPack pack;
        memset(&pack, 0, sizeof pack);
        const int32_t c = std::min(8, r.n_jobs - i);
        for (int32_t k = 0; k < c; ++k) {
            const CellDims &d = P.d[i + k];
            pack.j[k] = r.table[i + k];
            pack.g[k] = Grid{d.ncx, d.ncy, d.ncz, d.ex, d.ey, d.ez, d.zlo, base,
                             quotient_factor(d.ex), quotient_factor(d.ey), quotient_factor(d.ez)};
            base += (uint32_t)d.cells;
        }
        hipLaunchKernelGGL(k_cells_jobs, dim3(1), dim3(256), 0, s, pack, (Job *)P.T.jobs + i, (Grid *)P.T.grids + i, c);
        HIP_TRY(hipGetLastError());
    }
    const uint32_t stop_at = (uint32_t)di.cus * kStopPerCu;
    hipLaunchKernelGGL(k_cells_setup, dim3(1024), dim3(256), 0, s, P.T, r.photons, (uint32_t)r.n_jobs, (uint32_t)P.cells,
                       P.slots, stop_at, (uint32_t)di.cus);
    HIP_TRY(hipGetLastError());
    const BatchEsc *esc = r.esc;
    if (r.hist) {
        BatchEsc e = *r.hist;
        e.rw = P.esc_copies;
        e.rn = P.esc_copies + (size_t)kEscReplicas * kEscMaxBins;
        if ((rc = fill((int64_t *)P.esc_copies, kEscCopyBytes / 8, s))) return rc;
        if ((rc = write_esc(&e, 1, P.esc, s))) return rc;
        esc = P.esc;
    }
    const int rounds = rounds_of(r, P, stop_at);
    if (r.fp64) rc = enqueue_general<double>(r, P, rounds, di.cus, esc, s);
    else rc = enqueue_general<float>(r, P, rounds, di.cus, esc, s);
    if (rc) return rc;
    return r.hist ? fold_esc(P.esc, 1, s) : MC_OK;
}

}  // namespace host
}  // namespace pmc
