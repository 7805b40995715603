// Exact top-k marking on the GPU: mask[i] = 1 for the k largest values of an
// array, equal values going to the lower index.  An MSB-first radix select over
// an order-preserving 64-bit key (11-bit digits) narrows the keys down to those
// that share their leading digits with the k-th largest key T; as soon as these
// candidates are few they are gathered with their indices, one workgroup finds T
// and the last index taken among the keys equal to T, and the mask is written.
// Where more keys than that are equal, all six digits are taken and a chunked scan
// in index order counts the equal ones.  Used by the rank binarisation of the
// spinodal generator.  Every kernel has internal linkage.
//
// Bound by reading the array: with 16.7e6 doubles two digits leave some 3000
// candidates, so it is read four times (two digits, gather, mark).  Measured there:
// 0.17 ms, against 0.97 with six digits each followed by a scan of its 2048 counts by
// one thread (107 us of the 151 a digit took).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "internal.hpp"

namespace pmc {
namespace sel {
namespace {

constexpr int kThreads = 256;
constexpr int kDigitBits = 11;
constexpr int kDigits = 1 << kDigitBits;
constexpr int kChunk = kThreads * 16;      // elements per marking workgroup

constexpr int kDigitThreads = 1024;
constexpr int kDigitBlocks = 256;          // each adds up to kDigits counts in memory: 256 of them, with 8 loads in flight a thread
constexpr int kInFlight = 8;
constexpr int kCopies = 16;               // of the digit counts in LDS: a first digit (sign, exponent) takes few values
constexpr int kCandidates = 8192;          // 64 KB of keys in LDS

struct SelectState {
    unsigned long long prefix;   // key bits chosen so far
    long long k;                 // rank still to find inside the current candidates (1-based, from the top)
    long long count;             // keys that share the bits chosen so far
    int shift;                   // the lowest bit chosen so far
    unsigned int ticket;         // workgroups of the running digit pass that are done
    unsigned int fill;           // candidates gathered so far
    unsigned int done;           // prefix is T and last its last index taken
    long long last;
    long long pad;
};

// order-preserving map to uint64 (-0.0 and +0.0 map alike)
__device__ __forceinline__ unsigned long long key_of(double v)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v + 0.0);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// the bits at and above `low`
__device__ __forceinline__ unsigned long long bits_from(int low) { return low >= 64 ? 0ull : (~0ull << low); }

// Of digit counts c(0 .. nbins), find the digit that holds the k-th largest entry.  The
// thread that finds it (exactly one where 1 <= k <= their sum) calls
// found(digit, rank inside it, its count).  All kDigitThreads threads take part.
template <class Count, class Found>
__device__ __forceinline__ void find_digit(int nbins, long long k, unsigned long long *wsum, Count c, Found found)
{
    const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
    // thread t holds digits nbins-1-2t and nbins-2-2t: the prefix over threads runs from the top digit down
    static_assert(kDigits <= 2 * kDigitThreads, "two digits a thread");
    const int hi = nbins - 1 - 2 * t, lo = hi - 1;
    const unsigned long long chi = hi >= 0 ? c(hi) : 0ull, clo = lo >= 0 ? c(lo) : 0ull;
    unsigned long long incl = chi + clo;
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += wsum[w];
    const long long excl = (long long)(incl - chi - clo);
    if (excl < k && k <= (long long)incl) {
        const bool in_hi = excl + (long long)chi >= k;
        found(in_hi ? hi : lo, k - (in_hi ? excl : excl + (long long)chi), (long long)(in_hi ? chi : clo));
    }
    __syncthreads();
}

// One digit: counts of the candidates' digit in LDS, added up in hist (all zero before
// and after); the last workgroup picks the digit of the k-th largest.  Nothing is left
// to do once at most `cap` candidates remain.
template <typename T>
__global__ __launch_bounds__(kDigitThreads) void k_digit(const T *__restrict__ f, long long n, SelectState *st,
                                                         unsigned long long *hist, int shift, int bits, long long cap)
{
    __shared__ unsigned int h[kDigits * kCopies];
    __shared__ unsigned long long wsum[kDigitThreads / 64];
    __shared__ unsigned int s_last;
    if (st->count <= cap) return;
    const int t = (int)threadIdx.x, nbins = 1 << bits;
    for (int i = t; i < nbins * kCopies; i += kDigitThreads) h[i] = 0u;
    __syncthreads();
    const unsigned long long chosen = bits_from(shift + bits), prefix = st->prefix;
    const unsigned copy = threadIdx.x % kCopies;
    const long long step = (long long)gridDim.x * kDigitThreads;
    auto add = [&](unsigned long long key) {
        if ((key & chosen) == prefix) atomicAdd(&h[((unsigned)(key >> shift) & (unsigned)(nbins - 1)) * kCopies + copy], 1u);
    };
    long long i = (long long)blockIdx.x * kDigitThreads + t;
    for (; i + (kInFlight - 1) * step < n; i += kInFlight * step) {
        T v[kInFlight];
#pragma unroll
        for (int j = 0; j < kInFlight; ++j) v[j] = f[i + j * step];
#pragma unroll
        for (int j = 0; j < kInFlight; ++j) add(key_of(v[j]));
    }
    for (; i < n; i += step) add(key_of(f[i]));
    __syncthreads();
    for (int b0 = t; b0 < nbins; b0 += kDigitThreads) {
        const int b = (b0 + (int)blockIdx.x * 64) & (nbins - 1);     // the workgroups add to different bins at a time
        unsigned long long c = 0ull;
        for (int j = 0; j < kCopies; ++j) c += h[b * kCopies + j];
        if (c) atomicAdd(&hist[b], c);
    }
    // every wavefront waits for its additions; one thread's fence then orders them before the
    // ticket (a fence of each of the 4096 wavefronts writes its L2 back as often)
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (t == 0) {
        __threadfence();
        s_last = atomicAdd(&st->ticket, 1u) == gridDim.x - 1u ? 1u : 0u;
        __threadfence();
    }
    __syncthreads();
    if (!s_last) return;
    find_digit(nbins, st->k, wsum,
               [&](int b) { return __hip_atomic_load(&hist[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
               [&](int d, long long k, long long count) {
                   st->k = k;
                   st->count = count;
                   st->prefix = prefix | ((unsigned long long)d << shift);
                   st->shift = shift;
                   st->ticket = 0u;
               });
    for (int b = t; b < nbins; b += kDigitThreads) hist[b] = 0ull;
}

// The candidates, where they are few, with their indices, in any order
template <typename T>
__global__ __launch_bounds__(kDigitThreads) void k_gather(const T *__restrict__ f, long long n, SelectState *st,
                                                          unsigned long long *keys, long long *index, long long cap)
{
    if (st->count > cap) return;
    const unsigned long long chosen = bits_from(st->shift), prefix = st->prefix;
    const long long step = (long long)gridDim.x * kDigitThreads;
    auto take = [&](unsigned long long key, long long i) {
        if ((key & chosen) == prefix) {
            const unsigned at = atomicAdd(&st->fill, 1u);     // at most st->count of them
            keys[at] = key;
            index[at] = i;
        }
    };
    long long i = (long long)blockIdx.x * kDigitThreads + threadIdx.x;
    for (; i + (kInFlight - 1) * step < n; i += kInFlight * step) {
        T v[kInFlight];
#pragma unroll
        for (int j = 0; j < kInFlight; ++j) v[j] = f[i + j * step];
#pragma unroll
        for (int j = 0; j < kInFlight; ++j) take(key_of(v[j]), i + j * step);
    }
    for (; i < n; i += step) take(key_of(f[i]), i);
}

// One workgroup: the k-th largest of v[0 .. nc) in LDS, whose bits at and above `low`
// equal prefix's where they count; on return prefix is that key and k the rank among
// the entries equal to it, *equal their number.
__device__ __forceinline__ void select_lds(const unsigned long long *v, int nc, unsigned int *h, unsigned long long *wsum,
                                           SelectState *pick, unsigned long long &prefix, long long &k, int low,
                                           long long *equal)
{
    const int t = (int)threadIdx.x;
    *equal = nc;
    while (low > 0) {
        const int bits = low < kDigitBits ? low : kDigitBits, shift = low - bits, nbins = 1 << bits;
        for (int i = t; i < nbins; i += kDigitThreads) h[i] = 0u;
        __syncthreads();
        const unsigned long long chosen = bits_from(low);
        for (int i = t; i < nc; i += kDigitThreads)
            if ((v[i] & chosen) == prefix) atomicAdd(&h[(unsigned)(v[i] >> shift) & (unsigned)(nbins - 1)], 1u);
        __syncthreads();
        find_digit(nbins, k, wsum, [&](int b) { return (unsigned long long)h[b]; },
                   [&](int d, long long rank, long long count) {
                       pick->k = rank;
                       pick->count = count;
                       pick->prefix = prefix | ((unsigned long long)d << shift);
                   });
        prefix = pick->prefix;
        k = pick->k;
        *equal = pick->count;
        low = shift;
        __syncthreads();
    }
}

// One workgroup: T among the gathered candidates, and the last index taken of those
// equal to it.
__global__ __launch_bounds__(kDigitThreads) void k_pick(SelectState *st, const unsigned long long *keys,
                                                        const long long *index, long long n, long long cap)
{
    __shared__ unsigned long long v[kCandidates];
    __shared__ unsigned int h[kDigits];
    __shared__ unsigned long long wsum[kDigitThreads / 64];
    __shared__ SelectState pick;
    if (st->count > cap) return;
    const int t = (int)threadIdx.x, nc = (int)st->count;
    for (int i = t; i < nc; i += kDigitThreads) v[i] = keys[i];
    unsigned long long prefix = st->prefix;
    long long k = st->k, equal = 0;
    select_lds(v, nc, h, wsum, &pick, prefix, k, st->shift, &equal);
    long long last = n;
    if (k < equal) {
        // the k-th smallest index is the k-th largest complement; no complement is 0
        for (int i = t; i < nc; i += kDigitThreads) v[i] = v[i] == prefix ? ~(unsigned long long)index[i] : 0ull;
        unsigned long long c = 0ull;
        long long r = k, same = 0;
        select_lds(v, nc, h, wsum, &pick, c, r, 64, &same);
        last = (long long)~c;
    }
    if (t == 0) {
        st->prefix = prefix;
        st->last = last;
        st->done = 1u;
    }
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_count_eq(const T *__restrict__ f, long long n, const SelectState *st,
                                                       long long *counts)
{
    __shared__ int wsum[kThreads / 64];
    if (st->done) return;
    const unsigned long long key_t = st->prefix;
    const long long base = (long long)blockIdx.x * kChunk;
    int c = 0;
    for (int it = 0; it < kChunk / kThreads; ++it) {
        const long long i = base + it * kThreads + threadIdx.x;
        if (i < n && key_of(f[i]) == key_t) ++c;
    }
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long t = 0;
        for (int w = 0; w < kThreads / 64; ++w) t += wsum[w];
        counts[blockIdx.x] = t;
    }
}

// exclusive scan of the per-chunk counts, one workgroup: each thread scans a
// contiguous segment
__global__ __launch_bounds__(kThreads) void k_scan(const SelectState *st, long long *counts, int nchunks)
{
    __shared__ long long seg[kThreads];
    if (st->done) return;
    const int per = (nchunks + kThreads - 1) / kThreads;
    const int b0 = (int)threadIdx.x * per, b1 = std::min(nchunks, b0 + per);
    long long s = 0;
    for (int b = b0; b < b1; ++b) s += counts[b];
    seg[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long run = 0;
        for (int t = 0; t < kThreads; ++t) {
            const long long v = seg[t];
            seg[t] = run;
            run += v;
        }
    }
    __syncthreads();
    long long run = seg[threadIdx.x];
    for (int b = b0; b < b1; ++b) {
        const long long v = counts[b];
        counts[b] = run;
        run += v;
    }
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_mark(const T *__restrict__ f, long long n, const SelectState *st,
                                                   const long long *__restrict__ offsets, uint8_t *mask)
{
    __shared__ int wcount[kThreads / 64];
    const unsigned long long key_t = st->prefix;
    const long long need = st->k;
    const long long base = (long long)blockIdx.x * kChunk;
    if (st->done) {
        const long long last = st->last;
#pragma unroll 4
        for (int it = 0; it < kChunk / kThreads; ++it) {
            const long long i = base + it * kThreads + threadIdx.x;
            if (i < n) {
                const unsigned long long key = key_of(f[i]);
                mask[i] = (uint8_t)(key > key_t || (key == key_t && i <= last));
            }
        }
        return;
    }
    long long run = offsets[blockIdx.x];
    const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6);
    for (int it = 0; it < kChunk / kThreads; ++it) {
        const long long i = base + it * kThreads + threadIdx.x;
        unsigned long long key = 0ull;
        if (i < n) key = key_of(f[i]);
        const bool eq = i < n && key == key_t;
        const unsigned long long bal = __ballot(eq);
        const int before = __popcll(bal & ((1ull << lane) - 1ull));
        if (lane == 0) wcount[wave] = __popcll(bal);
        __syncthreads();
        int woff = 0;
        for (int w = 0; w < wave; ++w) woff += wcount[w];
        int tot = 0;
        for (int w = 0; w < kThreads / 64; ++w) tot += wcount[w];
        if (i < n) mask[i] = (uint8_t)(key > key_t || (eq && run + woff + before < need));
        run += tot;
        __syncthreads();
    }
}

__global__ void k_fill_u8(uint8_t *p, long long n, uint8_t v)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_init_state(SelectState *st, unsigned long long *hist, long long n, long long k)
{
    if (threadIdx.x == 0) *st = SelectState{0ull, k, n, 64, 0u, 0u, 0u, 0, 0};
    for (int i = (int)threadIdx.x; i < kDigits; i += (int)blockDim.x) hist[i] = 0ull;
}

inline size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// device workspace of enqueue_top for n elements
inline size_t workspace_bytes(long long n)
{
    const size_t nchunks = (size_t)((n + kChunk - 1) / kChunk);
    return align256(sizeof(SelectState)) + align256(sizeof(unsigned long long) * kDigits) +
           align256(sizeof(long long) * nchunks);
}

// mask = the k largest of f[0..n) (ties to the lower index), 1 <= n, 0 <= k <= n;
// asynchronous on s.  The caller has validated the arguments and the workspace.
template <typename T>
int enqueue_top(const T *f, long long n, long long k, uint8_t *mask, void *ws, hipStream_t s)
{
    const unsigned grid = (unsigned)std::min<long long>(4096, (n + kThreads - 1) / kThreads);
    if (k == 0 || k == n) {
        hipLaunchKernelGGL(k_fill_u8, dim3(grid), dim3(kThreads), 0, s, mask, n, (uint8_t)(k == n ? 1 : 0));
        HIP_TRY(hipGetLastError());
        return MC_OK;
    }
    char *b = (char *)ws;
    SelectState *st = (SelectState *)b;
    unsigned long long *hist = (unsigned long long *)(b + align256(sizeof(SelectState)));
    long long *counts = (long long *)(b + align256(sizeof(SelectState)) + align256(sizeof(unsigned long long) * kDigits));
    // the candidates wait in the mask, which nothing reads before its bytes are written at the end
    char *const c0 = (char *)(((uintptr_t)mask + 15) & ~(uintptr_t)15);
    const long long room = (mask + n - (uint8_t *)c0) / 16;
    const long long cap = std::max(0ll, std::min<long long>(kCandidates, room));
    unsigned long long *keys = (unsigned long long *)c0;
    long long *index = (long long *)c0 + cap;
    const unsigned blocks = (unsigned)std::min<long long>(kDigitBlocks, (n + kDigitThreads - 1) / kDigitThreads);
    hipLaunchKernelGGL(k_init_state, dim3(1), dim3(kDigitThreads), 0, s, st, hist, n, k);
    // digits from the top: bits 63..53, 52..42, 41..31, 30..20, 19..9, 8..0
    for (int shift = 64 - kDigitBits; shift > -kDigitBits; shift -= kDigitBits) {
        const int sh = std::max(shift, 0);
        const int bits = shift >= 0 ? kDigitBits : kDigitBits + shift;
        hipLaunchKernelGGL(k_digit<T>, dim3(blocks), dim3(kDigitThreads), 0, s, f, n, st, hist, sh, bits, cap);
    }
    const long long nchunks = (n + kChunk - 1) / kChunk;
    hipLaunchKernelGGL(k_gather<T>, dim3(blocks), dim3(kDigitThreads), 0, s, f, n, st, keys, index, cap);
    hipLaunchKernelGGL(k_pick, dim3(1), dim3(kDigitThreads), 0, s, st, keys, index, n, cap);
    hipLaunchKernelGGL(k_count_eq<T>, dim3((unsigned)nchunks), dim3(kThreads), 0, s, f, n, st, counts);
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(kThreads), 0, s, st, counts, (int)nchunks);
    hipLaunchKernelGGL(k_mark<T>, dim3((unsigned)nchunks), dim3(kThreads), 0, s, f, n, st, counts, mask);
    HIP_TRY(hipGetLastError());
    return MC_OK;
}

}  // namespace
}  // namespace sel
}  // namespace pmc
