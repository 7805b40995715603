// The deposit log of the walks that carry several jobs, device side.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "walk.hpp"

namespace pmc {

// Line-coalesced deposits for the batch: as the plain walk's log (8-byte
// entries, 16 slots per lane, issued transposed once some lane has filled its
// slots, the run of entries in the line a photon still deposits into held back,
// uint32 staging words in each job's own layout, planes or lines, carries of
// wrapped words into the job's int64 tally).  Where a launch carries several jobs (JOBS)
// the job index takes the top 6 bits of the 32-bit entry index, which leaves 26 bits
// for the word index into the job's staging tally (such a launch logs only when every
// job's staging tally is that small); a job alone has all 32 bits for the word.  A deposit of 2^31 quanta or more goes to the job's tally directly.  The
// log's 33 KB of LDS per 256-thread workgroup, with the job table and the per-job
// channels, still lets three workgroups share a CU.
constexpr int kBLogK = 16;
constexpr int kBLogStride = 65;
#ifndef MC_LOG_HOLD
#define MC_LOG_HOLD 6
#endif
constexpr int kBLogHold = MC_LOG_HOLD;
constexpr uint32_t kBNoLine = 0xFFFFFFFFu;
constexpr int kJobShift = 26;
constexpr uint32_t kIdxMask = (1u << kJobShift) - 1u;
constexpr uint64_t kBatchLogWords = 1ull << kJobShift;   // largest staging tally a logged batch job may have

// The job's bits of an entry's index, and an entry's job and word.
template <bool JOBS> __host__ __device__ __forceinline__ uint32_t log_tag(int32_t job) { return JOBS ? (uint32_t)job << kJobShift : 0u; }
template <bool JOBS> __host__ __device__ __forceinline__ uint32_t log_job(uint32_t e) { return JOBS ? e >> kJobShift : 0u; }
template <bool JOBS> __host__ __device__ __forceinline__ uint32_t log_word(uint32_t e) { return JOBS ? e & kIdxMask : e; }
// The largest staging tally the entries of a launch of so many jobs can index.
inline uint64_t log_words(int32_t n_jobs) { return n_jobs > 1 ? kBatchLogWords : 1ull << 32; }
// The words of a job's staging tally.
inline uint64_t stage_words(const Job &J)
{
    if (J.stage_planes) return plane_dims(J.nx, J.ny, J.nz).words;
    return (uint64_t)J.lnx * (uint64_t)J.lny * (((uint64_t)J.nz + 3) / 4) * 16;
}

struct BatchLoggedSink {
    uint32_t *lidx;
    uint32_t *lval;
    uint32_t lane;
    uint32_t head, count;       // this lane's ring of kBLogK slots
    uint32_t tag;               // log_tag of the job
    template <typename R> __device__ __forceinline__ void segment(const Photon<R> &, const Job &, R, bool) {}
    template <typename R> __device__ __forceinline__ void deflect(Photon<R> &, const Job &, R) {}
    template <typename R> __device__ __forceinline__ void flush(const Job &J, const Photon<R> &p, uint64_t a)
    {
        if (a != 0ull) {
            if (a >> 31) {
                __hip_atomic_fetch_add((unsigned long long *)(J.fluence + voxel_index(J, p)),
                                       (unsigned long long)a << kDepositShift, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            } else {
                const uint32_t s = log_slot<kBLogStride, kBLogK>(lane, head, count);
                lidx[s] = stage_word(J, p) | tag;
                lval[s] = (uint32_t)a;
                ++count;
            }
        }
    }
};

// Issue the wavefront's log; HOLD: the newest run of each lane's log that lies in
// `line` (job bits included; kBNoLine: none) stays as the lane's ring.  The FP64
// transport holds nothing.
template <bool HOLD, bool JOBS>
__device__ __forceinline__ void flush_batch_log(uint32_t *lidx, uint32_t *lval, const Job *jobs, uint32_t lane,
                                                uint32_t line, uint32_t &head, uint32_t &count)
{
    const uint32_t held = HOLD ? log_mark_run<kBLogStride, kBLogK, kBLogHold>(lidx, lval, lane, head, count, line) : 0u;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // in two halves, each issuing its adds before it looks at what they returned
#pragma unroll
    for (int h = 0; h < kBLogK; h += kBLogK / 2) {
        uint32_t old[kBLogK / 2];
#pragma unroll
        for (int i = 0; i < kBLogK / 2; ++i) {
            const uint32_t src = (uint32_t)(h + i) * (64 / kBLogK) + lane / kBLogK;
            const uint32_t e = (lane % kBLogK) * kBLogStride + src;
            const uint32_t v = lval[e];
            old[i] = 0u;
            if (v != 0u && (!HOLD || v < kLogHeld)) {
                const uint32_t w = lidx[e];
                old[i] = __hip_atomic_fetch_add(jobs[log_job<JOBS>(w)].stage + log_word<JOBS>(w), v, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
            }
        }
#pragma unroll
        for (int i = 0; i < kBLogK / 2; ++i) {
            const uint32_t src = (uint32_t)(h + i) * (64 / kBLogK) + lane / kBLogK;
            const uint32_t e = (lane % kBLogK) * kBLogStride + src;
            const uint32_t v = lval[e];
            if (v != 0u && (!HOLD || v < kLogHeld)) {
                if (old[i] > 0xFFFFFFFFu - v) {
                    // the word wrapped: its lost 2^32 quanta go to the voxel's int64 word
                    const uint32_t w = lidx[e];
                    const Job &J = jobs[log_job<JOBS>(w)];
                    __hip_atomic_fetch_add((unsigned long long *)(J.fluence + stage_voxel(J, log_word<JOBS>(w))),
                                           1ull << (32 + kDepositShift), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                lval[e] = 0u;
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (HOLD) {
        log_keep_run<kBLogStride, kBLogK, kBLogHold>(lval, lane, head, count, held);
    } else {
        head = 0u;
        count = 0u;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

}  // namespace pmc
