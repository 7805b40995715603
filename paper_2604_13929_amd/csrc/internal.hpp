// Host-side helpers shared by the translation units of the library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "photonmc.h"
#include "walk.hpp"

struct EscHist;  // the escape-path histogram of a walk (photonmc.hip)

namespace pmc {

// The escape-path histogram of one job (table order), NULL w: none.  Read only
// when a photon escapes, so it stays in global memory, not in the LDS job table.
// The walk adds into kEscReplicas copies in the workspace, a workgroup's copy
// chosen by its index: a batch runs its jobs longest first, so at any time most
// of the chip's escapes go to a few bins of one job, and one 64-byte line takes
// only ~1e8 atomics per second at the memory side.  k_esc_fold adds the copies
// into the caller's bins after the walk.
constexpr int kEscReplicas = 16;
struct BatchEsc {
    unsigned long long *w;    // [nbins] escaped Q31 weight (the caller's)
    unsigned long long *n;    // [nbins] escaped photons (the caller's)
    unsigned long long *rw;   // [kEscReplicas][kEscMaxBins] copies of w (workspace)
    unsigned long long *rn;   // [kEscReplicas][kEscMaxBins] copies of n (workspace)
    double width;
    int32_t nbins;
    int32_t pad;
};

namespace host {

int fail(int status, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

#define HIP_TRY(expr)                                                                                    \
    do {                                                                                                 \
        hipError_t e_ = (expr);                                                                          \
        if (e_ != hipSuccess) return ::pmc::host::fail(MC_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

constexpr size_t kHeaderBytes = 256;  // queue counter(s) at the start of a run workspace
constexpr int kBinW = 8;              // int64 words per depth bin of the reduction
constexpr int kEscMaxBins = 512;      // escape-path bins; 6 KB of LDS leaves four walk workgroups per CU
// A walk stages its deposits in the plane layout (three tables) where those fit in
// this many bytes, else in the line layout (one table): tripled, the 256^3 tally
// stays within the 256 MiB Infinity Cache, beyond which memory-side atomics slow
// down.
#ifndef MC_PLANE_STAGE_MAX_BYTES
#define MC_PLANE_STAGE_MAX_BYTES (192ull << 20)
#endif
constexpr uint64_t kPlaneStageMaxBytes = MC_PLANE_STAGE_MAX_BYTES;

struct Dims {
    int32_t nxb, nyb, nzb;       // 4x4x4 mask bricks
    uint64_t nbricks, nvox;
    int32_t lnx, lny, lnz;       // staging lines of 2x2x4 voxels (line layout)
    uint64_t line_words;         // uint32 words of the line layout
    bool planes;                 // the single-run walk stages in the plane layout
    uint64_t stage_words;        // uint32 words of the single-run walk's staging tally
    bool logged;                 // the staging tally fits 32-bit indices
};
size_t run_workspace_bytes(const Dims &d);
size_t stage_offset(const Dims &d);
Dims dims_of(const mc_volume *v);
int check_volume(const mc_volume *v);
int make_job(const mc_volume *vol, const mc_optics *opt, uint64_t photon_begin, uint64_t n_photons, uint64_t seed,
             uint32_t stream_id, Job *J);

struct DeviceInfo {
    int cus = 0;
};
int device_info(DeviceInfo *out);

// The launch shape: the caller's fields where > 0, else the defaults, with defer_default
// (when > 0) in place of the plain walk's default defer.
mc_tune resolve_tune(const mc_tune *t, int32_t defer_default = 0);
// The default defer of a walk: the gradient walk, the paper's boundary model and the FP64
// transport are bound by their VALU and run their interactions in larger groups.
constexpr int32_t kDeferVALUBound = 8;
int check_tune(const mc_tune &t);
// What a walk of so many wavefronts does with a tune for so many photons.  With fewer photons than
// lanes every wavefront takes its even share and no more lanes than that: a wavefront of one photon
// steps in 0.7 us, one of 64 in 1.3 to 3 us, and the run lasts as long as its longest photon.  Few
// lanes also wait less for each other's interactions; a full wavefront waits for as many as the tune says.
struct WalkShape {
    int32_t cap, chunk, refill, defer;
};
inline WalkShape walk_shape(const mc_tune &t, uint64_t waves, uint64_t photons)
{
    const uint64_t share = std::max<uint64_t>(1, (photons + waves - 1) / waves);
    WalkShape s;
    s.cap = (int32_t)std::min<uint64_t>(64, share);
    s.chunk = (int32_t)std::min<uint64_t>((uint64_t)t.chunk, share);
    s.refill = std::min(t.refill, s.cap);
    s.defer = s.cap < 64 ? std::min(t.defer, std::max(1, s.cap / 8)) : t.defer;
    return s;
}

// asynchronous building blocks on a stream
int fill(int64_t *p, uint64_t n, hipStream_t s);
int pack(const mc_volume *vol, uint64_t *bricks, hipStream_t s);
int unstage(const uint32_t *stage, int64_t *fluence, const mc_volume *vol, bool planes, hipStream_t s);
// zero (unless accumulating), pack, walk and move the staged tally into the caller's
// fluence, with the queue, packed mask and staging tally in the workspace ws
// (cells, cells_bytes: scratch of the cell walk, or NULL)
int run_walk(const mc_volume *vol, Job J, int flags, const mc_tune &t, char *ws, char *cells, size_t cells_bytes,
             unsigned long long *grad_bins, hipStream_t s, const EscHist *esc = nullptr);
// the histogram table's entries from the host, and the copies added into the callers' bins
int write_esc(const BatchEsc *e, int32_t n, BatchEsc *dst, hipStream_t s);
int fold_esc(const BatchEsc *table, int32_t n, hipStream_t s);
int enqueue_reduce(const mc_volume *vol, const int64_t *fluence, const int64_t *scalars, double *summary,
                   double *depth, unsigned long long *bins, hipStream_t s);

// the walk-kernel timer (MC_TIMED)
struct Timing {
    hipEvent_t start = nullptr, stop = nullptr;
    bool armed = false;
};
Timing &timing();
int time_begin(hipStream_t s);
int time_end(hipStream_t s);

}  // namespace host
}  // namespace pmc
