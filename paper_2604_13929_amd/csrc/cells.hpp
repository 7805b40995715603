// The cell walk: large runs walk their photons through one cell of the volume at a time, the cell's
// mask and tally held in LDS (cells.hip).  Interface to the runs (photonmc.hip) and the batch (batch.hip).
#pragma once
#include "internal.hpp"

namespace pmc {
namespace host {

// The cells of one job's volume.
struct CellDims {
    int32_t ncx, ncy, ncz;      // cells along each axis
    int32_t ex, ey, ez;         // voxels of a cell along each axis (the last cell may hold fewer)
    int32_t zlo;                // first z layer walked in: -1 (the top air pad) under the paper's boundary model, else 0
    uint64_t cells;
};
CellDims cell_dims(const mc_volume *vol, bool paper);

// Scratch a cell walk of so many photons makes full use of; 0 if it would not be taken.
size_t cell_workspace_bytes(const CellDims *dims, int32_t n_jobs, uint64_t photons);

struct CellRun {
    const Job *table;           // host, n_jobs entries in queue order, every pointer set
    int32_t n_jobs;
    uint64_t photons;           // of all jobs
    bool general, fp64;
    unsigned long long *grad;   // device score bins, or NULL (one job only)
    const BatchEsc *esc;        // device, one per job of the table, or NULL
    const BatchEsc *hist;       // host: a single run's histogram without its copies, or NULL
    char *ws;
    size_t ws_bytes;
    bool batch;
    bool always;                // MC_CELLS: wherever it can, not where it is faster
};
// Whether this run walks in cells: it can, and it is faster that way with this scratch.
bool cell_walk_fits(const CellRun &r);
// The walk alone: tallies and staging tallies zeroed and masks packed beforehand, the staging tallies
// (which the tail logs into) added to the fluence afterwards.
int cell_walk(const CellRun &r, hipStream_t s);

}  // namespace host
}  // namespace pmc
