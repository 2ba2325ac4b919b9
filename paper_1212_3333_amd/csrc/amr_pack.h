// Device packing of cell-centred patches: what the host hands to the kernels of amr_pack.hip.
#pragma once
#include <stdint.h>

#include <vector>

#include "amr_internal.h"

namespace amr {

struct PackPatch {                   // one patch
    int64_t cells, shell, pool;      // first float of its staged cells, double of its shell, float of its brick
    int64_t floats;                  // brick floats with the padding to the next brick
    int64_t lo[3];                   // level cell coordinates of the lower corner
    int64_t blo[3], bhi[3];          // box in finest-level cells
    int64_t scale;                   // finest-level cells per cell
    int32_t n[3], nb[3];             // cells per axis; 4^3 blocks per axis of the padded brick
    int32_t level, nbr0, nbr1;       // its neighbours in PackPlan::nbr
    int32_t pad_;
};

struct PackLeaf {                    // cells that a sample of a leaf record can read, in padded terms:
    int32_t patch, lo[3], hi[3];     // index lo .. hi, both included, -1 and n the ghost layer
};

struct PackPlan {
    int layout = 0;
    int64_t B_lo[3], B_hi[3];        // the root box, finest-level cells
    int64_t cell_floats = 0, shell_doubles = 0, pool_floats = 0;
    std::vector<PackPatch> patches;
    std::vector<const float *> cells;            // per patch
    std::vector<int32_t> nbr;                    // patches of own or coarser level near each patch
    std::vector<std::vector<int32_t>> levels;    // patch ids per level
    std::vector<PackLeaf> leaves;                // per leaf record (patch -1: none)
};

// Shell (ghost layer) cells of a patch: the slabs k = -1 and n_z, then j = -1 and n_y, then i = -1 and n_x.
#ifdef __HIPCC__
#define AMR_HD __host__ __device__
#else
#define AMR_HD
#endif
AMR_HD inline int64_t shell_count(const int32_t *n) {
    const int64_t sx = n[0] + 2, sy = n[1] + 2;
    return 2 * (sx * sy + sx * n[2] + (int64_t)n[1] * n[2]);
}
AMR_HD inline int64_t shell_index(const int32_t *n, int64_t i, int64_t j, int64_t k) {
    const int64_t sx = n[0] + 2, sy = n[1] + 2;
    if (k < 0 || k >= n[2]) return (k < 0 ? 0 : sx * sy) + (j + 1) * sx + i + 1;
    int64_t base = 2 * sx * sy;
    if (j < 0 || j >= n[1]) return base + (j < 0 ? 0 : sx * n[2]) + k * sx + i + 1;
    base += 2 * sx * n[2];
    return base + (i < 0 ? 0 : (int64_t)n[1] * n[2]) + k * n[1] + j;
}

// Device memory that the packing needs besides pool and metadata, for the duration of the call.  It is
// allocated, filled and freed in the order of the caller's stream, so that a call waits for the work
// on that stream alone.  hipFree waits for the whole GPU, and a copy on a stream of one's own waits
// for whatever stream the runtime has put on the same hardware queue (there are four): with 2.5 s of
// other work on the GPU a pack of 10 ms took 2.5 s either way.  Four threads that copied, each on its
// own stream, saved 2.6 of 18.7 ms (250 patches, 60 M cells, tree build and pack); on one stream they
// save nothing.  The memory pool is the call's own: the GPU's default pool keeps what is freed into it.
struct PackStage {
    void *mem = nullptr, *stream = nullptr, *pool = nullptr;
    float *cells = nullptr;
    double *shell = nullptr;
    PackPatch *patches = nullptr;
    int32_t *nbr = nullptr, *ids = nullptr;
    PackLeaf *leaves = nullptr;
    float *ranges = nullptr;         // [np][2]
};

// False when the device has no room.  nleaves: an upper bound of plan.leaves.
bool pack_stage_alloc(const PackPlan &plan, int64_t nleaves, int device, void *stream, PackStage *st);
// The same for the neighbour list, once plan.nbr is known.
bool pack_stage_neighbours(const PackPlan &plan, PackStage *st);
// After the work on the stream; nothing to do where nothing was allocated.
void pack_stage_free(PackStage *st);
// Copies the patches' cells to the stage on GPU `device`, and waits.
int pack_upload_cells(const PackPlan &plan, const PackStage &st, int device);
// Uploads tables and metadata, fills the pool and the value ranges of the metadata's patch headers and
// leaf records, and waits; the range of all cells in *vmin, *vmax.
int pack_run(const PackPlan &plan, const PackStage &st, void *d_pool, void *d_meta, const void *meta, int64_t meta_bytes,
             int64_t o_leaves, int64_t o_patch, float *vmin, float *vmax, void *stream);

}  // namespace amr
