// lbm_internal.hpp -- launchers shared between the ABI (lbm_abi.cpp) and the kernel files.
#pragma once

#include <hip/hip_runtime.h>

#include "lbm_device.hpp"

namespace lbm {

constexpr int kTileX = 256;      // nodes (work-items) per work-group of the step kernel
constexpr int kObserveWG = 508;  // most work-groups of the observables pass over the nodes
constexpr int kBatchObsWG = 60;  // most of them for one cavity of a batch
constexpr int kObsThreads = 512; // most work-items per work-group of the observables pass
constexpr int kNuWG = 12;        // most work-groups of the walls' Nusselt sums
constexpr int kObsParts = 6;     // partial results per work-group of the observables pass
constexpr int kObsOut = 2 + kObsParts;  // results of the observables pass (Nu sums, ...)
constexpr int kPitchAlign = 64;  // row pitch in elements
// Elements between the end of one plane's rows and the start of the next (4 KiB + 128 B in
// FP32).  Without it the planes of a 4096-wide power-of-two grid lie exactly 64 MiB apart and
// the 14 + 2 streams of a row fall on the same memory channel and bank; with it the two-step
// kernel on the 4096^2 workload ran 1-2 % faster (71.5k against 69.5k-70.7k MLUPS, with the
// same fetched bytes).  A stride of +64 or +4160 elements measured within 0.5 % of this one.
constexpr int kPlanePad = 1056;

// Elements per plane: ny rows of the pitch, then the pad.
inline long long plane_elems(long long pitch, long long ny) { return pitch * ny + kPlanePad; }

// Tiles of the batch: columns and rows, steps per launch, and the code that goes with the rows in
// the tuner's cache (1, 2 and 4: two steps, a region of 64 / code columns; 3: more steps).
struct BatchTile {
    int cols, rows, steps, code;
};
constexpr BatchTile kBatchTiles[] = {
    {62, 2, 2, 1}, {30, 2, 2, 2}, {14, 2, 2, 4}, {62, 3, 2, 1}, {30, 3, 2, 2}, {14, 3, 2, 4},
    {62, 4, 2, 1}, {30, 4, 2, 2}, {14, 4, 2, 4}, {62, 5, 2, 1}, {30, 5, 2, 2}, {14, 5, 2, 4},
    {62, 6, 2, 1}, {30, 6, 2, 2}, {14, 6, 2, 4}, {62, 8, 2, 1}, {30, 8, 2, 2}, {14, 8, 2, 4},
    {62, 12, 2, 1}, {30, 12, 2, 2}, {14, 12, 2, 4},
    {28, 12, 3, 3}, {28, 28, 3, 3}, {16, 16, 4, 3},
};
constexpr int kBatchMinCols = 14, kBatchMinRows = 2;

// Tile side and steps per launch of the forms for small grids (lbm_tile.hip).
constexpr int kTileSide = 16;
constexpr int kTileSteps = 4;
constexpr int kTinyTileSide = 8;
constexpr int kTinyTileSteps = 8;

// What steps_per_launch = 2 asks of a state: 1 where its 14 planes, 2 where only each half of them
// (7 planes) is below 2 GiB, 0 beyond.
inline int tb2_halves(const Geo& G, size_t elem_bytes) {
    const unsigned long long pb = (unsigned long long)G.plane * elem_bytes;
    if (kPlanes * pb < (1ull << 31)) return 1;
    if (kPlanes / 2 * pb < (1ull << 31)) return 2;
    return 0;
}

// Launchers take S, the storage type of populations and medium planes, and R, the arithmetic
// type; instantiated for (float, float), (double, double) and (float, double).

template <typename S, typename R>
hipError_t launch_step(const void* src, void* dst, const void* med, const Geo& G,
                       const Phys<R>& P, hipStream_t s);
// Steps per launch of the time loop that are fastest for this grid and these types
template <typename S, typename R>
int default_steps(const Geo& G, bool per_node_medium);
// Steps per launch of the adjoint's recompute in segments of so many steps
template <typename S, typename R>
int recompute_steps(const Geo& G, bool per_node_medium, int segment);
// k (2, 3, kTileSteps or kTinyTileSteps) steps of the pull layout in one launch from src to dst,
// each tile of the grid advanced in LDS
template <typename S, typename R>
hipError_t launch_tile_step(const void* src, void* dst, const void* med, const Geo& G,
                            const Phys<R>& P, int k, hipStream_t s);
// The same, keeping every state: step s at dst + (s - 1) * stride (elements)
template <typename S, typename R>
hipError_t launch_tile_trace(const void* src, void* dst, size_t stride, const void* med,
                             const Geo& G, const Phys<R>& P, int k, hipStream_t s);
// Rows per tile and work-groups per launch of launch_tile_step
template <typename S, typename R>
void tile_shape(const Geo& G, int k, int* rows, int* nwg);
// AA-pattern step in place; parity 0: the state is in the kAAOpp form, 1: kAAOwn
template <typename S, typename R>
hipError_t launch_aa_step(void* buf, const void* med, const Geo& G, const Phys<R>& P,
                          int parity, hipStream_t s);
// Work-groups of launch_step, or of launch_aa_step
int one_step_groups(const Geo& G, size_t elem_bytes, bool aa);
// layout: the PopLayout form the state is in.  Fields (each may be NULL), and with part (room for
// kObsParts * kObserveWG + 2 * kNuWG doubles) the kObsOut results at out: the unscaled sums of Eq.
// (38) at the west and east walls, max |u|, sum f', non-finite flag, min T, max T, max
// |phi p - rho0 cs^2|.
template <typename S, typename R>
hipError_t launch_observe(const void* src, const void* med, const Geo& G, const Phys<R>& P,
                          int layout, void* ux, void* uy, void* p, void* T, double* part,
                          double* out, hipStream_t s);
template <typename S, typename R>
hipError_t launch_stream_function(const void* src, const void* med, const Geo& G,
                                  const Phys<R>& P, int layout, void* psi, hipStream_t s);
template <typename R>
hipError_t launch_rest(void* dst, const Geo& G, double g0, double g1, hipStream_t s);
template <typename R>
hipError_t launch_pitch_copy(void* dst, const void* src, const Geo& G, double v, hipStream_t s);

// Adjoint (lbm_adjoint.hip)
template <typename S, typename R>
hipError_t launch_adjoint_seed(const void* state, void* lam, const Geo& G, const Phys<R>& P,
                               double L_over_dT, hipStream_t s);
template <typename S, typename R>
hipError_t launch_adjoint_step(const void* state, const void* lam_in, void* lam_out,
                               const void* med, double* gphi, double* gK, const Geo& G,
                               const Phys<R>& P, hipStream_t s);
// Whether kAdjSteps backward steps per launch are faster than one (small grids, not FP64 arithmetic
// on FP32 storage)
template <typename S, typename R>
bool adjoint_by_tiles(const Geo& G);
// kAdjSteps backward steps in one launch, each tile of kAdjSide^2 nodes in LDS; states: X^n,
// X^{n-1}, ...; lam_in: adjoint of X^{n+1}; lam_out: adjoint of the last of the states
constexpr int kAdjSide = 16, kAdjSteps = 3;
template <typename S, typename R>
hipError_t launch_adjoint_tiles(const void* const states[kAdjSteps], const void* lam_in,
                                void* lam_out, const void* med, double* gphi, double* gK,
                                const Geo& G, const Phys<R>& P, hipStream_t s);
template <typename R>
hipError_t launch_fill(void* dst, size_t n, hipStream_t s);
hipError_t launch_fill_f64(double* dst, size_t n, hipStream_t s);
hipError_t launch_unpitch_scale(double* dst, const double* src, const Geo& G, double scale,
                                hipStream_t s);

// Batched form (lbm_batch.hip)
struct BatchCavity {
    Geo G;
    long long off;     // element offset of the cavity's state inside a state buffer
    int tile0;         // first tile id of the cavity
    int tiles_x;       // tiles along x
};

template <typename R>
struct BatchTable {
    const BatchCavity* cav;  // device array [n]
    const Phys<R>* phys;     // device array [n]
    const int* tile_cav;     // device array [ntiles]: cavity of each tile
    int ncav;
    int ntiles;
};

// f.steps steps per launch for every cavity of a batch, in tiles f: one of kBatchTiles, or one of
// those with three or four steps for two steps.
// T.tile_cav maps each of the T.ntiles tiles to its cavity, whose tile0 is its first tile and
// tiles_x its tiles along x.
template <typename S, typename R>
hipError_t launch_batch_tiles(const void* src, void* dst, const BatchTable<R>& T,
                              const BatchTile& f, hipStream_t s);

// Observables of every cavity (no fields): results of cavity i at out[kObsOut * i]; part has room
// for kObsParts * kBatchObsWG + 2 * kNuWG doubles per cavity; largest: nodes of the largest one.
template <typename S, typename R>
hipError_t launch_batch_observe(const void* src, const BatchTable<R>& T, long long largest,
                                double* part, double* out, hipStream_t s);

// rows: rows per tile (work-group = 64 * rows work-items); nodes_x: 64-node segments per
// work-item along x; nwg >= ntiles: one tile per work-group, else chunked persistent.
template <typename S, typename R>
hipError_t launch_batch_step(const void* src, void* dst, const BatchTable<R>& T, int nodes_x,
                             int rows, int nwg, hipStream_t s);

}  // namespace lbm
