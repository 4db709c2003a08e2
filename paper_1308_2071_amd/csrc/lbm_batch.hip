// lbm_batch.hip -- one launch steps many independent cavities of uneven size and parameters.
//
// The cavities' states sit back to back in two population buffers.  The tiles of all cavities
// form one queue (cavity by cavity, tile row by tile row).  A tile -> cavity table and
// per-cavity geometry / parameter tables (read through the scalar cache: every work-item of a
// tile belongs to the same cavity) give each tile its setting.
// The per-node arithmetic is the plain step's (uniform medium per cavity), so every cavity's
// result is bitwise that of its own plain run.
#include "lbm_device.hpp"
#include "lbm_internal.hpp"
#include "lbm_tile.hpp"

namespace lbm {

// Tile = 64 * NPT consecutive nodes along x (one wavefront per 64) times TH rows (one
// wavefront per row), so narrow cavities still fill every wavefront.  CHUNKED: each
// work-group walks one contiguous run of the tile queue (consecutive tiles mostly share a
// cavity, so its parameters stay in the scalar cache); otherwise one tile per work-group.
// S: storage type, R: arithmetic type.
template <typename S, typename R, int TH, int NPT, bool CHUNKED>
__global__ __launch_bounds__(64 * TH) void batch_step_kernel(const S* __restrict__ src,
                                                             S* __restrict__ dst,
                                                             const BatchCavity* __restrict__ cav,
                                                             const Phys<R>* __restrict__ phys,
                                                             const int* __restrict__ tile_cav,
                                                             int ntiles) {
    int t0, t1;
    if constexpr (CHUNKED) {
        t0 = int((long long)ntiles * blockIdx.x / gridDim.x);
        t1 = int((long long)ntiles * (blockIdx.x + 1) / gridDim.x);
    } else {
        t0 = blockIdx.x;
        t1 = t0 + 1;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int t = t0; t < t1; ++t) {
        const int c = tile_cav[t];
        const BatchCavity C = cav[c];
        const Phys<R> P = phys[c];
        const int lt = t - C.tile0;
        const int ty = lt / C.tiles_x;
        const int y = ty * TH + wave;
        if (y >= C.G.ny) continue;
        const int x0 = (lt - ty * C.tiles_x) * (64 * NPT) + lane;
        const S* s = src + C.off;
        S* d = dst + C.off;
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int x = x0 + k * 64;
            if (x < C.G.nx) {
                R f[9], g[5];
                Mac<R> m;
                Med<R> md;
                node_state<R, false, S>(s, nullptr, C.G, P, x, y, f, g, m, md);
                collide<R>(f, g, m, md, P);
                const unsigned o =
                    (unsigned(y) * unsigned(C.G.pitch) + unsigned(x)) * unsigned(sizeof(S));
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    __builtin_nontemporal_store(S(f[i]), &at(plane(d, i, C.G.plane), o));
#pragma unroll
                for (int i = 0; i < 5; ++i)
                    __builtin_nontemporal_store(S(g[i]), &at(plane(d, 9 + i, C.G.plane), o));
            }
        }
    }
}

template <typename S, typename R, int TH, int NPT>
static hipError_t launch_v(const void* src, void* dst, const BatchTable<R>& T, int nwg,
                           hipStream_t s) {
    if (nwg >= T.ntiles)
        batch_step_kernel<S, R, TH, NPT, false><<<T.ntiles, 64 * TH, 0, s>>>(
            (const S*)src, (S*)dst, T.cav, T.phys, T.tile_cav, T.ntiles);
    else
        batch_step_kernel<S, R, TH, NPT, true><<<nwg, 64 * TH, 0, s>>>(
            (const S*)src, (S*)dst, T.cav, T.phys, T.tile_cav, T.ntiles);
    return hipGetLastError();
}

// Supported tile shapes: rows per work-group (work-group = 64 * rows work-items) and 64-node
// segments per work-item along x; nwg >= ntiles launches one tile per work-group, fewer runs
// the chunked persistent form.
template <typename S, typename R>
hipError_t launch_batch_step(const void* src, void* dst, const BatchTable<R>& T, int nodes_x,
                             int rows, int nwg, hipStream_t s) {
    switch (rows * 8 + nodes_x) {
        case 1 * 8 + 1: return launch_v<S, R, 1, 1>(src, dst, T, nwg, s);
        case 1 * 8 + 2: return launch_v<S, R, 1, 2>(src, dst, T, nwg, s);
        case 1 * 8 + 4: return launch_v<S, R, 1, 4>(src, dst, T, nwg, s);
        case 2 * 8 + 1: return launch_v<S, R, 2, 1>(src, dst, T, nwg, s);
        case 2 * 8 + 2: return launch_v<S, R, 2, 2>(src, dst, T, nwg, s);
        case 2 * 8 + 4: return launch_v<S, R, 2, 4>(src, dst, T, nwg, s);
        case 4 * 8 + 1: return launch_v<S, R, 4, 1>(src, dst, T, nwg, s);
        case 4 * 8 + 2: return launch_v<S, R, 4, 2>(src, dst, T, nwg, s);
        case 4 * 8 + 4: return launch_v<S, R, 4, 4>(src, dst, T, nwg, s);
        case 8 * 8 + 1: return launch_v<S, R, 8, 1>(src, dst, T, nwg, s);
        default: return hipErrorInvalidValue;
    }
}

// K steps per launch for every cavity: tiles of TX x TY nodes in LDS as in the single cavity's
// kernels, uniform medium per cavity.  The tiles of all cavities form one list, of which each XCD
// takes a contiguous run: wg_cav[t] is the cavity of tile t, C.tile0 its first tile and C.tiles_x
// its tiles along x.
template <typename S, typename R, int TX, int TY, int K, int NT>
__global__ __launch_bounds__(NT, (sizeof(R) == 8 ? 4 : NT > 896 ? 8 : 6)) void batch_tile_kernel(
    const S* __restrict__ src, S* __restrict__ dst, const BatchCavity* __restrict__ cav,
    const Phys<R>* __restrict__ phys, const int* __restrict__ wg_cav) {
    const int t = tile_index();
    const int c = wg_cav[t];
    const BatchCavity C = cav[c];
    const Phys<R> P = phys[c];
    const int lt = t - C.tile0, ty = lt / C.tiles_x;
    tile_steps_body<S, R, false, TX, TY, K, NT>(src + C.off, dst + C.off, (const S*)nullptr, C.G,
                                                P, lt - ty * C.tiles_x, ty);
}

template <typename S, typename R, int TX, int TY, int K>
static hipError_t launch_tiles(const void* src, void* dst, const BatchTable<R>& T,
                               hipStream_t s) {
    constexpr int NT = (TileRegion<TX, TY, K>::N + 63) / 64 * 64;
    constexpr size_t lds = tile_lds_bytes<S, R, false, TX, TY, K>();
    static_assert(lds <= 160 * 1024, "tile region exceeds the LDS of a CU");
    batch_tile_kernel<S, R, TX, TY, K, NT><<<T.ntiles, NT, lds, s>>>((const S*)src, (S*)dst,
                                                                     T.cav, T.phys, T.tile_cav);
    return hipGetLastError();
}

template <typename S, typename R, int TY>
static hipError_t launch_two_steps(const void* src, void* dst, const BatchTable<R>& T, int cols,
                                   hipStream_t s) {
    switch (cols) {
        case 62: return launch_tiles<S, R, 62, TY, 2>(src, dst, T, s);
        case 30: return launch_tiles<S, R, 30, TY, 2>(src, dst, T, s);
        case 14: return launch_tiles<S, R, 14, TY, 2>(src, dst, T, s);
        default: return hipErrorInvalidValue;
    }
}

template <typename S, typename R>
hipError_t launch_batch_tiles(const void* src, void* dst, const BatchTable<R>& T,
                              const BatchTile& f, hipStream_t s) {
    if (f.steps == 2 && f.cols == 28) {          // the remainder of three steps
        if (f.rows == 12) return launch_tiles<S, R, 28, 12, 2>(src, dst, T, s);
        if (f.rows == 28) return launch_tiles<S, R, 28, 28, 2>(src, dst, T, s);
    } else if (f.steps == 2 && f.cols == 16) {   // and of four
        if (f.rows == 16) return launch_tiles<S, R, 16, 16, 2>(src, dst, T, s);
    } else if (f.steps == 2) {
        switch (f.rows) {
            case 2: return launch_two_steps<S, R, 2>(src, dst, T, f.cols, s);
            case 3: return launch_two_steps<S, R, 3>(src, dst, T, f.cols, s);
            case 4: return launch_two_steps<S, R, 4>(src, dst, T, f.cols, s);
            case 5: return launch_two_steps<S, R, 5>(src, dst, T, f.cols, s);
            case 6: return launch_two_steps<S, R, 6>(src, dst, T, f.cols, s);
            case 8: return launch_two_steps<S, R, 8>(src, dst, T, f.cols, s);
            case 12: return launch_two_steps<S, R, 12>(src, dst, T, f.cols, s);
        }
    } else if (f.steps == 3 && f.cols == 28) {
        if (f.rows == 12) return launch_tiles<S, R, 28, 12, 3>(src, dst, T, s);
        if (f.rows == 28) return launch_tiles<S, R, 28, 28, 3>(src, dst, T, s);
    } else if (f.steps == 4 && f.cols == 16 && f.rows == 16) {
        return launch_tiles<S, R, 16, 16, 4>(src, dst, T, s);
    }
    return hipErrorInvalidValue;
}

template hipError_t launch_batch_step<float, float>(const void*, void*, const BatchTable<float>&,
                                                    int, int, int, hipStream_t);
template hipError_t launch_batch_step<double, double>(const void*, void*,
                                                      const BatchTable<double>&, int, int, int,
                                                      hipStream_t);
template hipError_t launch_batch_step<float, double>(const void*, void*,
                                                     const BatchTable<double>&, int, int, int,
                                                     hipStream_t);
template hipError_t launch_batch_tiles<float, float>(const void*, void*, const BatchTable<float>&,
                                                     const BatchTile&, hipStream_t);
template hipError_t launch_batch_tiles<double, double>(const void*, void*,
                                                       const BatchTable<double>&,
                                                       const BatchTile&, hipStream_t);
template hipError_t launch_batch_tiles<float, double>(const void*, void*,
                                                      const BatchTable<double>&,
                                                      const BatchTile&, hipStream_t);

}  // namespace lbm
