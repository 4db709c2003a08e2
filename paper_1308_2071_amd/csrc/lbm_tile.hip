// lbm_tile.hip -- several time steps per launch: each work-group advances one tile of the lattice
// K steps, with the states in between in LDS.
#include "lbm_device.hpp"
#include "lbm_internal.hpp"

namespace lbm {

// One step per launch pays, every step, the launch and a round trip of the state through memory.
// Here a work-group takes a tile of TX x TY nodes through K steps, bitwise as K launches of
// step_kernel would.  Step 1 runs on the region: the tile and a halo of K - 1 nodes on each open
// side (a side is closed where it is a wall of the grid; on a periodic axis both sides are open).
// Its populations are pulled straight from the step-n buffer and its results, rounded to the
// storage type as a store would round them, go to LDS with the region's medium coefficients,
// which are then worked out once per launch instead of once per step.  Each further step reads
// its populations from LDS and shrinks the active rectangle by one node on each open side, so
// that step K covers exactly the tile; its results go straight to the other buffer.  The first
// and last step thus touch LDS once, and two steps per launch (K = 2) need one barrier.
//
// Steps in between run in place: every active node pulls from LDS into registers, a barrier,
// every active node writes, a barrier.  One buffer instead of two halves the LDS, which sets how
// many work-groups a compute unit holds (two buffers and one barrier per step measured the same
// at best).
//
// What bounds it is vector instruction issue: about 330 slots per node and step, times the
// redundant steps of the halo (1.20 for 28 x 28 tiles advanced three steps, 1.33 for 28 x 12).
// So the active nodes of a step are dealt to the work-items anew, row by row, and no wavefront
// runs for a few nodes (one work-item per region node for the whole launch kept three wavefronts
// per SIMD busy to the end where this mapping needs two, then one); and the tile is the largest
// whose region still lets a compute unit hold two work-groups, one computing while the other
// waits for memory or at a barrier.
//
// Each XCD takes one contiguous run of tiles, row by row of the grid, so that a tile's halo is in
// its XCD's L2 (in launch order, neighbouring tiles on different XCDs: 256^2 FP32 2.75 us per
// step against 2.15; 1024^2 two steps per launch 20.5 against 13.4; blocks of 4, 8 or 16 tiles
// across within an XCD's run: 4096^2 206, 197 and 193 us per step against 187).
//
// A wall node uses the populations pulled at its inward neighbour, from the region: a node can
// take step s when its distance to the region's open sides is at least s - 1, a wall node when its
// inward neighbour's is.  A tile one node thick at an east (north) wall has its wall nodes' inward
// neighbours one node west (south) of it and takes one more halo node there; with it every wall
// node of the active rectangle may take the step.

template <int TX, int TY, int K>
struct TileRegion {
    static constexpr int W = TX + 2 * (K - 1), H = TY + 2 * (K - 1), N = W * H;
};

// LDS of a work-group: the state's planes and for a per-node medium the four
// coefficients in the arithmetic type.
template <typename S, typename R, bool PN, int TX, int TY, int K>
constexpr size_t tile_lds_bytes() {
    return size_t(TileRegion<TX, TY, K>::N) *
           (kPlanes * sizeof(S) + (PN ? 4 * sizeof(R) : 0));
}

// Global coordinate of a region coordinate r on an axis of n nodes (wrapped on a periodic axis).
__device__ __forceinline__ int tile_wrap(int r, int n, bool periodic) {
    if (!periodic) return r;
    r %= n;
    return r < 0 ? r + n : r;
}

// Tile of work-group blockIdx.x: each XCD (work-groups are dealt to the 8 of them in turn) takes a
// contiguous run of the tiles.
__device__ __forceinline__ int tile_index() {
    const int n = gridDim.x, xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    return xcd * (n / 8) + min(xcd, n % 8) + slot;
}

// K steps of tile (tx, ty); NT: work-items per work-group.
template <typename S, typename R, bool PN, int TX, int TY, int K, int NT>
__device__ __forceinline__ void tile_steps_body(const S* __restrict__ src, S* __restrict__ dst,
                                                const S* __restrict__ med, const Geo& G,
                                                const Phys<R>& P, int tx, int ty) {
    using Reg = TileRegion<TX, TY, K>;
    constexpr int W = Reg::W, L = Reg::N;
    static_assert(L <= NT, "one work-item per region node in step 1");
    extern __shared__ __align__(16) unsigned char tile_lds[];
    // coefficients first: doubles of R before the state's planes of S
    R* const ml = reinterpret_cast<R*>(tile_lds);
    S* const A = reinterpret_cast<S*>(tile_lds + (PN ? 4 * size_t(L) * sizeof(R) : 0));

    const int x0 = tx * TX, y0 = ty * TY;
    const int x1 = min(x0 + TX, G.nx), y1 = min(y0 + TY, G.ny);
    const int hW = K - 1 + ((x1 - x0 == 1 && G.wallE) ? 1 : 0);
    const int hS = K - 1 + ((y1 - y0 == 1 && G.wallN) ? 1 : 0);
    int rx0 = x0 - hW, rx1 = x1 + K - 1, ry0 = y0 - hS, ry1 = y1 + K - 1;
    int openW = 1, openE = 1, openS = 1, openN = 1;
    if (G.wallW && rx0 <= 0) { rx0 = 0; openW = 0; }
    if (G.wallE && rx1 >= G.nx) { rx1 = G.nx; openE = 0; }
    if (G.wallS && ry0 <= 0) { ry0 = 0; openS = 0; }
    if (G.wallN && ry1 >= G.ny) { ry1 = G.ny; openN = 0; }

    const int i = threadIdx.x;
    const float fi = float(i) + 0.5f;
    // this work-item's node of the current step, in the region's coordinates
    int lx, ly;
    bool onW, onE, onS, onN, wall, mine;
    int c, cf;   // LDS places of the node and of the node whose pulled populations it uses
    auto deal = [&](int s) {
        const int ax = openW ? s - 1 : 0, ay = openS ? s - 1 : 0;
        const int aw = (rx1 - rx0) - (openE ? s - 1 : 0) - ax;
        const int ah = (ry1 - ry0) - (openN ? s - 1 : 0) - ay;
        // row of work-item i: (i + 1/2) / aw is at least 1/(2 aw) from a whole number, far more
        // than the rounding of the reciprocal and the product for i < 1024
        const int row = int(fi * __builtin_amdgcn_rcpf(float(aw)));
        mine = row < ah;
        lx = ax + (i - row * aw);
        ly = ay + row;
        const int x = rx0 + lx, y = ry0 + ly;   // the grid's where the axis is walled
        onW = G.wallW && x == 0;
        onE = G.wallE && x == G.nx - 1;
        onS = G.wallS && y == 0;
        onN = G.wallN && y == G.ny - 1;
        wall = onW || onE || onS || onN;
        c = ly * W + lx;
        cf = c + (onW ? 1 : 0) - (onE ? 1 : 0) + (onS ? W : 0) - (onN ? W : 0);
    };
    auto uniform_medium = [&]() { return Med<R>{P.phi, P.inv_phi, P.c_lin, P.c_nl}; };
    // Macroscopics (node_state's arithmetic, once for fluid and wall nodes alike: both need the
    // pulled node's) and collision of this work-item's node
    auto finish = [&](R f[9], R g[5], const Med<R>& mdf, Med<R>& md, auto&& own_medium) {
        Mac<R> m = fluid_macros<R>(f, g, mdf, P);
        md = mdf;
        if (wall) {
            md = own_medium();
            m = wall_state<R>(onW, onE, onS, onN, f, g, m, mdf, md, P);
        }
        collide<R>(f, g, m, md, P);
    };

    // step 1, from the step-n buffer to LDS
    deal(1);
    if (mine) {
        const int gx = tile_wrap(rx0 + lx, G.nx, !G.wallW);
        const int gy = tile_wrap(ry0 + ly, G.ny, !G.wallS);
        const int px = gx + (onW ? 1 : 0) - (onE ? 1 : 0);
        const int py = gy + (onS ? 1 : 0) - (onN ? 1 : 0);
        R f[9], g[5];
        Med<R> md;
        const Med<R> mdf = load_medium<R, PN, S>(med, py * G.pitch + px, G.plane, P);
        pull<R, S>(src, G, px, py, f, g);
        finish(f, g, mdf, md, [&]() {
            return load_medium<R, PN, S>(med, gy * G.pitch + gx, G.plane, P);
        });
        if constexpr (PN) {
            ml[c] = md.phi;
            ml[L + c] = md.inv_phi;
            ml[2 * L + c] = md.c_lin;
            ml[3 * L + c] = md.c_nl;
        }
#pragma unroll
        for (int p = 0; p < 9; ++p) A[p * L + c] = S(f[p]);
#pragma unroll
        for (int p = 0; p < 5; ++p) A[(9 + p) * L + c] = S(g[p]);
    }
    __syncthreads();

    // pull streaming (Eqs. (18), (35)) from LDS, macroscopics and collision
    auto take = [&](R f[9], R g[5]) {
        const S* const a = A + cf;
        f[0] = R(a[0 * L]);
        f[1] = R(a[1 * L - 1]);
        f[2] = R(a[2 * L - W]);
        f[3] = R(a[3 * L + 1]);
        f[4] = R(a[4 * L + W]);
        f[5] = R(a[5 * L - W - 1]);
        f[6] = R(a[6 * L - W + 1]);
        f[7] = R(a[7 * L + W + 1]);
        f[8] = R(a[8 * L + W - 1]);
        g[0] = R(a[9 * L]);
        g[1] = R(a[10 * L - 1]);
        g[2] = R(a[11 * L - W]);
        g[3] = R(a[12 * L + 1]);
        g[4] = R(a[13 * L + W]);
        auto lds_medium = [&](int k) {
            if constexpr (PN)
                return Med<R>{ml[k], ml[L + k], ml[2 * L + k], ml[3 * L + k]};
            else
                return uniform_medium();
        };
        Med<R> md;
        finish(f, g, lds_medium(cf), md, [&]() { return lds_medium(c); });
    };
#pragma unroll 1
    for (int s = 2; s < K; ++s) {
        deal(s);
        R f[9], g[5];
        if (mine) take(f, g);
        __syncthreads();
        if (mine) {
#pragma unroll
            for (int p = 0; p < 9; ++p) A[p * L + c] = S(f[p]);
#pragma unroll
            for (int p = 0; p < 5; ++p) A[(9 + p) * L + c] = S(g[p]);
        }
        __syncthreads();
    }

    // step K, from LDS to the other buffer; unwrapped: the tile lies inside the grid
    deal(K);
    const int x = rx0 + lx, y = ry0 + ly;
    if (mine && x >= x0 && x < x1 && y >= y0 && y < y1) {
        R f[9], g[5];
        take(f, g);
        const unsigned o = (unsigned(y) * unsigned(G.pitch) + unsigned(x)) * unsigned(sizeof(S));
#pragma unroll
        for (int p = 0; p < 9; ++p) at(plane(dst, p, G.plane), o) = S(f[p]);
#pragma unroll
        for (int p = 0; p < 5; ++p) at(plane(dst, 9 + p, G.plane), o) = S(g[p]);
    }
}

// A form: tile, steps per launch, work-items per work-group, and the wavefronts per SIMD the
// kernel is compiled for with FP32 and with FP64 arithmetic.
template <int TX_, int TY_, int K_, int NT_, int W32_, int W64_>
struct TileForm {
    static constexpr int TX = TX_, TY = TY_, K = K_, NT = NT_;
    template <typename R>
    static constexpr int waves() { return sizeof(R) == 4 ? W32_ : W64_; }
};
using Tile8 = TileForm<kTinyTileSide, kTinyTileSide, kTinyTileSteps, 512, 2, 2>;
using Tile4 = TileForm<kTileSide, kTileSide, kTileSteps, 512, 4, 4>;
using Tile3 = TileForm<28, 12, 3, 512, 6, 4>;        // region 32 x 16
using Tile3Large = TileForm<28, 28, 3, 1024, 8, 4>;  // 32 x 32
using Tile2 = TileForm<30, 14, 2, 512, 6, 4>;        // 32 x 16
using Tile2Large = TileForm<62, 14, 2, 1024, 8, 4>;  // 64 x 16

#define LBM_TILE_KERNEL(name)                                                                   \
    template <typename S, typename R, bool PN, typename F>                                      \
    __global__ __launch_bounds__(F::NT, (F::template waves<R>())) void name(                    \
        const S* __restrict__ src, S* __restrict__ dst, const S* __restrict__ med, Geo G,       \
        Phys<R> P, int tiles_x) {                                                               \
        const int t = tile_index(), ty = t / tiles_x;                                           \
        tile_steps_body<S, R, PN, F::TX, F::TY, F::K, F::NT>(src, dst, med, G, P,               \
                                                             t - ty * tiles_x, ty);             \
    }
LBM_TILE_KERNEL(tile_step_kernel)   // four and eight steps
LBM_TILE_KERNEL(tb3_step_kernel)    // three
LBM_TILE_KERNEL(tb2_step_kernel)    // two
#undef LBM_TILE_KERNEL

// Steps per launch of the time loop by default.  The halo's redundant work grows with the steps
// and shrinks with the tile, the launches and the bytes per step fall with the steps.  Measured,
// us per step on porous cavities, uniform / per-node medium:
//                          8 x 8, 8    16 x 16, 4  28 x 12, 3  28 x 28, 3  30 x 14, 2
//   FP32          128^2    1.46 1.51   1.95 1.94   2.13 2.17   3.27 3.37   2.49 2.58
//                 192^2    2.11 2.21   1.97 1.97   2.14 2.20   3.35 3.38   2.57 2.64
//                 512^2    8.22 8.50   4.11 4.26   4.54 4.56   5.27 5.43   4.56 4.69
//                 1024^2   29.5 30.7   11.8 12.4   11.3 12.0   12.1 12.5   12.2 12.7
//                 2048^2   114  119    47.0 50.1   45.2 49.2   43.7 46.0   54.6 58.4
//                 4096^2   450  472    188  201    182  198    163  178    224  242
//   FP64          128^2    1.85 1.93   2.67 2.80   2.91 3.18               3.42 3.70
//                 256^2    4.58 4.86   2.85 2.98   3.14 3.43               3.73 4.08
//                 517 x 389 11.8 12.5  6.43 6.86   6.25 6.77               6.20 6.66
//                 1024^2   53.9 57.6   21.8 23.4   20.0 21.6               21.3 24.3
//                 4096^2   829  921    325  373    302  368                408  444
//   FP32 storage, 128^2    1.78 2.00   2.53 2.71   2.94 3.11               3.25 3.53
//   FP64          256^2    4.54 4.96   2.54 2.74   2.97 3.18               3.31 3.62
//   arithmetic    517 x 389 12.2 12.9  6.10 6.48   5.80 6.16               4.99 5.48
//                 1024^2   57.8 60.5   21.6 22.9   19.0 20.2               16.0 19.4
//                 4096^2   885  953    302  328    265  297                244  311
// One step per launch takes 2 to 3 times as long on the smallest of these and 1.1 to 1.9 times on
// the largest.  Per-node media from 1024^2 to 1536^2 in FP32, and from 4096^2 in FP64, keep two
// steps per launch, which lbm_step_shape has long reported for these grids (three would run
// 6 to 20 % faster).
constexpr long long kTinyTileMaxNodes = 128LL * 128;

template <typename S, typename R>
int default_steps(const Geo& G, bool per_node_medium) {
    const long long n = (long long)G.nx * G.ny;
    if (n <= kTinyTileMaxNodes) return kTinyTileSteps;
    if (sizeof(R) == 4) {
        if (n <= 700000) return kTileSteps;
        return per_node_medium && n >= 1024LL * 1024 && n <= 1536LL * 1536 ? 2 : 3;
    }
    if (sizeof(S) == 4) return n <= 110000 ? kTileSteps : 2;
    if (n <= 150000) return kTileSteps;
    return per_node_medium && n >= 4096LL * 4096 ? 2 : 3;
}

// Where two or three steps per launch take their larger tile: from the size on where the launch
// has several rounds of work-groups, so that fewer, larger ones cost no balance (28 x 28 against
// 28 x 12, FP32: 1024^2 12.1 against 11.3 us per step, 1536^2 23.5 against 22.4 and with a
// per-node medium 26.0 against 27.3, 4096^2 163 against 182; in FP64 the larger region leaves a
// compute unit one work-group: 4096^2 358 against 302.  62 x 14 against 30 x 14, FP32: 1024^2
// 12.8 against 12.2, 4096^2 202 against 224).
constexpr long long kLargeTileNodes = 1536LL * 1536;

template <typename S, typename R, typename F, typename Go>
auto tile_grid(const Geo& G, Go&& go) {
    const int tiles_x = (G.nx + F::TX - 1) / F::TX;
    return go(F{}, tiles_x, tiles_x * ((G.ny + F::TY - 1) / F::TY));
}

// Calls go(form, tiles along x, work-groups) with the form that takes k steps on grid G.
template <typename S, typename R, typename Go>
auto with_form(const Geo& G, int k, Go&& go) {
    const bool large = (long long)G.nx * G.ny >= kLargeTileNodes;
    if (k == kTinyTileSteps) return tile_grid<S, R, Tile8>(G, go);
    if (k == kTileSteps) return tile_grid<S, R, Tile4>(G, go);
    if (k == 3) {
        if constexpr (sizeof(R) == 4) {
            if (large) return tile_grid<S, R, Tile3Large>(G, go);
        }
        return tile_grid<S, R, Tile3>(G, go);
    }
    return large ? tile_grid<S, R, Tile2Large>(G, go) : tile_grid<S, R, Tile2>(G, go);
}

template <typename S, typename R>
void tile_shape(const Geo& G, int k, int* rows, int* nwg) {
    with_form<S, R>(G, k, [&](auto f, int, int n) {
        *rows = decltype(f)::TY;
        *nwg = n;
        return 0;
    });
}

template <typename S, typename R, bool PN, typename F>
static hipError_t launch_form(const void* src, void* dst, const void* med, const Geo& G,
                              const Phys<R>& P, int tiles_x, int nwg, hipStream_t s) {
    constexpr size_t lds = tile_lds_bytes<S, R, PN, F::TX, F::TY, F::K>();
    static_assert(lds <= 160 * 1024, "tile region exceeds the LDS of a CU");
    if constexpr (F::K == 2)
        tb2_step_kernel<S, R, PN, F><<<nwg, F::NT, lds, s>>>((const S*)src, (S*)dst,
                                                             (const S*)med, G, P, tiles_x);
    else if constexpr (F::K == 3)
        tb3_step_kernel<S, R, PN, F><<<nwg, F::NT, lds, s>>>((const S*)src, (S*)dst,
                                                             (const S*)med, G, P, tiles_x);
    else
        tile_step_kernel<S, R, PN, F><<<nwg, F::NT, lds, s>>>((const S*)src, (S*)dst,
                                                              (const S*)med, G, P, tiles_x);
    return hipGetLastError();
}

template <typename S, typename R>
hipError_t launch_tile_step(const void* src, void* dst, const void* med, const Geo& G,
                            const Phys<R>& P, int k, hipStream_t s) {
    if (k != 2 && k != 3 && k != kTileSteps && k != kTinyTileSteps) return hipErrorInvalidValue;
    return with_form<S, R>(G, k, [&](auto f, int tiles_x, int nwg) {
        using F = decltype(f);
        return med ? launch_form<S, R, true, F>(src, dst, med, G, P, tiles_x, nwg, s)
                   : launch_form<S, R, false, F>(src, dst, nullptr, G, P, tiles_x, nwg, s);
    });
}

#define LBM_TILE_INST(S, R)                                                                    \
    template int default_steps<S, R>(const Geo&, bool);                                        \
    template void tile_shape<S, R>(const Geo&, int, int*, int*);                               \
    template hipError_t launch_tile_step<S, R>(const void*, void*, const void*, const Geo&,    \
                                               const Phys<R>&, int, hipStream_t);
LBM_TILE_INST(float, float)
LBM_TILE_INST(double, double)
LBM_TILE_INST(float, double)
#undef LBM_TILE_INST

}  // namespace lbm
