// lbm_tile.hpp -- several time steps per launch: each work-group advances one tile of the lattice
// K steps, with the states in between in LDS.  Shared by the single cavity and the batch.
#pragma once

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
// many work-groups a compute unit holds (two buffers and one barrier per step were no faster where
// several share a compute unit; on grids of at most one tile per compute unit a sweep of forms showed
// 8 %, which is not built).
//
// What bounds it is vector instruction issue: 289 slots per node and step in the one-step kernel (FP32),
// times the redundant steps of the halo (1.15 times the nodes for 28 x 28 tiles advanced three steps,
// 1.26 for 28 x 12; in whole wavefronts 1.25 and 1.40 as mapped here), plus the LDS: 375 slots per node
// and step of 28 x 28 tiles with a per-node medium.  So the active nodes of a step are dealt to the
// work-items anew, row by row, and no wavefront runs for a few nodes (one work-item per region node for
// the whole launch kept three wavefronts per SIMD busy to the end where this mapping needs two, then
// one), except where a region's rows are half wavefronts (kKept below); and the tile is the largest
// whose region still lets a compute unit hold two work-groups, one computing while the other
// waits for memory or at a barrier (but 62 x 14 in FP64, on grids where its size pays all the same).
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

// K steps of tile (tx, ty) from src to dst; NT: work-items per work-group.  EVERY: the states in
// between are kept too, step s at dst + (s - 1) * stride (elements); otherwise stride is unused.
template <typename S, typename R, bool PN, int TX, int TY, int K, int NT, bool EVERY = false>
__device__ __forceinline__ void tile_steps_body(const S* __restrict__ src, S* __restrict__ dst,
                                                const S* __restrict__ med, const Geo& G,
                                                const Phys<R>& P, int tx, int ty,
                                                size_t stride = 0) {
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
    // this work-item's node of the current step, in the region's coordinates
    int lx, ly;
    bool onW, onE, onS, onN, wall, mine;
    int c, cf;   // LDS places of the node and of the node whose pulled populations it uses
    auto place = [&]() {
        const int x = rx0 + lx, y = ry0 + ly;   // the grid's where the axis is walled
        onW = G.wallW && x == 0;
        onE = G.wallE && x == G.nx - 1;
        onS = G.wallS && y == 0;
        onN = G.wallN && y == G.ny - 1;
        wall = onW || onE || onS || onN;
        c = ly * W + lx;
        cf = c + (onW ? 1 : 0) - (onE ? 1 : 0) + (onS ? W : 0) - (onN ? W : 0);
    };
    // Whether a work-item keeps its node for all K steps instead of being dealt one anew.  A region
    // 32 nodes wide loses little by it (a wavefront holds two whole rows, so that rows fall out as they
    // become inactive; the second step keeps two half-idle ones: 22 wavefront-steps against 21 for
    // 28 x 12, 46 against 44 for 28 x 28), and the place, the walls and the LDS addresses are worked
    // out once: three steps per launch, us per step, dealt / kept: 28 x 12 FP32 1021 x 509 6.77 / 6.33
    // and with a per-node medium 7.08 / 6.84, FP64 11.0 / 10.9; 28 x 28 FP32 uniform 1536^2 21.4 / 20.5,
    // 3500^2 112.7 / 111.4.  Not with 28 x 28 and a per-node medium (3500^2 125 / 129: the kept
    // values are spilled there), and not for two steps, where only one step would be spared
    // (FP32 storage with FP64 arithmetic, 1024^2, 15.7 / 18.0).
    constexpr bool kKept = K > 2 && (W & (W - 1)) == 0 && !(PN && NT > 512);
    if constexpr (kKept) {
        lx = i & (W - 1);
        ly = i / W;
        place();
    }
    auto deal = [&](int s) {
        const int ax = openW ? s - 1 : 0, ay = openS ? s - 1 : 0;
        const int aw = (rx1 - rx0) - (openE ? s - 1 : 0) - ax;
        const int ah = (ry1 - ry0) - (openN ? s - 1 : 0) - ay;
        if constexpr (kKept) {
            mine = unsigned(lx - ax) < unsigned(aw) && unsigned(ly - ay) < unsigned(ah);
        } else {
            // row of work-item i: (i + 1/2) / aw is at least 1/(2 aw) from a whole number, far
            // more than the rounding of the reciprocal and the product for i < 1024
            const int row = int((float(i) + 0.5f) * __builtin_amdgcn_rcpf(float(aw)));
            mine = row < ah;
            lx = ax + (i - row * aw);
            ly = ay + row;
            place();
        }
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

    // this work-item's node, if it is the tile's, to the state of step s in global memory;
    // unwrapped: the tile lies inside the grid
    auto store = [&](int s, const R f[9], const R g[5]) {
        const int x = rx0 + lx, y = ry0 + ly;
        if (x < x0 || x >= x1 || y < y0 || y >= y1) return;
        S* const to = dst + (EVERY ? size_t(s - 1) * stride : 0);
        const unsigned o = (unsigned(y) * unsigned(G.pitch) + unsigned(x)) * unsigned(sizeof(S));
#pragma unroll
        for (int p = 0; p < 9; ++p) at(plane(to, p, G.plane), o) = S(f[p]);
#pragma unroll
        for (int p = 0; p < 5; ++p) at(plane(to, 9 + p, G.plane), o) = S(g[p]);
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
        if constexpr (EVERY) store(1, f, g);
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
            if constexpr (EVERY) store(s, f, g);
        }
        __syncthreads();
    }

    // step K, from LDS to the other buffer
    deal(K);
    const int x = rx0 + lx, y = ry0 + ly;
    if (mine && x >= x0 && x < x1 && y >= y0 && y < y1) {
        R f[9], g[5];
        take(f, g);
        store(K, f, g);
    }
}

}  // namespace lbm
