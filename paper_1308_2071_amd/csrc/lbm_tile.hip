// lbm_tile.hip -- several time steps per launch of one cavity: the forms (tile, steps, work-items)
// and which one a grid takes.
#include "lbm_tile.hpp"

namespace lbm {

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

// Wavefronts per SIMD of the form that keeps every state.  Its extra addresses are spilled at the four
// of 16 x 16 tiles with FP64 arithmetic: 76 bytes per lane with a uniform medium, which takes three
// instead (256^2 FP64, us per 100 steps of lbm_grad: 1373 / 1243), 28 with a per-node one, which does
// not (330^2 1763 / 1849).
template <typename F, typename R, bool PN>
constexpr int trace_waves() {
    return !PN && sizeof(R) == 8 && F::K == kTileSteps ? 3 : F::template waves<R>();
}

// F::K steps that keep every state, step s at dst + (s - 1) * stride.
template <typename S, typename R, bool PN, typename F>
__global__ __launch_bounds__(F::NT, (trace_waves<F, R, PN>())) void tile_trace_kernel(
    const S* __restrict__ src, S* __restrict__ dst, size_t stride, const S* __restrict__ med,
    Geo G, Phys<R> P, int tiles_x) {
    const int t = tile_index(), ty = t / tiles_x;
    tile_steps_body<S, R, PN, F::TX, F::TY, F::K, F::NT, true>(src, dst, med, G, P,
                                                               t - ty * tiles_x, ty, stride);
}

// Steps per launch of the time loop by default.  The halo's redundant work grows with the steps
// and shrinks with the tile, the launches and the bytes per step fall with the steps.  Measured,
// us per step on porous cavities, uniform / per-node medium:
//                          8 x 8, 8    16 x 16, 4  28 x 12, 3  28 x 28, 3  30 x 14, 2
//   FP32          128^2    1.46 1.51   1.95 1.94   1.96 2.01   3.27 3.37   2.49 2.58
//                 192^2    2.11 2.21   1.97 1.97   1.96 2.02   3.35 3.38   2.57 2.64
//                 512^2    8.22 8.50   4.11 4.26   4.24 4.48   5.27 5.43   4.56 4.69
//                 1024^2   29.5 30.7   11.8 12.4   10.6 12.2   12.1 12.5   12.2 12.7
//                 2048^2   114  119    47.0 50.1   45.2 49.2   40.0 45.3   54.6 58.4
//                 4096^2   450  472    188  201    182  198    150  167    224  242
//   FP64          128^2    1.85 1.93   2.67 2.80   2.91 3.18               3.42 3.70
//                 256^2    4.58 4.86   2.85 2.98   3.1  3.4                3.73 4.08
//                 517 x 389 11.8 12.5  6.43 6.86   5.95 6.36               6.20 6.66
//                 1024^2   53.9 57.6   21.8 23.4   18.5 21.8               21.3 24.3
//                 4096^2   829  921    325  373    292  368                408  444
//   FP32 storage, 128^2    1.78 2.00   2.53 2.71   2.94 3.11               3.25 3.53
//   FP64          256^2    4.54 4.96   2.54 2.74   2.97 3.18               3.31 3.62
//   arithmetic    517 x 389 12.2 12.9  6.10 6.48   5.80 6.16               4.99 5.48
//                 1024^2   57.8 60.5   21.6 22.9   19.0 20.2               16.0 19.4
//                 4096^2   885  953    302  328    265  297                244  311
// (28 x 28 below 2048^2 and 28 x 12 from there in FP32: measured with the nodes dealt anew in each
// step, which takes 3 to 6 % longer.)  One step per launch takes 2 to 3 times as long on the
// smallest of these and 1.1 to 1.9 times on the largest.  FP32 goes from four steps to three between
// 512^2 and 600 x 520 (uniform 4.65 / 4.42, per-node 4.90 / 4.77; 760 x 520 5.72 / 5.33, 5.96 /
// 5.65; 800^2 7.70 / 7.36, 8.5 / 8.05).  Per-node media from 1024^2 to 1536^2 in
// FP32, and from 4096^2 in FP64, keep the two steps per launch that lbm_step_shape has always reported
// for these grids, though three are faster there (us per step, two / three: FP32 1024^2 13.0 / 11.3,
// 1280^2 18.7 / 16.8, 1536^2 30.2 / 24.7; steps_per_launch = 3 asks for them in FP32).
constexpr long long kTinyTileMaxNodes = 128LL * 128;

template <typename S, typename R>
int default_steps(const Geo& G, bool per_node_medium) {
    const long long n = (long long)G.nx * G.ny;
    if (n <= kTinyTileMaxNodes) return kTinyTileSteps;
    if (sizeof(R) == 4) {
        if (n <= 300000) return kTileSteps;
        return per_node_medium && n >= 1024LL * 1024 && n <= 1536LL * 1536 ? 2 : 3;
    }
    if (sizeof(S) == 4) return n <= 110000 ? kTileSteps : 2;
    if (n <= 150000) return kTileSteps;
    return per_node_medium && n >= 4096LL * 4096 ? 2 : 3;
}

// Steps per launch of the adjoint's recompute, which runs beside the backward sweep: the default,
// except with FP64 arithmetic on small grids.  On FP32 storage up to 256^2 one backward step per
// launch sets the pace and a tile's work-group holds up the sweep's longer than a single step's does
// (lbm_grad, us per step, one / several recomputed per launch: 128^2 8.3 / 8.8, 256^2 9.1 / 9.9; FP64,
// whose sweep takes tiles there, 64^2 9.2 / 8.6, 256^2 13.1 / 10.8).  Where the default is four steps,
// segments of up to 40 are recomputed in pairs, on smaller tiles with twice the wavefronts: the
// sweep waits for a short segment, and four in a launch of two wavefronts per SIMD take longer than
// two launches (us per 100 steps, pairs / fours / one per launch before there were tiles, segments of
// 10 and of 100: FP64 uniform 256^2 1104 / 1153 / 1191 and 1318 / 1243 / 1639, FP64 per-node 380^2
// 1908 / 2101 / 2028 and 2202 / 2290 / 2641, FP32 storage per-node 330^2 1210 / 1335 / 1259 and 1575 /
// 1473 / 1721).
constexpr int kPairedSegment = 40;

template <typename S, typename R>
int recompute_steps(const Geo& G, bool per_node_medium, int segment) {
    if (sizeof(S) == 4 && sizeof(R) == 8 && (long long)G.nx * G.ny <= 256LL * 256) return 1;
    const int k = default_steps<S, R>(G, per_node_medium);
    return sizeof(R) == 8 && k == kTileSteps && segment <= kPairedSegment ? 2 : k;
}

// Where two or three steps per launch take their larger tile: from the size on where the launch
// has several rounds of work-groups, so that fewer, larger ones cost no balance (28 x 28 against
// 28 x 12, FP32: 1024^2 12.1 against 11.3 us per step, 1536^2 23.5 against 22.4 and with a
// per-node medium 26.0 against 27.3, 4096^2 163 against 182; in FP64 the larger region leaves a
// compute unit one work-group: 4096^2 358 against 302.  62 x 14 against 30 x 14, FP32: 1024^2
// 12.8 against 12.2, 4096^2 202 against 224).  The region of 62 x 14 takes 90 KB of LDS with FP64
// arithmetic on FP32 storage and 147 KB in FP64 (per-node medium), one work-group per compute unit:
// us per step against 30 x 14, FP32 storage uniform 1540^2 39.6 / 35.4, 4096^2 257 / 236, 8192^2 993 /
// 901; FP64 per-node 1540^2 71.4 / 69.5, 2048^2 115 / 113, but from there on, where 147 KB of state
// in flight count for more, 3000^2 235 / 242, 4096^2 418 / 436, 6100^2 928 / 977.
constexpr long long kLargeTileNodes = 1536LL * 1536, kLargeTileNodes64 = 2500LL * 2500;

template <typename S, typename R, typename F, typename Go>
auto tile_grid(const Geo& G, Go&& go) {
    const int tiles_x = (G.nx + F::TX - 1) / F::TX;
    return go(F{}, tiles_x, tiles_x * ((G.ny + F::TY - 1) / F::TY));
}

// Whether k steps per launch have a form: three do not with FP64 arithmetic on FP32 storage, where four
// are faster up to 110,000 nodes and two beyond.
template <typename S, typename R>
constexpr bool has_form(int k) {
    return k == 2 || (k == 3 && sizeof(S) == sizeof(R)) || k == kTileSteps || k == kTinyTileSteps;
}

// Calls go(form, tiles along x, work-groups) with the form that takes k steps on grid G.
template <typename S, typename R, typename Go>
auto with_form(const Geo& G, int k, Go&& go) {
    const long long n = (long long)G.nx * G.ny;
    if (k == kTinyTileSteps) return tile_grid<S, R, Tile8>(G, go);
    if (k == kTileSteps) return tile_grid<S, R, Tile4>(G, go);
    if constexpr (sizeof(S) == sizeof(R)) {
        if (k == 3) {
            if constexpr (sizeof(R) == 4) {
                if (n >= kLargeTileNodes) return tile_grid<S, R, Tile3Large>(G, go);
            }
            return tile_grid<S, R, Tile3>(G, go);
        }
        if (n >= (sizeof(R) == 4 ? kLargeTileNodes : kLargeTileNodes64))
            return tile_grid<S, R, Tile2Large>(G, go);
    }
    return tile_grid<S, R, Tile2>(G, go);
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
    if (!has_form<S, R>(k)) return hipErrorInvalidValue;
    return with_form<S, R>(G, k, [&](auto f, int tiles_x, int nwg) {
        using F = decltype(f);
        return med ? launch_form<S, R, true, F>(src, dst, med, G, P, tiles_x, nwg, s)
                   : launch_form<S, R, false, F>(src, dst, nullptr, G, P, tiles_x, nwg, s);
    });
}

template <typename S, typename R, bool PN, typename F>
static hipError_t launch_trace(const void* src, void* dst, size_t stride, const void* med,
                               const Geo& G, const Phys<R>& P, int tiles_x, int nwg,
                               hipStream_t s) {
    constexpr size_t lds = tile_lds_bytes<S, R, PN, F::TX, F::TY, F::K>();
    tile_trace_kernel<S, R, PN, F><<<nwg, F::NT, lds, s>>>((const S*)src, (S*)dst, stride,
                                                           (const S*)med, G, P, tiles_x);
    return hipGetLastError();
}

template <typename S, typename R>
hipError_t launch_tile_trace(const void* src, void* dst, size_t stride, const void* med,
                             const Geo& G, const Phys<R>& P, int k, hipStream_t s) {
    if (!has_form<S, R>(k)) return hipErrorInvalidValue;
    return with_form<S, R>(G, k, [&](auto f, int tiles_x, int nwg) {
        using F = decltype(f);
        // grids of eight steps recompute one per launch with FP64 arithmetic on FP32 storage
        if constexpr (F::K == kTinyTileSteps && sizeof(S) != sizeof(R))
            return hipErrorInvalidValue;
        else
            return med ? launch_trace<S, R, true, F>(src, dst, stride, med, G, P, tiles_x, nwg, s)
                       : launch_trace<S, R, false, F>(src, dst, stride, nullptr, G, P, tiles_x,
                                                      nwg, s);
    });
}

#define LBM_TILE_INST(S, R)                                                                    \
    template int default_steps<S, R>(const Geo&, bool);                                        \
    template int recompute_steps<S, R>(const Geo&, bool, int);                                 \
    template void tile_shape<S, R>(const Geo&, int, int*, int*);                               \
    template hipError_t launch_tile_step<S, R>(const void*, void*, const void*, const Geo&,    \
                                               const Phys<R>&, int, hipStream_t);              \
    template hipError_t launch_tile_trace<S, R>(const void*, void*, size_t, const void*,       \
                                                const Geo&, const Phys<R>&, int, hipStream_t);
LBM_TILE_INST(float, float)
LBM_TILE_INST(double, double)
LBM_TILE_INST(float, double)
#undef LBM_TILE_INST

}  // namespace lbm
