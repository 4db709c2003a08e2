// lbm_kernels.hip -- single-cavity kernels: the time step (one step per launch, and the in-place
// AA-layout forms), the observables pass with the wall Nusselt sums
// (also over a batch), the stream function and state initialisation.
#include "lbm_device.hpp"
#include "lbm_internal.hpp"

namespace lbm {

// One time step for every node: pull (Eqs. (18), (35)) -> wall reconstruction -> macroscopic
// recovery (Eqs. (36), (22), (21), (23), (4)) -> collision (Eqs. (17), (34)) -> store.
// One work-item per node; a work-group covers kTileX consecutive nodes of one row.  S is the
// storage type, R the arithmetic type.
template <typename S, typename R, bool PN>
__global__ __launch_bounds__(kTileX) void step_kernel(const S* __restrict__ src,
                                                      S* __restrict__ dst,
                                                      const S* __restrict__ med, Geo G,
                                                      Phys<R> P, int tiles_x, int by_xcd) {
    // Work-groups in launch order walk the lattice row by row, or each XCD takes one contiguous
    // band of rows: the latter for a state that the XCDs' 8 x 4 MiB of L2 hold (us per step: FP32
    // 256^2 4.5 to 3.6, 512^2 7.9 to 7.0, FP64 256^2 5.7 to 4.5), not for a larger one, where it
    // concentrates each XCD's stream on one address range (FP64 1536^2 100 to 104, FP32 4096^2 7 %
    // slower).
    const int t = by_xcd ? tile_index() : int(blockIdx.x);
    const int y = t / tiles_x;
    const int x = (t - y * tiles_x) * kTileX + threadIdx.x;
    if (x >= G.nx) return;
    R f[9], g[5];
    Mac<R> m;
    Med<R> md;
    node_state<R, PN, S>(src, med, G, P, x, y, f, g, m, md);
    collide<R>(f, g, m, md, P);
    const unsigned o = (unsigned(y) * unsigned(G.pitch) + unsigned(x)) * unsigned(sizeof(S));
#pragma unroll
    for (int i = 0; i < 9; ++i)
        __builtin_nontemporal_store(S(f[i]), &at(plane(dst, i, G.plane), o));
#pragma unroll
    for (int i = 0; i < 5; ++i)
        __builtin_nontemporal_store(S(g[i]), &at(plane(dst, 9 + i, G.plane), o));
}

// One AA-pattern time step in place (layout L = kAAOpp or kAAOwn read, the other written).
// The per-node arithmetic is step_kernel's.  A wall node is stepped by the thread of its inward
// neighbour, which already holds the populations the reconstruction needs: a wall thread reading
// them itself could see the neighbour's new values.  The thread of node x writes only slots that
// it alone read (its own and those of the wall nodes it steps), so the step is race-free.
template <typename S, typename R, bool PN, int L>
__global__ __launch_bounds__(kTileX) void aa_step_kernel(S* __restrict__ buf,
                                                         const S* __restrict__ med, Geo G,
                                                         Phys<R> P, int tiles_x) {
    const int t = blockIdx.x;
    const int y = t / tiles_x;
    const int x = (t - y * tiles_x) * kTileX + threadIdx.x;
    if (x >= G.nx) return;
    if ((G.wallW && x == 0) || (G.wallE && x == G.nx - 1) || (G.wallS && y == 0) ||
        (G.wallN && y == G.ny - 1))
        return;
    R f[9], g[5];
    pull<R, S, L>(buf, G, x, y, f, g);
    const Med<R> md = load_medium<R, PN, S>(med, y * G.pitch + x, G.plane, P);
    const Mac<R> m = fluid_macros<R>(f, g, md, P);
    step_wall_neighbours<R, PN, S>(med, G, P, x, y, f, g, m, md,
                                   [&](int xb, int yb, const R* fb, const R* gb) {
                                       aa_store<S, R, L>(buf, G, xb, yb, fb, gb);
                                   });
    collide<R>(f, g, m, md, P);
    aa_store<S, R, L>(buf, G, x, y, f, g);
}

// The same step for states that fit the Infinity Cache (see aa_in_tiles): tiles of kAATX x kAATY
// nodes in which a wall node, which pulls at its inward neighbour, shares the work-group of that
// neighbour, which overwrites those slots; the work-group reads everything before it writes
// anything.  A wall node costs its own wavefront a branch, where aa_step_kernel's wavefronts along
// the walls step up to four nodes in turn (64^2 FP32 6.3 us per step against 3.6), and each XCD
// takes a contiguous run of tiles, so that rows shared by neighbouring tiles stay in its L2
// (1024^2 FP32 22.1 us per step, here 20.9 in launch order and 19.2 so).
constexpr int kAATX = 128, kAATY = 2;
template <typename S, typename R, bool PN, int L>
__global__ __launch_bounds__(kAATX* kAATY) void aa_tile_step_kernel(S* buf,
                                                                    const S* __restrict__ med,
                                                                    Geo G, Phys<R> P,
                                                                    WallTiles T) {
    const int t = tile_index(), ty = t / T.nx_tiles, tx = t - ty * T.nx_tiles;
    int x0, x1, y0, y1;
    wall_span(tx, T.nx_tiles, kAATX, T.last_x0, G.nx, x0, x1);
    wall_span(ty, T.ny_tiles, kAATY, T.last_y0, G.ny, y0, y1);
    const int x = x0 + int(threadIdx.x) % kAATX, y = y0 + int(threadIdx.x) / kAATX;
    const bool active = x < x1 && y < y1;
    R f[9], g[5];
    if (active) {
        Mac<R> m;
        Med<R> md;
        node_state<R, PN, S, L>(buf, med, G, P, x, y, f, g, m, md);
        collide<R>(f, g, m, md, P);
    }
    __syncthreads();   // every slot read before any is written
    if (active) aa_store<S, R, L>(buf, G, x, y, f, g);
}

// Maximum and minimum that propagate a NaN (fmax and fmin would drop it), so that a
// non-finite value always reaches the result of a reduction.
__device__ __forceinline__ double obs_max(double a, double b) {
    return (a >= b || a != a) ? a : b;
}
__device__ __forceinline__ double obs_min(double a, double b) {
    return (a <= b || a != a) ? a : b;
}

// Wave-level reductions over the 64 lanes of a wavefront.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = obs_max(v, __shfl_down(v, off, 64));
    return v;
}
__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = obs_min(v, __shfl_down(v, off, 64));
    return v;
}

// The partial results of the observables (observe_nodes): over a wavefront, and two sets into one.
__device__ __forceinline__ void obs_wave_reduce(double v[kObsParts]) {
    v[0] = wave_max(v[0]);
    v[1] = wave_sum(v[1]);
    v[2] = wave_max(v[2]);
    v[3] = wave_min(v[3]);
    v[4] = wave_max(v[4]);
    v[5] = wave_max(v[5]);
}
__device__ __forceinline__ void obs_merge(double v[kObsParts], const double q[kObsParts]) {
    v[0] = obs_max(v[0], q[0]);
    v[1] += q[1];
    v[2] = obs_max(v[2], q[2]);
    v[3] = obs_min(v[3], q[3]);
    v[4] = obs_max(v[4], q[4]);
    v[5] = obs_max(v[5], q[5]);
}

// Temperature deviation theta = T - T0 at (x, y) after streaming and wall reconstruction.
template <typename S, typename R, int L>
__device__ __forceinline__ double node_theta(const S* __restrict__ src, const Geo& G,
                                             const Phys<R>& P, int x, int y) {
    const bool onW = G.wallW && x == 0;
    const bool onE = G.wallE && x == G.nx - 1;
    const bool onS = G.wallS && y == 0;
    const bool onN = G.wallN && y == G.ny - 1;
    const int xf = x + (onW ? 1 : 0) - (onE ? 1 : 0);
    const int yf = y + (onS ? 1 : 0) - (onN ? 1 : 0);
    R f[9], g[5];
    pull<R, S, L>(src, G, xf, yf, f, g);
    const R th = ((g[0] + g[1]) + (g[2] + g[3]) + g[4]) + P.hQs;
    if (!(onW || onE || onS || onN)) return double(th);
    return double(wall_theta<R>(onW, onE, onS, onN, th, P));
}

// Eq. (38): Nu(y) = -L dT/dx / dT at the west (hot) and east (cold) walls with the fourth-order
// one-sided five-point derivative, averaged by the trapezoid rule over the ny wall nodes.  The
// rows are split into nu_groups(ny) runs of nu_rows(ny), one work-group each, which writes the
// west and east sums of its run before the factor -L / (dT (ny - 1)) to nu[2 run], nu[2 run + 1].
// The split and the order of the sums depend on ny alone, so that a cavity of a batch gives the
// bits of its own run.  (One work-group for all rows: 145 us at 64^2 and 279 us at 4096^2, whose
// 200,000 loads, each from a line of its own, one compute unit cannot keep in flight.)
__host__ __device__ inline int nu_rows(int ny) { return max(64, (ny + kNuWG - 1) / kNuWG); }
__host__ __device__ inline int nu_groups(int ny) { return (ny + nu_rows(ny) - 1) / nu_rows(ny); }

template <typename S, typename R, int L>
__device__ __forceinline__ void nusselt_rows(const S* __restrict__ src, const Geo& G,
                                             const Phys<R>& P, int run,
                                             double* __restrict__ nu) {
    double h = 0.0, c = 0.0;
    const int rows = nu_rows(G.ny), y0 = run * rows, y1 = min(y0 + rows, G.ny);
    if (G.nx >= 5 && threadIdx.x < 256) {
        for (int y = y0 + threadIdx.x; y < y1; y += 256) {
            double Th[5], Tc[5];
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                Th[k] = node_theta<S, R, L>(src, G, P, k, y);
                Tc[k] = node_theta<S, R, L>(src, G, P, G.nx - 1 - k, y);
            }
            const double dh = (-25.0 * Th[0] + 48.0 * Th[1] - 36.0 * Th[2] + 16.0 * Th[3] -
                               3.0 * Th[4]) / 12.0;
            const double dc = (25.0 * Tc[0] - 48.0 * Tc[1] + 36.0 * Tc[2] - 16.0 * Tc[3] +
                               3.0 * Tc[4]) / 12.0;
            const double w = (y == 0 || y == G.ny - 1) ? 0.5 : 1.0;
            h += w * dh;
            c += w * dc;
        }
    }
    __shared__ double red[2][kObsThreads / 64];
    h = wave_sum(h);
    c = wave_sum(c);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        red[0][wv] = h;
        red[1][wv] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < 4; ++i) {   // 256 work-items summed rows
            h += red[0][i];
            c += red[1][i];
        }
        nu[2 * run] = h;
        nu[2 * run + 1] = c;
    }
}

// Macroscopic fields at the current time level and the partial results of the observables: the
// work of one work-group `wg` of `nwg` over the nodes of one cavity (grid-stride).  part (may be
// NULL: fields only) receives kObsParts results per work-group at part[kObsParts * wg + k]: k = 0
// max |u|, 1 the sum of stored f' (mass deviation), 2 a flag (1 when u, p, T or |v| of Eq. (22)
// is not finite), 3 min T, 4 max T, 5 max |phi p - rho0 cs^2|.
template <typename S, typename R, bool PN, int L>
__device__ __forceinline__ void observe_nodes(const S* __restrict__ src,
                                              const S* __restrict__ med, const Geo& G,
                                              const Phys<R>& P, S* __restrict__ ux_out,
                                              S* __restrict__ uy_out, S* __restrict__ p_out,
                                              S* __restrict__ T_out, double* __restrict__ part,
                                              int wg, int nwg) {
    const int n = G.nx * G.ny;
    double v[kObsParts] = {0.0, 0.0, 0.0, INFINITY, -INFINITY, 0.0};
    for (int k = wg * blockDim.x + threadIdx.x; k < n; k += nwg * blockDim.x) {
        const int y = k / G.nx, x = k - y * G.nx;
        R f[9], g[5];
        Mac<R> m;
        Med<R> md;
        node_state<R, PN, S, L>(src, med, G, P, x, y, f, g, m, md);
        // the pressure of Eq. (23) less its rest value rho0 cs^2 / phi: FP32 could not hold
        // the dynamic part, often below 1e-3 of p, on top of that background
        const R p = m.P * md.inv_phi;
        const R T = P.T0 + m.theta;
        if (ux_out) ux_out[k] = S(m.ux);
        if (uy_out) uy_out[k] = S(m.uy);
        if (p_out) p_out[k] = S(p);
        if (T_out) T_out[k] = S(T);
        if (!part) continue;
        const double sp = sqrt(double(m.ux) * double(m.ux) + double(m.uy) * double(m.uy));
        const double Td = double(T), Pd = fabs(double(m.P));
        v[0] = obs_max(v[0], sp);
        if (!isfinite(sp) || !isfinite(double(p)) || !isfinite(Td) || !isfinite(double(m.vv)))
            v[2] = 1.0;
        v[3] = obs_min(v[3], Td);
        v[4] = obs_max(v[4], Td);
        v[5] = obs_max(v[5], Pd);
        const int o = y * G.pitch + x;
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 9; ++i) s += double(src[i * G.plane + o]);
        v[1] += s;
    }
    if (!part) return;
    __shared__ double red[kObsParts][kObsThreads / 64];
    obs_wave_reduce(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < kObsParts; ++k) red[k][w] = v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < (int)(blockDim.x >> 6); ++i) {
            double q[kObsParts];
#pragma unroll
            for (int k = 0; k < kObsParts; ++k) q[k] = red[k][i];
            obs_merge(v, q);
        }
#pragma unroll
        for (int k = 0; k < kObsParts; ++k) part[kObsParts * wg + k] = v[k];
    }
}

// Work-groups 0 .. nwg - 1 take the nodes, those after them (with part) the walls' sums, which go
// to the last 2 * kNuWG of the `per` doubles of partial results.
template <typename S, typename R, bool PN, int L>
__global__ __launch_bounds__(kObsThreads) void observe_kernel(
    const S* __restrict__ src, const S* __restrict__ med, Geo G, Phys<R> P,
    S* __restrict__ ux_out, S* __restrict__ uy_out, S* __restrict__ p_out, S* __restrict__ T_out,
    double* __restrict__ part, int per, int nwg) {
    if (int(blockIdx.x) >= nwg)
        nusselt_rows<S, R, L>(src, G, P, blockIdx.x - nwg, part + per - 2 * kNuWG);
    else
        observe_nodes<S, R, PN, L>(src, med, G, P, ux_out, uy_out, p_out, T_out, part,
                                   blockIdx.x, nwg);
}

// The observables of every cavity of a batch in one launch: work-group (b, c) is share b of
// cavity c, as in observe_kernel.  (A launch pair per cavity, each of 64 work-groups, took 64
// times 43 us on the 64-cavity workload.)
template <typename S, typename R>
__global__ __launch_bounds__(kObsThreads) void batch_observe_kernel(
    const S* __restrict__ src, const BatchCavity* __restrict__ cav,
    const Phys<R>* __restrict__ phys, double* __restrict__ part, int per, int nwg) {
    const int c = blockIdx.y;
    const BatchCavity C = cav[c];
    const Phys<R> P = phys[c];
    double* const mine = part + size_t(c) * per;
    const int run = int(blockIdx.x) - nwg;
    if (run >= 0) {
        if (run < nu_groups(C.G.ny))
            nusselt_rows<S, R, kPull>(src + C.off, C.G, P, run, mine + per - 2 * kNuWG);
        return;
    }
    observe_nodes<S, R, false, kPull>(src + C.off, (const S*)nullptr, C.G, P, (S*)nullptr,
                                      (S*)nullptr, (S*)nullptr, (S*)nullptr, mine, blockIdx.x,
                                      nwg);
}

// The results of one cavity's observables by one work-group of 256: out[0] and out[1] the west and
// east walls' Nusselt sums, then out[2 + k] the reduction of partial result k over the nparts
// work-groups of observe_nodes.  A work-item merges every 256th set of partial results, then the
// wavefronts reduce (one work-item merging 512 sets in turn took 140 us of every look at the
// observables, whatever the grid).
__device__ __forceinline__ void observe_results(const double* __restrict__ part,
                                                const double* __restrict__ nu, int nparts,
                                                int nnu, double* __restrict__ out) {
    double v[kObsParts] = {0.0, 0.0, 0.0, INFINITY, -INFINITY, 0.0};
    for (int i = threadIdx.x; i < nparts; i += 256) {
        double q[kObsParts];
#pragma unroll
        for (int k = 0; k < kObsParts; ++k) q[k] = part[kObsParts * i + k];
        obs_merge(v, q);
    }
    // the last wavefront's first lanes hold the walls' sums
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double h = w == 3 && lane < nnu ? nu[2 * lane] : 0.0;
    double c = w == 3 && lane < nnu ? nu[2 * lane + 1] : 0.0;
    __shared__ double red[kObsParts][4];
    obs_wave_reduce(v);
    h = wave_sum(h);
    c = wave_sum(c);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < kObsParts; ++k) red[k][w] = v[k];
        if (w == 3) {
            out[0] = h;
            out[1] = c;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < 4; ++i) {
            double q[kObsParts];
#pragma unroll
            for (int k = 0; k < kObsParts; ++k) q[k] = red[k][i];
            obs_merge(v, q);
        }
#pragma unroll
        for (int k = 0; k < kObsParts; ++k) out[2 + k] = v[k];
    }
}

// Results of cavity blockIdx.x (0 for a single one) at out[kObsOut * cavity]; per: doubles of
// partial results per cavity, the last 2 * kNuWG of them the walls' sums; nu_groups(ny) of them
// are in use.
__global__ __launch_bounds__(256) void observe_results_kernel(const double* __restrict__ part,
                                                              int per, int nparts, int ny,
                                                              double* __restrict__ out) {
    observe_results(part, part + per - 2 * kNuWG, nparts, nu_groups(ny), out);
}
__global__ __launch_bounds__(256) void batch_observe_results_kernel(
    const double* __restrict__ part, const BatchCavity* __restrict__ cav, int per, int nparts,
    double* __restrict__ out) {
    const double* const mine = part + size_t(blockIdx.x) * per;
    observe_results(mine, mine + per - 2 * kNuWG, nparts, nu_groups(cav[blockIdx.x].G.ny),
                    out + kObsOut * blockIdx.x);
}

// Stream function: u_x (Eq. (21)) integrated along y with the trapezoid rule in FP64,
// psi(x, 0) = 0.  A work-group owns COLS columns and takes kPsiPer * SLOTS rows at a time: a
// work-item sums kPsiPer consecutive rows of one column, the sums of the SLOTS work-items of
// a column are scanned in LDS, and the column's total carries over to the next rows.  (One
// work-item per column, row after row, is a chain of ny dependent gathers: 97 us at 301 x 199
// against 10.5 us this way.)
constexpr int kPsiPer = 4;

template <typename S, typename R, bool PN, int L, int COLS, int SLOTS>
__global__ __launch_bounds__(COLS* SLOTS) void stream_function_kernel(
    const S* __restrict__ src, const S* __restrict__ med, Geo G, Phys<R> P,
    S* __restrict__ psi) {
    __shared__ double edge[SLOTS][COLS];   // u of each slot's last row
    __shared__ double sums[2][SLOTS][COLS];
    const int col = threadIdx.x % COLS, slot = threadIdx.x / COLS;
    const int x = blockIdx.x * COLS + col;
    double carry = 0.0, before = 0.0;   // psi and u at the last row of the rows done so far
    for (int base = 0; base < G.ny; base += kPsiPer * SLOTS) {
        const int y0 = base + slot * kPsiPer;
        double u[kPsiPer];
#pragma unroll
        for (int j = 0; j < kPsiPer; ++j) {
            u[j] = 0.0;
            if (x < G.nx && y0 + j < G.ny) {
                R f[9], g[5];
                Mac<R> m;
                Med<R> md;
                node_state<R, PN, S, L>(src, med, G, P, x, y0 + j, f, g, m, md);
                u[j] = double(m.ux);
            }
        }
        edge[slot][col] = u[kPsiPer - 1];
        __syncthreads();
        const double prev = slot > 0 ? edge[slot - 1][col] : before;
        before = edge[SLOTS - 1][col];
        // increments up to each of this work-item's rows (none into row 0)
        double inc[kPsiPer];
        double acc = y0 > 0 ? 0.5 * (prev + u[0]) : 0.0;
        inc[0] = acc;
#pragma unroll
        for (int j = 1; j < kPsiPer; ++j) {
            acc += 0.5 * (u[j - 1] + u[j]);
            inc[j] = acc;
        }
        int cur = 0;
        sums[0][slot][col] = acc;
        __syncthreads();
        for (int d = 1; d < SLOTS; d <<= 1) {
            double t = sums[cur][slot][col];
            if (slot >= d) t += sums[cur][slot - d][col];
            sums[1 - cur][slot][col] = t;
            cur = 1 - cur;
            __syncthreads();
        }
        const double start = carry + (slot > 0 ? sums[cur][slot - 1][col] : 0.0);
        carry += sums[cur][SLOTS - 1][col];
#pragma unroll
        for (int j = 0; j < kPsiPer; ++j)
            if (x < G.nx && y0 + j < G.ny) psi[(y0 + j) * G.nx + x] = S(start + inc[j]);
        __syncthreads();   // edge and sums are written again for the next rows
    }
}

// Rest state (u = 0, phi p = rho0 cs^2, T = T_init) as deviations: f' = 0, g' = wt (T_init - T0).
template <typename R>
__global__ void rest_kernel(R* __restrict__ dst, Geo G, R g0, R g1) {
    const int n = G.plane;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
#pragma unroll
        for (int i = 0; i < 9; ++i) dst[i * n + k] = R(0);
        dst[9 * n + k] = g0;
#pragma unroll
        for (int i = 1; i < 5; ++i) dst[(9 + i) * n + k] = g1;
    }
}

// Pitched copy of a dense [ny][nx] field into a [ny][pitch] plane; a NULL source fills v.
template <typename R>
__global__ void pitch_copy_kernel(R* __restrict__ dst, const R* __restrict__ src, Geo G, R v) {
    const int n = G.nx * G.ny;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
        const int y = k / G.nx, x = k - y * G.nx;
        dst[y * G.pitch + x] = src ? src[k] : v;
    }
}

// ---- launchers --------------------------------------------------------------------------------

// Whether the AA step runs in tiles: for a state that fits the 256 MiB Infinity Cache, where the
// XCDs' L2 hits matter more than the order in which memory is streamed.  us per step, rows in
// launch order / tiles by XCD: FP32 64^2 6.3 / 3.6, 512^2 8.9 / 5.8, 1024^2 22.1 / 19.2, 2048^2
// (235 MB) 74.8 / 69.3, 2500^2 127 / 136, 4096^2 353 / 366; FP64 128^2 6.8 / 4.9, 1536^2 (264 MB)
// 83.2 / 78.2, 2000 x 1500 118 / 125, 4096^2 706 / 720.
static size_t state_bytes(const Geo& G, size_t elem_bytes) {
    return size_t(kPlanes) * size_t(G.plane) * elem_bytes;
}
static bool aa_in_tiles(const Geo& G, size_t elem_bytes) {
    return state_bytes(G, elem_bytes) <= size_t(256) << 20;
}

int one_step_groups(const Geo& G, size_t elem_bytes, bool aa) {
    if (aa && aa_in_tiles(G, elem_bytes)) {
        const WallTiles T = wall_tiles(G, kAATX, kAATY);
        return T.nx_tiles * T.ny_tiles;
    }
    return (G.nx + kTileX - 1) / kTileX * G.ny;
}

template <typename S, typename R>
hipError_t launch_step(const void* src, void* dst, const void* med, const Geo& G,
                       const Phys<R>& P, hipStream_t s) {
    const int tiles_x = (G.nx + kTileX - 1) / kTileX;
    const int nwg = one_step_groups(G, sizeof(S), false);
    const int by_xcd = state_bytes(G, sizeof(S)) <= size_t(32) << 20 ? 1 : 0;
    if (med)
        step_kernel<S, R, true><<<nwg, kTileX, 0, s>>>((const S*)src, (S*)dst, (const S*)med, G,
                                                       P, tiles_x, by_xcd);
    else
        step_kernel<S, R, false><<<nwg, kTileX, 0, s>>>((const S*)src, (S*)dst, nullptr, G, P,
                                                        tiles_x, by_xcd);
    return hipGetLastError();
}

template <typename S, typename R, int L>
static hipError_t aa_launch(S* b, const S* m, const Geo& G, const Phys<R>& P, hipStream_t s) {
    const int nwg = one_step_groups(G, sizeof(S), true);
    if (aa_in_tiles(G, sizeof(S))) {
        const WallTiles T = wall_tiles(G, kAATX, kAATY);
        if (m)
            aa_tile_step_kernel<S, R, true, L><<<nwg, kAATX * kAATY, 0, s>>>(b, m, G, P, T);
        else
            aa_tile_step_kernel<S, R, false, L><<<nwg, kAATX * kAATY, 0, s>>>(b, m, G, P, T);
    } else {
        const int tiles_x = (G.nx + kTileX - 1) / kTileX;
        if (m)
            aa_step_kernel<S, R, true, L><<<nwg, kTileX, 0, s>>>(b, m, G, P, tiles_x);
        else
            aa_step_kernel<S, R, false, L><<<nwg, kTileX, 0, s>>>(b, m, G, P, tiles_x);
    }
    return hipGetLastError();
}

// parity 0: the state is in the kAAOpp form (even step count); 1: kAAOwn (odd)
template <typename S, typename R>
hipError_t launch_aa_step(void* buf, const void* med, const Geo& G, const Phys<R>& P,
                          int parity, hipStream_t s) {
    return parity == 0 ? aa_launch<S, R, kAAOpp>((S*)buf, (const S*)med, G, P, s)
                       : aa_launch<S, R, kAAOwn>((S*)buf, (const S*)med, G, P, s);
}

// Work-groups and their size for the observables of n nodes: one node per work-item of 256 while
// `most` work-groups suffice, then work-groups of kObsThreads.
static void observe_shape(long long n, int most, int* nwg, int* threads) {
    *threads = n <= 256LL * most ? 256 : kObsThreads;
    *nwg = int(min((n + *threads - 1) / *threads, (long long)most));
}

template <typename S, typename R, int L>
static hipError_t observe_l(const void* src, const void* med, const Geo& G, const Phys<R>& P,
                            void* ux, void* uy, void* p, void* T, double* part, double* out,
                            hipStream_t s) {
    constexpr int per = kObsParts * kObserveWG + 2 * kNuWG;
    int nwg = 0, threads = 0;
    observe_shape((long long)G.nx * G.ny, kObserveWG, &nwg, &threads);
    const int all = nwg + (part ? nu_groups(G.ny) : 0);
    if (med)
        observe_kernel<S, R, true, L><<<all, threads, 0, s>>>(
            (const S*)src, (const S*)med, G, P, (S*)ux, (S*)uy, (S*)p, (S*)T, part, per, nwg);
    else
        observe_kernel<S, R, false, L><<<all, threads, 0, s>>>(
            (const S*)src, nullptr, G, P, (S*)ux, (S*)uy, (S*)p, (S*)T, part, per, nwg);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !part) return e;
    observe_results_kernel<<<1, 256, 0, s>>>(part, per, nwg, G.ny, out);
    return hipGetLastError();
}

// layout: kPull, kAAOpp or kAAOwn, the form the state is in
template <typename S, typename R>
hipError_t launch_observe(const void* src, const void* med, const Geo& G, const Phys<R>& P,
                          int layout, void* ux, void* uy, void* p, void* T, double* part,
                          double* out, hipStream_t s) {
    switch (layout) {
        case kPull:
            return observe_l<S, R, kPull>(src, med, G, P, ux, uy, p, T, part, out, s);
        case kAAOpp:
            return observe_l<S, R, kAAOpp>(src, med, G, P, ux, uy, p, T, part, out, s);
        case kAAOwn:
            return observe_l<S, R, kAAOwn>(src, med, G, P, ux, uy, p, T, part, out, s);
        default: return hipErrorInvalidValue;
    }
}

// Cavities per launch of the batch's observables: the cavity is the grid's y index, of which a device
// takes 65,536 at most, while a batch holds up to about 130,000 cavities of the smallest size.
constexpr int kBatchObsCavities = 32768;

template <typename S, typename R>
hipError_t launch_batch_observe(const void* src, const BatchTable<R>& T, long long largest,
                                double* part, double* out, hipStream_t s) {
    constexpr int per = kObsParts * kBatchObsWG + 2 * kNuWG;
    int nwg = 0, threads = 0;
    observe_shape(largest, kBatchObsWG, &nwg, &threads);
    for (int c = 0; c < T.ncav; c += kBatchObsCavities) {
        const int n = min(T.ncav - c, kBatchObsCavities);
        double* const mine = part + size_t(c) * per;
        batch_observe_kernel<S, R><<<dim3(nwg + kNuWG, n), threads, 0, s>>>(
            (const S*)src, T.cav + c, T.phys + c, mine, per, nwg);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        batch_observe_results_kernel<<<n, 256, 0, s>>>(mine, T.cav + c, per, nwg,
                                                       out + size_t(kObsOut) * c);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename S, typename R, int L>
static hipError_t stream_function_l(const void* src, const void* med, const Geo& G,
                                    const Phys<R>& P, void* psi, hipStream_t s) {
    auto go = [&](auto cols, auto slots) {
        constexpr int C = decltype(cols)::value, N = decltype(slots)::value;
        const int nb = (G.nx + C - 1) / C;
        if (med)
            stream_function_kernel<S, R, true, L, C, N><<<nb, C * N, 0, s>>>(
                (const S*)src, (const S*)med, G, P, (S*)psi);
        else
            stream_function_kernel<S, R, false, L, C, N><<<nb, C * N, 0, s>>>(
                (const S*)src, nullptr, G, P, (S*)psi);
    };
    // Work-groups of 16 columns and 256 rows at a time; on wide grids, whose columns alone fill the
    // GPU, of 64 columns and 32 rows, which read whole cache lines and leave no work-item without a
    // row where there are few (us, 16 x 256 / 64 x 32: FP32 8192 x 40 23.4 / 19.3, 20000 x 5 25.7 /
    // 15.7, 20000 x 200 104 / 65, 50000 x 400 443 / 304, 100000 x 5 88 / 20; FP64 20000 x 100 70 / 62,
    // 50000 x 400 577 / 582; where the columns do not suffice: FP64 8192 x 1000 233 / 270, FP32
    // 4096 x 1000 101 / 143).
    if (G.nx >= 32768 || (G.nx >= 8192 && G.ny <= 256))
        go(std::integral_constant<int, 64>{}, std::integral_constant<int, 8>{});
    else
        go(std::integral_constant<int, 16>{}, std::integral_constant<int, 64>{});
    return hipGetLastError();
}

template <typename S, typename R>
hipError_t launch_stream_function(const void* src, const void* med, const Geo& G,
                                  const Phys<R>& P, int layout, void* psi, hipStream_t s) {
    switch (layout) {
        case kPull: return stream_function_l<S, R, kPull>(src, med, G, P, psi, s);
        case kAAOpp: return stream_function_l<S, R, kAAOpp>(src, med, G, P, psi, s);
        case kAAOwn: return stream_function_l<S, R, kAAOwn>(src, med, G, P, psi, s);
        default: return hipErrorInvalidValue;
    }
}

template <typename R>
hipError_t launch_rest(void* dst, const Geo& G, double g0, double g1, hipStream_t s) {
    rest_kernel<R><<<1024, 256, 0, s>>>((R*)dst, G, R(g0), R(g1));
    return hipGetLastError();
}

template <typename R>
hipError_t launch_pitch_copy(void* dst, const void* src, const Geo& G, double v, hipStream_t s) {
    pitch_copy_kernel<R><<<1024, 256, 0, s>>>((R*)dst, (const R*)src, G, R(v));
    return hipGetLastError();
}

#define LBM_INSTANCES(S, R)                                                                      \
    template hipError_t launch_step<S, R>(const void*, void*, const void*, const Geo&,           \
                                          const Phys<R>&, hipStream_t);                          \
    template hipError_t launch_aa_step<S, R>(void*, const void*, const Geo&, const Phys<R>&,     \
                                             int, hipStream_t);                                  \
    template hipError_t launch_observe<S, R>(const void*, const void*, const Geo&,               \
                                             const Phys<R>&, int, void*, void*, void*, void*,    \
                                             double*, double*, hipStream_t);                     \
    template hipError_t launch_batch_observe<S, R>(const void*, const BatchTable<R>&, long long, \
                                                   double*, double*, hipStream_t);               \
    template hipError_t launch_stream_function<S, R>(const void*, const void*, const Geo&,       \
                                                     const Phys<R>&, int, void*, hipStream_t);
LBM_INSTANCES(float, float)
LBM_INSTANCES(double, double)
LBM_INSTANCES(float, double)
#undef LBM_INSTANCES
template hipError_t launch_rest<float>(void*, const Geo&, double, double, hipStream_t);
template hipError_t launch_rest<double>(void*, const Geo&, double, double, hipStream_t);
template hipError_t launch_pitch_copy<float>(void*, const void*, const Geo&, double, hipStream_t);
template hipError_t launch_pitch_copy<double>(void*, const void*, const Geo&, double,
                                              hipStream_t);

}  // namespace lbm
