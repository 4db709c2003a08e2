// lbm_adjoint.hip -- discrete adjoint of the fused time step: the exact vector-Jacobian product
// of one step of the forward map (streaming, wall reconstruction, macroscopic recovery,
// collision; Eqs. (18), (35), (36), (22), (21), (23), (4), (17), (34) of arXiv:1308.2071), plus
// the accumulation of dJ/dphi and dJ/dK at every node, and the seed of J = Nu_hot (Eq. (38)).
//
// Race freedom without atomics: in the forward pull, node x reads slot (i, x - e_i) of the
// previous state, and the map x -> (i, x - e_i) is a bijection; a wall node reads nothing of its
// own slots but the slots of its inward neighbour x_f.  So the thread of node x writes the
// adjoint of exactly its own slots: its own collision's contribution plus the contributions of
// every wall node whose inward neighbour is x, which the wall nodes' threads hand over through
// LDS.  Wall threads write zeros to their own slots.
#include "lbm_device.hpp"
#include "lbm_internal.hpp"

namespace lbm {

// Adjoints of the macroscopic quantities a collision consumes.
template <typename R>
struct MacAdj {
    R theta, ux, uy, P, Fx, Fy, ip;
};

// Reverse of collide(): given the adjoints lf, lg of the post-collision populations, adds the
// adjoints of the post-streaming populations to af, ag and of the macroscopics to A.
template <typename R>
__device__ __forceinline__ void collide_vjp(const R f[9], const R g[5], const Mac<R>& m,
                                            const Med<R>& md, const Phys<R>& P, const R lf[9],
                                            const R lg[5], R af[9], R ag[5], MacAdj<R>& A) {
    const R r0 = P.rho0, ux = m.ux, uy = m.uy, Fx = m.Fx, Fy = m.Fy;
    const R rip = r0 * md.inv_phi;
    const R uu = ux * ux + uy * uy;
    // f+ = M^T a  =>  adjoint of a = M lf (rows 1..8 of Eq. (11)), then the 1/|row|^2 scaling
    const R s14 = (lf[1] + lf[2]) + (lf[3] + lf[4]);
    const R s58 = (lf[5] + lf[6]) + (lf[7] + lf[8]);
    const R qx = (lf[5] - lf[6]) - (lf[7] - lf[8]);
    const R qy = (lf[5] + lf[6]) - (lf[7] + lf[8]);
    const R lA1 = (R(2) * s58 - s14 - R(4) * lf[0]) * R(1.0 / 36.0);
    const R lA2 = (s58 - R(2) * s14 + R(4) * lf[0]) * R(1.0 / 36.0);
    const R lA3 = ((lf[1] - lf[3]) + qx) * R(1.0 / 6.0);
    const R lA4 = (qx - R(2) * (lf[1] - lf[3])) * R(1.0 / 12.0);
    const R lA5 = ((lf[2] - lf[4]) + qy) * R(1.0 / 6.0);
    const R lA6 = (qy - R(2) * (lf[2] - lf[4])) * R(1.0 / 12.0);
    const R lA7 = ((lf[1] - lf[2]) + (lf[3] - lf[4])) * R(0.25);
    const R lA8 = ((lf[5] - lf[6]) + (lf[7] - lf[8])) * R(0.25);
    // relaxation (Eq. (17))
    const R lm1 = (R(1) - P.s_e) * lA1, lm2 = (R(1) - P.s_eps) * lA2;
    const R lm4 = (R(1) - P.s_q) * lA4, lm6 = (R(1) - P.s_q) * lA6;
    const R lm7 = (R(1) - P.s_v) * lA7, lm8 = (R(1) - P.s_v) * lA8;
    const R le = P.s_e * lA1, leps = P.s_eps * lA2;
    const R lpxx = P.s_v * lA7, lpxy = P.s_v * lA8;
    const R lS1 = P.os_e * lA1 - P.os_eps * lA2;
    const R lS7 = P.os_v * lA7, lS8 = P.os_v * lA8;
    R lux = r0 * lA3 - P.s_q * r0 * lA4;
    R luy = r0 * lA5 - P.s_q * r0 * lA6;
    R lFx = R(0.5) * r0 * lA3 - P.os_q * r0 * lA4;
    R lFy = R(0.5) * r0 * lA5 - P.os_q * r0 * lA6;
    // equilibrium moments (Eq. (16)) and forcing (Eq. (19))
    A.P += R(6) * le - R(9) * leps;
    const R lRU = R(3) * (le - leps);           // adjoint of rip * uu
    R lrip = lRU * uu;
    R luu = lRU * rip;
    lrip += lpxx * (ux * ux - uy * uy) + lpxy * ux * uy;
    lux += R(2) * rip * ux * lpxx + rip * uy * lpxy;
    luy += -R(2) * rip * uy * lpxx + rip * ux * lpxy;
    const R uF = ux * Fx + uy * Fy;
    const R luF = R(6) * rip * lS1;
    lrip += R(6) * uF * lS1 + R(2) * (ux * Fx - uy * Fy) * lS7 + (ux * Fy + uy * Fx) * lS8;
    lux += luF * Fx + R(2) * rip * Fx * lS7 + rip * Fy * lS8;
    luy += luF * Fy - R(2) * rip * Fy * lS7 + rip * Fx * lS8;
    lFx += luF * ux + R(2) * rip * ux * lS7 + rip * uy * lS8;
    lFy += luF * uy - R(2) * rip * uy * lS7 + rip * ux * lS8;
    lux += R(2) * ux * luu;
    luy += R(2) * uy * luu;
    A.ip += r0 * lrip;
    // moments m' = M f' (rows 1, 2, 4, 6, 7, 8)
    af[0] += R(-4) * lm1 + R(4) * lm2;
    af[1] += -lm1 - R(2) * lm2 - R(2) * lm4 + lm7;
    af[2] += -lm1 - R(2) * lm2 - R(2) * lm6 - lm7;
    af[3] += -lm1 - R(2) * lm2 + R(2) * lm4 + lm7;
    af[4] += -lm1 - R(2) * lm2 + R(2) * lm6 - lm7;
    af[5] += R(2) * lm1 + lm2 + lm4 + lm6 + lm8;
    af[6] += R(2) * lm1 + lm2 - lm4 + lm6 - lm8;
    af[7] += R(2) * lm1 + lm2 - lm4 - lm6 + lm8;
    af[8] += R(2) * lm1 + lm2 + lm4 - lm6 - lm8;

    // thermal (Eq. (34)): g+ = N^T b  =>  adjoint of b = N lg
    const R lb0 = (lg[0] + lg[1]) + (lg[2] + lg[3]) + lg[4];
    const R lb1 = lg[1] - lg[3];
    const R lb2 = lg[2] - lg[4];
    const R lb3 = (lg[1] + lg[2]) + (lg[3] + lg[4]) - R(4) * lg[0];
    const R lb4 = (lg[1] - lg[2]) + (lg[3] - lg[4]);
    const R T = P.T0 + m.theta;
    const R ln1 = R(0.5) * (R(1) - P.z_T) * lb1;
    const R ln2 = R(0.5) * (R(1) - P.z_T) * lb2;
    const R ln3 = R(0.05) * (R(1) - P.z3) * lb3;
    const R ln4 = R(0.25) * (R(1) - P.z4) * lb4;
    const R kz = R(0.5) * P.z_T * P.inv_sigma;
    lux += kz * T * lb1;
    luy += kz * T * lb2;
    A.theta += R(0.2) * lb0 + R(0.05) * P.z3 * P.varpi * lb3 + kz * (ux * lb1 + uy * lb2);
    ag[0] += R(-4) * ln3;
    ag[1] += ln1 + ln3 + ln4;
    ag[2] += ln2 + ln3 - ln4;
    ag[3] += -ln1 + ln3 + ln4;
    ag[4] += -ln2 + ln3 - ln4;
    A.ux += lux;
    A.uy += luy;
    A.Fx += lFx;
    A.Fy += lFy;
}

// Reverse of fluid_macros(): adds to af, ag and to the medium adjoints lphi, lK.
template <typename R>
__device__ __forceinline__ void macros_vjp(const R f[9], const R g[5], R phi, R K,
                                           const Med<R>& md, const Phys<R>& P,
                                           const MacAdj<R>& A0, R af[9], R ag[5], R& lphi,
                                           R& lK) {
    // forward recompute, exactly as the forward step computes it
    const Vel<R> v = velocity<R>(f, g, md, P);
    const R Gx = v.Gx, Gy = v.Gy, hphi = R(0.5) * phi;
    const R vx = v.vx, vy = v.vy, l0 = v.l0, l1 = v.l1, vm = v.vm, q = v.q;
    const R inv_den = reciprocal(v.den), rq = recip(q), rK = recip(K);
    const R ux = v.ux, uy = v.uy, uu = v.uu, um = v.um, drag = v.drag;
    // reverse
    R lux = A0.ux, luy = A0.uy, lth = A0.theta, lip = A0.ip;
    R lGx = phi * A0.Fx, lGy = phi * A0.Fy;
    lphi += Gx * A0.Fx + Gy * A0.Fy;
    const R ldrag = -(ux * A0.Fx + uy * A0.Fy);
    lux -= drag * A0.Fx;
    luy -= drag * A0.Fy;
    R lclin = ldrag, lcnl = um * ldrag;
    const R lum = md.c_nl * ldrag;
    if (um > R(0)) {                  // d|u|/du, taken as 0 at u = 0
        lux += lum * ux / um;
        luy += lum * uy / um;
    }
    // P = 0.6 (sum18 - (2/3) rho0 uu / phi)
    const R lsum18 = R(0.6) * A0.P;
    const R luu = R(-0.4) * P.rho0 * md.inv_phi * A0.P;
    lip += R(-0.4) * P.rho0 * uu * A0.P;
    lux += R(2) * ux * luu;
    luy += R(2) * uy * luu;
    // u = v / den, den = l0 + sqrt(l0^2 + l1 |v|)
    R lvx = lux * inv_den, lvy = luy * inv_den;
    const R lden = -(lux * ux + luy * uy) * inv_den;
    const R lq = lden;
    const R ll0 = lden + quotient(lq * l0, q, rq);
    const R ll1 = quotient(lq * vm, R(2) * q, R(0.5) * rq);
    const R lvm = quotient(lq * l1, R(2) * q, R(0.5) * rq);
    if (vm > R(0)) {                  // d|v|/dv, taken as 0 at v = 0
        lvx += lvm * vx / vm;
        lvy += lvm * vy / vm;
    }
    lclin += R(0.25) * ll0;
    lcnl += R(0.5) * ll1;
    // v = j / rho0 + phi G / 2
    lphi += R(0.5) * (Gx * lvx + Gy * lvy);
    lGx += hphi * lvx;
    lGy += hphi * lvy;
    const R ljx = lvx * P.inv_rho0, ljy = lvy * P.inv_rho0;
    lth += P.gbeta * lGy;
    (void)lGx;
    // medium: ip = 1/phi, c_lin = phi nu / K, c_nl = C phi^(-1/2) K^(-1/2)
    lphi += -md.inv_phi * md.inv_phi * lip;
    lphi += md.c_lin * md.inv_phi * lclin;
    lK += quotient(-md.c_lin, K, rK) * lclin;
    lphi += R(-0.5) * md.c_nl * md.inv_phi * lcnl;
    lK += quotient(R(-0.5) * md.c_nl, K, rK) * lcnl;
    // populations
    af[1] += ljx + lsum18;
    af[2] += ljy + lsum18;
    af[3] += -ljx + lsum18;
    af[4] += -ljy + lsum18;
    af[5] += ljx + ljy + lsum18;
    af[6] += -ljx + ljy + lsum18;
    af[7] += -ljx - ljy + lsum18;
    af[8] += ljx - ljy + lsum18;
#pragma unroll
    for (int i = 0; i < 5; ++i) ag[i] += lth;
}

// Reverse of nee_wall() with respect to the neighbour's macroscopics: given the adjoints lfb,
// lgb of the rebuilt wall populations, adds to A the adjoints of the neighbour's ux, uy, 1/phi
// and theta.  The neighbour's pulled populations receive lfb and lgb unchanged.  Returns
// sum_i wt_i lgb_i, the adjoint of the wall temperature theta_b through the rebuilt g.
template <typename R>
__device__ __forceinline__ R nee_vjp(const Mac<R>& mf, const Med<R>& mdf, const Phys<R>& P,
                                     const R lfb[9], const R lgb[5], MacAdj<R>& A) {
    const R ux = mf.ux, uy = mf.uy, ip = mdf.inv_phi, r0 = P.rho0;
    // f_b,i = f_f,i - rho0 s_i(u; phi): s_i = w_i [3 e.u + 4.5 (e.u)^2 ip - 1.5 uu ip]
    const R ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    const R ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
    const R w[9] = {R(4.0 / 9.0), R(1.0 / 9.0), R(1.0 / 9.0), R(1.0 / 9.0), R(1.0 / 9.0),
                    R(1.0 / 36.0), R(1.0 / 36.0), R(1.0 / 36.0), R(1.0 / 36.0)};
    const R uu = ux * ux + uy * uy;
    R lux = 0, luy = 0, lip = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const R eu = ex[i] * ux + ey[i] * uy;
        const R c = -r0 * w[i] * lfb[i];
        lux += c * (R(3) * ex[i] + R(9) * eu * ex[i] * ip - R(3) * ux * ip);
        luy += c * (R(3) * ey[i] + R(9) * eu * ey[i] * ip - R(3) * uy * ip);
        lip += c * (R(4.5) * eu * eu - R(1.5) * uu);
    }
    // g_b,i = g_f,i + wt_i (theta_b - theta_f) - wt1 T_f u_coef (e_i . u)   (i >= 1)
    const R sw = P.wt0 * lgb[0] + P.wt1 * ((lgb[1] + lgb[2]) + (lgb[3] + lgb[4]));
    A.theta -= sw;                           // via theta_f
    const R k = P.wt1 * P.u_coef;
    const R Tf = P.T0 + mf.theta;
    const R dx = lgb[1] - lgb[3], dy = lgb[2] - lgb[4];
    lux -= k * Tf * dx;
    luy -= k * Tf * dy;
    A.theta -= k * (ux * dx + uy * dy);      // via T_f
    A.ux += lux;
    A.uy += luy;
    A.ip += lip;
    return sw;
}

template <typename R>
__device__ __forceinline__ bool on_wall(const Geo& G, int x, int y) {
    return (G.wallW && x == 0) || (G.wallE && x == G.nx - 1) || (G.wallS && y == 0) ||
           (G.wallN && y == G.ny - 1);
}

// Work-group tiles of the backward step, one work-item per node, one wavefront per row.
constexpr int kAdjTX = 64, kAdjTY = 4, kAdjThreads = kAdjTX * kAdjTY;
// What a wall node hands its inward neighbour: the adjoints of the neighbour's 14 pulled
// populations and of its ux, uy, 1/phi, theta and P.
constexpr int kHandoff = 19;

// A node's backward step up to the point where wall nodes hand their share over, and from there.
template <typename R>
struct AdjNode {
    R f[9], g[5], af[9], ag[5], phi, K;
    Med<R> md;
    MacAdj<R> A;
};

// Byte offsets, within a plane, of the node (x, y) and of the slots it owns: o[i] that of slot
// (i, x - e_i), wrapped (a slot beyond a wall is never used).  32-bit offsets from a plane's
// uniform base, as in pull: one vector register per place and no 64-bit arithmetic per access.
template <typename S>
struct AdjSlots {
    unsigned o[9];
    __device__ __forceinline__ AdjSlots(const Geo& G, int x, int y) {
        constexpr unsigned B = sizeof(S);
        const unsigned x0 = unsigned(x), xm = unsigned(x == 0 ? G.nx - 1 : x - 1);
        const unsigned xp = unsigned(x == G.nx - 1 ? 0 : x + 1);
        const unsigned pitch = unsigned(G.pitch), r0 = unsigned(y) * pitch;
        const unsigned rm = unsigned(y == 0 ? G.ny - 1 : y - 1) * pitch;
        const unsigned rp = unsigned(y == G.ny - 1 ? 0 : y + 1) * pitch;
        const unsigned q[9] = {r0 + x0, r0 + xm, rm + x0, r0 + xp, rp + x0,
                               rm + xm, rm + xp, rp + xp, rp + xm};
#pragma unroll
        for (int i = 0; i < 9; ++i) o[i] = q[i] * B;
    }
};

// Slots a node owns (population i at x - e_i), relative to the node.
__device__ constexpr int kEx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__device__ constexpr int kEy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};

// The medium at (px, py), the node whose pulled populations a node's state is built from: itself,
// or for a wall node its inward neighbour (the diagonal one at a corner).
template <typename S, typename R, bool PN>
__device__ __forceinline__ void adj_medium(const S* __restrict__ med, const Geo& G,
                                           const Phys<R>& P, int px, int py, AdjNode<R>& w) {
    if constexpr (PN) {
        const unsigned op = (unsigned(py) * unsigned(G.pitch) + unsigned(px)) * unsigned(sizeof(S));
        w.phi = R(at(med, op));
        w.K = R(at(plane(med, 1, G.plane), op));
        w.md = medium_from<R>(w.phi, w.K, P);
    } else {
        w.phi = P.phi;
        w.K = P.c_lin > R(0) ? w.phi * P.nu / P.c_lin : R(INFINITY);
        w.md = Med<R>{P.phi, P.inv_phi, P.c_lin, P.c_nl};
    }
}

// w.f, w.g: the populations of the forward state X^n (post-collision, entering step n) pulled at
// (px, py), with w's medium there; own_phi(): phi of a wall node itself; lout: adjoint of X^{n+1}
// in the node's own 14 slots.  A fluid node reverses its own collision.  A wall node runs the same
// macroscopics and collision VJP on its own reconstructed state (so both kinds of node stay in
// step), then reverses the reconstruction and calls at_wall(H, lphib): what its inward neighbour's
// macroscopics receive, and its own dJ/dphi.  Whatever a wall node does before the barrier goes in
// at_wall: in a branch of its own after this one it kept H and more alive for every node (vector
// registers of adjoint_step_kernel FP32 101 to 81, FP64 187 to 147, the wavefronts per SIMD 4 to 5
// and 2 to 3).
template <typename R, typename OwnPhi, typename AtWall>
__device__ __forceinline__ void adj_open(const Phys<R>& P, bool onW, bool onE, bool onS, bool onN,
                                         const R lout[14], AdjNode<R>& w, OwnPhi&& own_phi,
                                         AtWall&& at_wall) {
    const bool wall = onW || onE || onS || onN;
    R (&f)[9] = w.f;
    R (&g)[5] = w.g;
    const Mac<R> m = fluid_macros<R>(f, g, w.md, P);
    Mac<R> mc = m;
    Med<R> mdc = w.md;
    R theta_b = 0, phi_b = 0;
    if (wall) {
        // the wall node's state: rebuilt from its neighbour's, at rest, with its own phi
        theta_b = wall_theta<R>(onW, onE, onS, onN, m.theta, P);
        nee_wall<R>(f, g, m, w.md, theta_b, P);
        phi_b = own_phi();
        mc.theta = theta_b;
        mc.ux = R(0);
        mc.uy = R(0);
        mc.Fx = phi_b * P.ax;
        mc.Fy = phi_b * (P.ay + P.gbeta * theta_b);
        mdc = Med<R>{phi_b, reciprocal(phi_b), R(0), R(0)};
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) w.af[i] = R(0);
#pragma unroll
    for (int i = 0; i < 5; ++i) w.ag[i] = R(0);
    w.A = MacAdj<R>{};
    collide_vjp<R>(f, g, mc, mdc, P, lout, lout + 9, w.af, w.ag, w.A);
    if (wall) {
        // at rest the collision depends on 1/phi_b only through terms in u = 0, so phi_b
        // acts through F_b alone; theta_b through the collision, F_b and the rebuilt g
        const R Gy = P.ay + P.gbeta * theta_b;
        const R lphib = P.ax * w.A.Fx + Gy * w.A.Fy;
        const R lthb = w.A.theta + phi_b * P.gbeta * w.A.Fy;
        MacAdj<R> H{};
        const R sw = nee_vjp<R>(m, w.md, P, w.af, w.ag, H);
        const bool adiabatic = !((onW && P.iso[0]) || (onE && P.iso[1]) || (onS && P.iso[2]) ||
                                 (onN && P.iso[3]));
        if (adiabatic) H.theta += lthb + sw;    // theta_b = theta_f on an adiabatic side
        at_wall(H, lphib);
    }
}

// Value i of the kHandoff values a wall node hands over.
template <typename R, typename Put>
__device__ __forceinline__ void adj_hand_over(const AdjNode<R>& w, const MacAdj<R>& H, Put&& put) {
#pragma unroll
    for (int i = 0; i < 9; ++i) put(i, w.af[i]);
#pragma unroll
    for (int i = 0; i < 5; ++i) put(9 + i, w.ag[i]);
    put(14, H.ux);
    put(15, H.uy);
    put(16, H.ip);
    put(17, H.theta);
    put(18, w.A.P);
}

// A fluid node at (x, y) takes the hand-offs of the wall nodes whose inward neighbour it is, in a
// fixed order (get(i, dx, dy): value i of the wall node at (x + dx, y + dy)), then reverses its
// own macroscopics; af, ag become the adjoint of the slots it owns.
template <typename R, typename Get>
__device__ __forceinline__ void adj_close(const Geo& G, const Phys<R>& P, int x, int y,
                                          AdjNode<R>& w, R& lphi, R& lK, Get&& get) {
    const bool nearW = G.wallW && x == 1, nearE = G.wallE && x == G.nx - 2;
    const bool nearS = G.wallS && y == 1, nearN = G.wallN && y == G.ny - 2;
    if (nearW || nearE || nearS || nearN) {
        const bool has[8] = {nearW,          nearE,          nearS,          nearN,
                             nearW && nearS, nearE && nearS, nearW && nearN, nearE && nearN};
        const int dxs[8] = {-1, 1, 0, 0, -1, 1, -1, 1};
        const int dys[8] = {0, 0, -1, 1, -1, -1, 1, 1};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (!has[k]) continue;
#pragma unroll
            for (int i = 0; i < 9; ++i) w.af[i] += get(i, dxs[k], dys[k]);
#pragma unroll
            for (int i = 0; i < 5; ++i) w.ag[i] += get(9 + i, dxs[k], dys[k]);
            w.A.ux += get(14, dxs[k], dys[k]);
            w.A.uy += get(15, dxs[k], dys[k]);
            w.A.ip += get(16, dxs[k], dys[k]);
            w.A.theta += get(17, dxs[k], dys[k]);
            w.A.P += get(18, dxs[k], dys[k]);
        }
    }
    lphi = R(0);
    lK = R(0);
    macros_vjp<R>(w.f, w.g, w.phi, w.K, w.md, P, w.A, w.af, w.ag, lphi, lK);
}

// One backward step.  state: X^n; lam_in: adjoint of X^{n+1}; lam_out: adjoint of X^n (written);
// gphi, gK: FP64 gradient planes [ny][pitch] accumulated in place.  S: storage type of state,
// adjoint and medium; R: arithmetic type.
//
// A wall node's work-item adds its dJ/dphi (through F_b = phi_b G_b), writes zeros to its own
// slots (the forward step never reads them) and hands its inward neighbour, through LDS, what
// flows back through the reconstruction.  After one barrier the neighbour adds up to three
// hand-offs (two sides and their corner) before reversing its own macroscopics.
template <typename S, typename R, bool PN>
__global__ __launch_bounds__(kAdjThreads) void adjoint_step_kernel(
    const S* __restrict__ state, const S* __restrict__ lam_in, S* __restrict__ lam_out,
    const S* __restrict__ med, double* __restrict__ gphi, double* __restrict__ gK, Geo G,
    Phys<R> P, WallTiles T) {
    __shared__ R handoff[kHandoff][kAdjThreads];
    const int t = tile_index(), ty = t / T.nx_tiles, tx = t - ty * T.nx_tiles;
    int x0, x1, y0, y1;
    wall_span(tx, T.nx_tiles, kAdjTX, T.last_x0, G.nx, x0, x1);
    wall_span(ty, T.ny_tiles, kAdjTY, T.last_y0, G.ny, y0, y1);
    const int me = threadIdx.x;
    const int x = x0 + me % kAdjTX, y = y0 + me / kAdjTX;
    const bool active = x < x1 && y < y1;
    const bool onW = G.wallW && x == 0, onE = G.wallE && x == G.nx - 1;
    const bool onS = G.wallS && y == 0, onN = G.wallN && y == G.ny - 1;
    const bool wall = onW || onE || onS || onN;
    const int P1 = G.plane;
    const AdjSlots<S> sl(G, active ? x : 0, active ? y : 0);
    const unsigned og = (unsigned(y) * unsigned(G.pitch) + unsigned(x)) * unsigned(sizeof(double));

    AdjNode<R> w;
    // the gradient planes are read before the barrier, which global loads do not cross, so
    // that their latency hides behind the step's arithmetic
    double gphi0 = 0, gK0 = 0;
    if (active) {
        gphi0 = at(gphi, og);
        if (!wall) gK0 = at(gK, og);
        R lout[14];
#pragma unroll
        for (int i = 0; i < 14; ++i) lout[i] = R(at(plane(lam_in, i, P1), sl.o[0]));
        const int px = x + (onW ? 1 : 0) - (onE ? 1 : 0);
        const int py = y + (onS ? 1 : 0) - (onN ? 1 : 0);
        pull<R, S>(state, G, px, py, w.f, w.g);
        adj_medium<S, R, PN>(med, G, P, px, py, w);
        adj_open<R>(
            P, onW, onE, onS, onN, lout, w,
            [&]() { return PN ? R(med[size_t(y) * G.pitch + x]) : P.phi; },
            [&](const MacAdj<R>& H, R lphib) {
                adj_hand_over<R>(w, H, [&](int i, R v) { handoff[i][me] = v; });
                const bool okx_m = !onW, okx_p = !onE, oky_m = !onS, oky_p = !onN;
                const bool ok[9] = {true, okx_m, oky_m, okx_p, oky_p, okx_m && oky_m,
                                    okx_p && oky_m, okx_p && oky_p, okx_m && oky_p};
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    if (ok[i]) at(plane(lam_out, i, P1), sl.o[i]) = S(0);
#pragma unroll
                for (int i = 0; i < 5; ++i)
                    if (ok[i]) at(plane(lam_out, 9 + i, P1), sl.o[i]) = S(0);
                at(gphi, og) = gphi0 + double(lphib);
            });
    }
    __syncthreads();
    if (!active || wall) return;
    R lphi, lK;
    adj_close<R>(G, P, x, y, w, lphi, lK, [&](int i, int dx, int dy) {
        return handoff[i][me + dy * kAdjTX + dx];
    });
#pragma unroll
    for (int i = 0; i < 9; ++i) at(plane(lam_out, i, P1), sl.o[i]) = S(w.af[i]);
#pragma unroll
    for (int i = 0; i < 5; ++i) at(plane(lam_out, 9 + i, P1), sl.o[i]) = S(w.ag[i]);
    at(gphi, og) = gphi0 + double(lphi);
    at(gK, og) = gK0 + double(lK);
}

// kAdjSteps backward steps per launch, bitwise as that many launches of adjoint_step_kernel would
// take them: the adjoint of a tile of kAdjSide^2 nodes and its halo stays in LDS from step
// to step.  On a small grid a backward step is latency, not work: at 256^2 its kernel took 6.8 us
// (7.8 with the gap to the next), of which the arithmetic of one wavefront per SIMD is a quarter;
// the launch and the round trip of the adjoint through memory are paid once per launch here.  The
// dataflow is the forward tile's with the arrows turned round: node x writes slot
// (i, x - e_i), so a node may take step s when its neighbours took step s - 1, and step 1 covers
// the tile and kAdjSteps - 1 nodes more on each open side.  A wall node and its inward neighbour
// need each other within a step, so a region that would stop one node short of a wall takes the
// wall in.  The forward states of the steps come from the recomputed segment; hand-offs are
// indexed by the wall nodes' place along the region's sides; the gradient's sums are kept in LDS
// and take each step's terms in the order of single steps.
//
// AHEAD: while every tile has a compute unit of its own, a work-item keeps its node for all steps,
// with the medium and the place worked out once, and loads the next step's forward state before
// the step's arithmetic; the registers this takes (142 against 122) are free there.  Beyond, where
// two work-groups share a compute unit, they cost one of the two its place, and the nodes are
// dealt anew in each step.  lbm_grad, FP32, us per step, dealt / AHEAD: 48^2 6.70 / 5.72, 128^2
// 6.33 / 5.65, 256^2 7.02 / 6.58 (256 tiles); 250 x 300 (304 tiles) 8.6 / 10.3, 330^2 10.4 / 11.4.
constexpr int kAdjRegion = kAdjSide + 2 * (kAdjSteps - 1) + 2;   // region side at most
constexpr int kAdjTileThreads = (kAdjRegion * kAdjRegion + 63) / 64 * 64;
constexpr int kAdjAheadWGs = 256;   // tiles up to which AHEAD is taken: one per compute unit
constexpr int kAdjRow = kAdjRegion + 2;   // row of the adjoint in LDS: a margin on each side takes
                                          // the slots of the region's edge nodes that nobody reads

template <typename S>
struct AdjStates {
    const S* X[kAdjSteps];   // forward states of steps 1, 2, ... (backward in time)
};

template <typename S, typename R>
constexpr size_t adjoint_tile_lds() {
    return 2 * kAdjSide * kAdjSide * sizeof(double) + kHandoff * 4 * kAdjRegion * sizeof(R) +
           14 * size_t(kAdjRow) * kAdjRow * sizeof(S);
}

template <typename S, typename R, bool PN, bool AHEAD>
__global__ __launch_bounds__(kAdjTileThreads) void adjoint_tile_kernel(
    AdjStates<S> X, const S* __restrict__ lam_in, S* __restrict__ lam_out,
    const S* __restrict__ med, double* __restrict__ gphi, double* __restrict__ gK, Geo G,
    Phys<R> P, int tiles_x) {
    constexpr int TS = kAdjSide, W = kAdjRegion, LW = kAdjRow, L = LW * LW, K = kAdjSteps;
    extern __shared__ __align__(16) unsigned char adj_lds[];
    double* const grad = reinterpret_cast<double*>(adj_lds);           // [2][TS * TS]
    R* const hand = reinterpret_cast<R*>(grad + 2 * TS * TS);          // [kHandoff][4 * W]
    S* const lam = reinterpret_cast<S*>(hand + kHandoff * 4 * W);      // [14][L]

    const int t = tile_index(), ty = t / tiles_x, tx = t - ty * tiles_x;
    const int x0 = tx * TS, y0 = ty * TS;
    const int x1 = min(x0 + TS, G.nx), y1 = min(y0 + TS, G.ny);
    int rx0 = x0 - (K - 1), rx1 = x1 + K - 1, ry0 = y0 - (K - 1), ry1 = y1 + K - 1;
    int openW = 1, openE = 1, openS = 1, openN = 1;
    if (G.wallW && rx0 <= 1) { rx0 = 0; openW = 0; }
    if (G.wallE && rx1 >= G.nx - 1) { rx1 = G.nx; openE = 0; }
    if (G.wallS && ry0 <= 1) { ry0 = 0; openS = 0; }
    if (G.wallN && ry1 >= G.ny - 1) { ry1 = G.ny; openN = 0; }
    const int RW = rx1 - rx0, RH = ry1 - ry0;   // at most W each

    const int me = threadIdx.x;
    struct Place {
        int lx, ly, x, y, px, py, c, tn;   // in the region, the grid, pulled at, in LDS
        bool onW, onE, onS, onN, wall, inner, mine;
    };
    // the active nodes of step s, dealt row by row as in the forward tile
    auto deal = [&](int s) {
        const int ax = openW ? s - 1 : 0, ay = openS ? s - 1 : 0;
        const int aw = RW - (openE ? s - 1 : 0) - ax, ah = RH - (openN ? s - 1 : 0) - ay;
        const int row = int((float(me) + 0.5f) * __builtin_amdgcn_rcpf(float(aw)));
        Place q;
        q.mine = row < ah;
        q.lx = ax + me - row * aw;
        q.ly = ay + row;
        const int ux = rx0 + q.lx, uy = ry0 + q.ly;   // unwrapped
        q.x = ux;
        q.y = uy;
        if (!G.wallW) { q.x %= G.nx; q.x += q.x < 0 ? G.nx : 0; }
        if (!G.wallS) { q.y %= G.ny; q.y += q.y < 0 ? G.ny : 0; }
        q.onW = G.wallW && q.x == 0;
        q.onE = G.wallE && q.x == G.nx - 1;
        q.onS = G.wallS && q.y == 0;
        q.onN = G.wallN && q.y == G.ny - 1;
        q.wall = q.onW || q.onE || q.onS || q.onN;
        q.px = q.x + (q.onW ? 1 : 0) - (q.onE ? 1 : 0);
        q.py = q.y + (q.onS ? 1 : 0) - (q.onN ? 1 : 0);
        q.inner = q.mine && ux >= x0 && ux < x1 && uy >= y0 && uy < y1;
        q.c = (q.ly + 1) * LW + q.lx + 1;
        q.tn = (uy - y0) * TS + (ux - x0);
        return q;
    };

    // AHEAD: this work-item's node, the same for all steps, with its medium and the next step's
    // forward state
    Place kept;
    AdjNode<R> next;
    R own_phi = P.phi;
    if constexpr (AHEAD) {
        kept = deal(1);
        if (kept.mine) {
            pull<R, S>(X.X[0], G, kept.px, kept.py, next.f, next.g);
            adj_medium<S, R, PN>(med, G, P, kept.px, kept.py, next);
            if (PN && kept.wall) own_phi = R(med[size_t(kept.y) * G.pitch + kept.x]);
        }
    }

    // slots whose owner lies beyond a wall are never written and read as zero
    for (int k = me; k < 14 * L; k += kAdjTileThreads) lam[k] = S(0);

#pragma unroll 1
    for (int s = 1; s <= K; ++s) {
        if constexpr (AHEAD) {
            if (s > 1) {
                const int ax = openW ? s - 1 : 0, ay = openS ? s - 1 : 0;
                const int aw = RW - (openE ? s - 1 : 0) - ax, ah = RH - (openN ? s - 1 : 0) - ay;
                kept.mine = kept.mine && unsigned(kept.lx - ax) < unsigned(aw) &&
                            unsigned(kept.ly - ay) < unsigned(ah);
            }
            // hide that these do not change, so that the offsets derived from them are worked out
            // where they are used instead of being kept in registers through the loop
            asm volatile("" : "+v"(kept.x), "+v"(kept.y), "+v"(kept.px), "+v"(kept.py),
                         "+v"(kept.c), "+v"(kept.tn), "+v"(kept.lx), "+v"(kept.ly));
        }
        const Place q = AHEAD ? kept : deal(s);
        const int lx = q.lx, ly = q.ly, x = q.x, y = q.y, px = q.px, py = q.py, c = q.c, tn = q.tn;
        const bool onW = q.onW, onE = q.onE, onS = q.onS, onN = q.onN;
        const bool wall = q.wall, inner = q.inner, mine = q.mine;
        const unsigned on = unsigned(y) * unsigned(G.pitch) + unsigned(x);
        const unsigned og = on * unsigned(sizeof(double));
        double gphi0 = 0, gK0 = 0;
        AdjNode<R> w;
        MacAdj<R> H;   // a wall node's
        R lphib;
        if (mine) {
            R lout[14];
            if (s == 1) {
                if (inner) {
                    gphi0 = at(gphi, og);
                    if (!wall) gK0 = at(gK, og);
                }
#pragma unroll
                for (int i = 0; i < 14; ++i)
                    lout[i] = R(at(plane(lam_in, i, G.plane), on * unsigned(sizeof(S))));
            } else {
                if (inner) {
                    gphi0 = grad[tn];
                    if (!wall) gK0 = grad[TS * TS + tn];
                }
#pragma unroll
                for (int i = 0; i < 14; ++i) lout[i] = R(lam[i * L + c]);
            }
            if constexpr (AHEAD) {
                w.phi = next.phi;
                w.K = next.K;
                w.md = next.md;
#pragma unroll
                for (int i = 0; i < 9; ++i) w.f[i] = next.f[i];
#pragma unroll
                for (int i = 0; i < 5; ++i) w.g[i] = next.g[i];
                if (s < K) pull<R, S>(X.X[s], G, px, py, next.f, next.g);
            } else {
                pull<R, S>(X.X[s - 1], G, px, py, w.f, w.g);
                adj_medium<S, R, PN>(med, G, P, px, py, w);
            }
            adj_open<R>(
                P, onW, onE, onS, onN, lout, w,
                [&]() { return AHEAD || !PN ? own_phi : R(med[size_t(y) * G.pitch + x]); },
                [&](const MacAdj<R>& h, R l) {
                    H = h;
                    lphib = l;
                });
            if (wall) {   // apart here, where in the FP64 form it spills less so (20 B against 36)
                const int j = onW ? ly : onE ? W + ly : onS ? 2 * W + lx : 3 * W + lx;
                adj_hand_over<R>(w, H, [&](int i, R v) { hand[i * 4 * W + j] = v; });
            }
        }
        __syncthreads();   // hand-offs written, the adjoint read
        if (mine) {
            R lphi = R(0), lK = R(0);
            if (!wall)
                adj_close<R>(G, P, x, y, w, lphi, lK, [&](int i, int dx, int dy) {
                    const int j = dx < 0 ? ly + dy : dx > 0 ? W + ly + dy
                                               : dy < 0 ? 2 * W + lx : 3 * W + lx;
                    return hand[i * 4 * W + j];
                });
            if (wall) {   // the forward step never reads a wall node's own slots
#pragma unroll
                for (int i = 0; i < 9; ++i) w.af[i] = R(0);
#pragma unroll
                for (int i = 0; i < 5; ++i) w.ag[i] = R(0);
                lphi = lphib;
            }
            const double gp = gphi0 + double(lphi), gk = gK0 + double(lK);
            if (s < K) {
#pragma unroll
                for (int i = 0; i < 9; ++i) lam[i * L + c - kEy[i] * LW - kEx[i]] = S(w.af[i]);
#pragma unroll
                for (int i = 0; i < 5; ++i)
                    lam[(9 + i) * L + c - kEy[i] * LW - kEx[i]] = S(w.ag[i]);
                if (inner) {
                    grad[tn] = gp;
                    if (!wall) grad[TS * TS + tn] = gk;
                }
            } else if (inner) {
                const AdjSlots<S> sl(G, x, y);
                const bool ok[9] = {true, !onW, !onS, !onE, !onN, !onW && !onS, !onE && !onS,
                                    !onE && !onN, !onW && !onN};
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    if (ok[i]) at(plane(lam_out, i, G.plane), sl.o[i]) = S(w.af[i]);
#pragma unroll
                for (int i = 0; i < 5; ++i)
                    if (ok[i]) at(plane(lam_out, 9 + i, G.plane), sl.o[i]) = S(w.ag[i]);
                at(gphi, og) = gp;
                if (!wall) at(gK, og) = gk;
            }
        }
        if (s < K) __syncthreads();
    }
}

// Seed: adjoint of X^N for J = Nu_hot(T at time N).  T(x) = T0 + sum_i g_i(x - e_i) at a fluid
// node; at a wall node T is the wall value (isothermal side) or the inward neighbour's T.  One
// work-item per node of the first six columns; all other slots must already be zero.
template <typename R>
__device__ __forceinline__ double nu_weight(const Geo& G, int x, int y, double scale) {
    if (x > 4) return 0.0;
    const double c[5] = {-25.0, 48.0, -36.0, 16.0, -3.0};
    const double w = (y == 0 || y == G.ny - 1) ? 0.5 : 1.0;
    return scale * w * c[x] / 12.0;
}

template <typename S, typename R>
__global__ void adjoint_seed_kernel(S* __restrict__ lam, Geo G, Phys<R> P, double scale) {
    const int ncol = G.nx < 6 ? G.nx : 6;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= ncol * G.ny) return;
    const int y = k / ncol, x = k - y * ncol;
    if (on_wall<R>(G, x, y)) return;
    double c = nu_weight<R>(G, x, y, scale);
    const int dxs[8] = {-1, 1, 0, 0, -1, 1, -1, 1};
    const int dys[8] = {0, 0, -1, 1, -1, -1, 1, 1};
    for (int d = 0; d < 8; ++d) {
        const int xb = x + dxs[d], yb = y + dys[d];
        if (xb < 0 || xb >= G.nx || yb < 0 || yb >= G.ny) continue;
        const bool bW = G.wallW && xb == 0, bE = G.wallE && xb == G.nx - 1;
        const bool bS = G.wallS && yb == 0, bN = G.wallN && yb == G.ny - 1;
        if (!(bW || bE || bS || bN)) continue;
        if (xb + (bW ? 1 : 0) - (bE ? 1 : 0) != x || yb + (bS ? 1 : 0) - (bN ? 1 : 0) != y)
            continue;
        const bool adiabatic = !((bW && P.iso[0]) || (bE && P.iso[1]) || (bS && P.iso[2]) ||
                                 (bN && P.iso[3]));
        if (adiabatic) c += nu_weight<R>(G, xb, yb, scale);
    }
    if (c == 0.0) return;
    const int xm = (x == 0) ? G.nx - 1 : x - 1;
    const int xp = (x == G.nx - 1) ? 0 : x + 1;
    const int ym = (y == 0) ? G.ny - 1 : y - 1;
    const int yp = (y == G.ny - 1) ? 0 : y + 1;
    const int sx[5] = {x, xm, x, xp, x};
    const int sy[5] = {y, y, ym, y, yp};
#pragma unroll
    for (int i = 0; i < 5; ++i) lam[(9 + i) * G.plane + sy[i] * G.pitch + sx[i]] = S(c);
}

template <typename R>
__global__ void fill_zero_kernel(R* __restrict__ p, size_t n) {
    for (size_t k = blockIdx.x * size_t(blockDim.x) + threadIdx.x; k < n;
         k += size_t(gridDim.x) * blockDim.x)
        p[k] = R(0);
}

__global__ void unpitch_scale_kernel(double* __restrict__ dst, const double* __restrict__ src,
                                     Geo G, double scale) {
    const int n = G.nx * G.ny;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
        const int y = k / G.nx, x = k - y * G.nx;
        dst[k] = scale * src[y * G.pitch + x];
    }
}

template <typename S, typename R>
hipError_t launch_adjoint_seed(const void* state, void* lam, const Geo& G, const Phys<R>& P,
                               double L_over_dT, hipStream_t s) {
    (void)state;
    const int ncol = G.nx < 6 ? G.nx : 6;
    const int n = ncol * G.ny;
    const double scale = -L_over_dT / double(G.ny - 1);
    adjoint_seed_kernel<S, R><<<(n + 255) / 256, 256, 0, s>>>((S*)lam, G, P, scale);
    return hipGetLastError();
}

template <typename S, typename R>
hipError_t launch_adjoint_step(const void* state, const void* lam_in, void* lam_out,
                               const void* med, double* gphi, double* gK, const Geo& G,
                               const Phys<R>& P, hipStream_t s) {
    const WallTiles T = wall_tiles(G, kAdjTX, kAdjTY);
    const int nwg = T.nx_tiles * T.ny_tiles;
    if (med)
        adjoint_step_kernel<S, R, true><<<nwg, kAdjThreads, 0, s>>>(
            (const S*)state, (const S*)lam_in, (S*)lam_out, (const S*)med, gphi, gK, G, P, T);
    else
        adjoint_step_kernel<S, R, false><<<nwg, kAdjThreads, 0, s>>>(
            (const S*)state, (const S*)lam_in, (S*)lam_out, nullptr, gphi, gK, G, P, T);
    return hipGetLastError();
}

static int adjoint_tiles(const Geo& G) {
    return ((G.nx + kAdjSide - 1) / kAdjSide) * ((G.ny + kAdjSide - 1) / kAdjSide);
}

// Where kAdjSteps backward steps per launch beat one (us per step of lbm_grad, FP32, one / three:
// 64^2 9.2 / 5.7, 128^2 9.4 / 5.7, 256^2 8.8 / 6.6, 320^2 10.9 / 10.0, 384^2 13.8 / 14.4, 1024^2
// 62.6 / 69.3): up to about 320^2, where the launch costs more than the halo's redundant work
// (1.27 times the tile's nodes).  FP64 takes them where the tiles are AHEAD (48^2 9.6 / 8.6, 128^2
// 9.4 / 8.9, 256^2 11.4 / 10.8); beyond, and with FP64 arithmetic on FP32 storage (64^2 8.4 / 9.4,
// 256^2 9.1 / 12.1), a step of 1,100 instructions in a register-bound kernel is faster alone.
template <typename S, typename R>
bool adjoint_by_tiles(const Geo& G) {
    if (sizeof(R) == 4) return (long long)G.nx * G.ny <= 110000;
    return sizeof(S) == 8 && adjoint_tiles(G) <= kAdjAheadWGs;
}

template <typename S, typename R>
hipError_t launch_adjoint_tiles(const void* const states[kAdjSteps], const void* lam_in,
                                void* lam_out, const void* med, double* gphi, double* gK,
                                const Geo& G, const Phys<R>& P, hipStream_t s) {
    if constexpr (sizeof(S) == sizeof(R)) {
        AdjStates<S> X;
        for (int k = 0; k < kAdjSteps; ++k) X.X[k] = (const S*)states[k];
        const int tiles_x = (G.nx + kAdjSide - 1) / kAdjSide;
        const int nwg = adjoint_tiles(G);
        constexpr size_t lds = adjoint_tile_lds<S, R>();
        static_assert(lds <= 160 * 1024, "adjoint region exceeds the LDS of a CU");
        auto go = [&](auto pn, auto ahead) {
            adjoint_tile_kernel<S, R, decltype(pn)::value, decltype(ahead)::value>
                <<<nwg, kAdjTileThreads, lds, s>>>(X, (const S*)lam_in, (S*)lam_out,
                                                   (const S*)med, gphi, gK, G, P, tiles_x);
        };
        using Yes = std::true_type;
        using No = std::false_type;
        if (sizeof(R) == 8 || nwg <= kAdjAheadWGs) {
            med ? go(Yes{}, Yes{}) : go(No{}, Yes{});
        } else {
            if constexpr (sizeof(R) == 4) med ? go(Yes{}, No{}) : go(No{}, No{});
        }
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;
    }
}

template <typename R>
hipError_t launch_fill(void* dst, size_t n, hipStream_t s) {
    fill_zero_kernel<R><<<1024, 256, 0, s>>>((R*)dst, n);
    return hipGetLastError();
}

hipError_t launch_fill_f64(double* dst, size_t n, hipStream_t s) {
    fill_zero_kernel<double><<<1024, 256, 0, s>>>(dst, n);
    return hipGetLastError();
}

hipError_t launch_unpitch_scale(double* dst, const double* src, const Geo& G, double scale,
                                hipStream_t s) {
    unpitch_scale_kernel<<<1024, 256, 0, s>>>(dst, src, G, scale);
    return hipGetLastError();
}

#define LBM_ADJ_INSTANCES(S, R)                                                                  \
    template hipError_t launch_adjoint_seed<S, R>(const void*, void*, const Geo&,                \
                                                  const Phys<R>&, double, hipStream_t);          \
    template hipError_t launch_adjoint_step<S, R>(const void*, const void*, void*, const void*,  \
                                                  double*, double*, const Geo&, const Phys<R>&,  \
                                                  hipStream_t);                                  \
    template hipError_t launch_adjoint_tiles<S, R>(const void* const*, const void*, void*,       \
                                                   const void*, double*, double*, const Geo&,    \
                                                   const Phys<R>&, hipStream_t);                 \
    template bool adjoint_by_tiles<S, R>(const Geo&);
LBM_ADJ_INSTANCES(float, float)
LBM_ADJ_INSTANCES(double, double)
LBM_ADJ_INSTANCES(float, double)
#undef LBM_ADJ_INSTANCES
template hipError_t launch_fill<float>(void*, size_t, hipStream_t);
template hipError_t launch_fill<double>(void*, size_t, hipStream_t);

}  // namespace lbm
