// k_warm.hip - warm start of a run: the surrogate's inputs from the particle
// state, its outputs turned into particle velocities, and the fluid started
// from the creeping flow around each particle instead of from rest.
//
// Surrogate inputs (one thread per particle): with R(q) the body -> lab
// rotation, F_b = R^T F_ext, T_b = R^T T_ext, the equal-volume radius
// Req = (abc)^(1/3) and the load scale s = sqrt(|F_b|^2 + |T_b|^2 / Req^2):
//   x = (ln(a / sqrt(bc)), a / L, F_b / s, T_b / (Req s)),
// L = (nx ny nz / n)^(1/3), the box's volume per particle (n particles).
// Outputs y are the body-frame velocities in units of the Stokes scales:
//   U_b = y[0:3] s / (6 pi mu Req),  Omega_b = y[3:6] s / (8 pi mu Req^2).
// A squirmer carries no load of its own; it enters with the equivalent
// propulsive force along its axis (body x), the drag of a prolate spheroid
// translating along its axis at the free swimming speed of eq. squirmervel:
//   F_eff = 6 pi mu a X^A(e) U_s,  U_s = B1 e^-1 (e^-1 - (e^-2 - 1) arcoth(1/e)),
// e = sqrt(1 - b^2 / a^2), X^A(e) = (8/3) e^3 / (-2 e + (1 + e^2) ln((1+e)/(1-e)))
// (the sphere's limits 1 and 2 B1 / 3 for e -> 0), added to F_b.
//
// Start field: the creeping flow the particles' loads drive in the periodic
// box.  Per node, the sum over the box's particles of the free-space flow
// and pressure that the particle's load drives (particle_flow: the exact
// flow of a prolate spheroid, else that of the equal-volume sphere;
// minimum-image offsets, rigid inside the body), computed once per node
// (k_stokes_free) -- whose Fourier modes |n_i| <= 2 are replaced by those of
// the periodic solution of the same loads (the force spread as the traction
// on the translating ellipsoid, the torque as that on the rotating prolate
// spheroid, or over the sphere of radius Req for other bodies),
// so the box's slowest shear modes start at their steady values.  A fluid
// node's density carries the pressure, rho = rho0 + (p - pbar) / c_s^2 (pbar
// the fluid's mean: the mass is unchanged; without it the pressure builds up
// through sound waves that ring in the box for hundreds of steps), and the
// uniform velocity that makes the box's total momentum (fluid sum rho u plus
// particles) zero is removed; nodes inside particle p have rho0 and move
// rigidly with its U, Omega.  Every node gets the second-order equilibrium
// at its density and velocity, written as pre-collision populations (slot
// (x - c_i, i)).
#include <algorithm>
#include <type_traits>

#include "lbell_dev.h"
#include "lbell_launch.h"

namespace lbd {

__device__ __forceinline__ void body_to_lab(const double q[4], double Rm[3][3]) {
    const double q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
    Rm[0][0] = 1 - 2 * (q2 * q2 + q3 * q3);
    Rm[0][1] = 2 * (q1 * q2 - q0 * q3);
    Rm[0][2] = 2 * (q1 * q3 + q0 * q2);
    Rm[1][0] = 2 * (q1 * q2 + q0 * q3);
    Rm[1][1] = 1 - 2 * (q1 * q1 + q3 * q3);
    Rm[1][2] = 2 * (q2 * q3 - q0 * q1);
    Rm[2][0] = 2 * (q1 * q3 - q0 * q2);
    Rm[2][1] = 2 * (q2 * q3 + q0 * q1);
    Rm[2][2] = 1 - 2 * (q1 * q1 + q2 * q2);
}

__device__ __forceinline__ double eq_radius(const PartDev& P) { return cbrt(P.axes[0] * P.axes[1] * P.axes[2]); }

// Equivalent propulsive force of a squirmer along its body x axis (0 for a
// passive particle); a prolate spheroid, b taken as sqrt(bc).  Below
// e = 1e-3 the sphere's limits hold to 1e-6.
__device__ double propulsive_force(const PartDev& P, double mu) {
    if (P.B1 == 0.0) return 0.0;
    const double a = P.axes[0], b = sqrt(P.axes[1] * P.axes[2]);
    const double e = a > b ? sqrt(1.0 - (b / a) * (b / a)) : 0.0;
    double XA = 1.0, Us = 2.0 * P.B1 / 3.0;
    if (e >= 1e-3) {
        const double lg = log((1.0 + e) / (1.0 - e));
        XA = (8.0 / 3.0) * e * e * e / (-2.0 * e + (1.0 + e * e) * lg);
        Us = P.B1 / e * (1.0 / e - (1.0 / (e * e) - 1.0) * 0.5 * lg);
    }
    return 6.0 * M_PI * mu * a * XA * Us;
}

__global__ void k_warm_features(const BoxDesc* __restrict__ boxes, const PartDev* __restrict__ parts, int np,
                                double mu, float* __restrict__ X, double* __restrict__ s_out) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    const PartDev& P = parts[p];
    const BoxDesc& B = boxes[P.box];
    int nbox = 0;  // the box's particles (a one-off pass; np is at most 65534)
    for (int k = 0; k < np; ++k) nbox += parts[k].box == P.box;
    double Rm[3][3];
    body_to_lab(P.q, Rm);
    double Fb[3], Tb[3];
    for (int k = 0; k < 3; ++k) {
        Fb[k] = Rm[0][k] * P.Fext[0] + Rm[1][k] * P.Fext[1] + Rm[2][k] * P.Fext[2];
        Tb[k] = Rm[0][k] * P.Text[0] + Rm[1][k] * P.Text[1] + Rm[2][k] * P.Text[2];
    }
    Fb[0] += propulsive_force(P, mu);
    const double R = eq_radius(P);
    const double s = sqrt(Fb[0] * Fb[0] + Fb[1] * Fb[1] + Fb[2] * Fb[2] +
                          (Tb[0] * Tb[0] + Tb[1] * Tb[1] + Tb[2] * Tb[2]) / (R * R));
    float* x = X + (long long)p * MLP_IN;
    x[0] = (float)log(P.axes[0] / sqrt(P.axes[1] * P.axes[2]));
    x[1] = (float)(P.axes[0] / cbrt((double)B.nx * B.ny * B.nz / nbox));
    for (int k = 0; k < 3; ++k) {
        x[2 + k] = s > 0 ? (float)(Fb[k] / s) : 0.f;
        x[5 + k] = s > 0 ? (float)(Tb[k] / (R * s)) : 0.f;
    }
    s_out[p] = s;
}

__global__ void k_warm_apply(PartDev* __restrict__ parts, int np, const float* __restrict__ Y,
                             const double* __restrict__ s_in, double mu, double* __restrict__ pred, int only_box) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    PartDev& P = parts[p];
    if (only_box >= 0 && P.box != only_box) return;
    double Rm[3][3];
    body_to_lab(P.q, Rm);
    const double R = eq_radius(P), s = s_in[p];
    const double cu = s / (6.0 * M_PI * mu * R), cw = s / (8.0 * M_PI * mu * R * R);
    const float* y = Y + (long long)p * MLP_OUT;
    double Ub[3] = {y[0] * cu, y[1] * cu, y[2] * cu}, Wb[3] = {y[3] * cw, y[4] * cw, y[5] * cw};
    {  // a prediction above the surface-speed limit of the solve is scaled down to it
        const double amax = fmax(P.axes[0], fmax(P.axes[1], P.axes[2]));
        const double sp = sqrt(Ub[0] * Ub[0] + Ub[1] * Ub[1] + Ub[2] * Ub[2]) +
                          sqrt(Wb[0] * Wb[0] + Wb[1] * Wb[1] + Wb[2] * Wb[2]) * amax;
        if (!(sp <= 0.5)) {
            const double f = sp > 0.5 && sp <= 1e300 ? 0.5 / sp : 0.0;  // a non-finite prediction becomes rest
            for (int k = 0; k < 3; ++k) {
                Ub[k] = f == 0.0 ? 0.0 : Ub[k] * f;
                Wb[k] = f == 0.0 ? 0.0 : Wb[k] * f;
            }
        }
    }
    for (int k = 0; k < 3; ++k) {
        P.U[k] = Rm[k][0] * Ub[0] + Rm[k][1] * Ub[1] + Rm[k][2] * Ub[2];
        P.W[k] = Rm[k][0] * Wb[0] + Rm[k][1] * Wb[1] + Rm[k][2] * Wb[2];
        pred[6 * p + k] = P.U[k];
        pred[6 * p + 3 + k] = P.W[k];
    }
}

// Normalised body-frame response of every particle at its current
// velocities (the training target of the surrogate; inverse of k_warm_apply).
__global__ void k_warm_targets(const PartDev* __restrict__ parts, int np, const double* __restrict__ s_in,
                               double mu, float* __restrict__ Y) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    const PartDev& P = parts[p];
    double Rm[3][3];
    body_to_lab(P.q, Rm);
    const double R = eq_radius(P), s = s_in[p];
    const double cu = s > 0 ? 6.0 * M_PI * mu * R / s : 0.0, cw = s > 0 ? 8.0 * M_PI * mu * R * R / s : 0.0;
    float* y = Y + (long long)p * MLP_OUT;
    for (int k = 0; k < 3; ++k) {
        y[k] = (float)(cu * (Rm[0][k] * P.U[0] + Rm[1][k] * P.U[1] + Rm[2][k] * P.U[2]));
        y[3 + k] = (float)(cw * (Rm[0][k] * P.W[0] + Rm[1][k] * P.W[1] + Rm[2][k] * P.W[2]));
    }
}

// minimum-image offset of node (x, y, z) from the particle centre
__device__ __forceinline__ void offset(const double xc[3], const BoxDesc& B, int x, int y, int z, double d[3]) {
    const int n[3] = {B.nx, B.ny, B.nz};
    const int c[3] = {x, y, z};
    for (int k = 0; k < 3; ++k) {
        double v = c[k] - xc[k];
        if (v >= 0.5 * n[k]) v -= n[k];
        if (v < -0.5 * n[k]) v += n[k];
        d[k] = v;
    }
}

constexpr int WK = 2;                  // modes |n_i| <= WK carry the periodic correction
constexpr int WM = (2 * WK + 1) * (2 * WK + 1) * (2 * WK + 1);  // mode slots per box (index 62 = n = 0)

__device__ __forceinline__ int wk_axis(int L) { return min(WK, (L - 1) / 2); }

// Gauss-Legendre rules on [-1, 1] of 32, 24, 16, 12 and 8 points, one table:
// the positive nodes and their weights of each (the rules are symmetric).
constexpr int GL32 = 0, GL24 = 16, GL16 = 28, GL12 = 36, GL8 = 42;
__constant__ double GLTAB[46][2] = {
    {0.04830766568773832, 0.0965400885147278}, {0.1444719615827965, 0.09563872007927486},
    {0.23928736225213706, 0.09384439908080457}, {0.33186860228212767, 0.09117387869576389},
    {0.42135127613063533, 0.08765209300440381}, {0.5068999089322294, 0.08331192422694675},
    {0.5877157572407623, 0.07819389578707031}, {0.6630442669302152, 0.0723457941088485},
    {0.7321821187402897, 0.06582222277636185}, {0.7944837959679424, 0.058684093478535544},
    {0.84936761373257, 0.050998059262376175}, {0.8963211557660521, 0.04283589802222668},
    {0.9349060759377397, 0.03427386291302143}, {0.9647622555875064, 0.02539206530926206},
    {0.9856115115452684, 0.01627439473090567}, {0.9972638618494816, 0.007018610009470096},
    {0.06405689286260563, 0.12793819534675216}, {0.1911188674736163, 0.1258374563468283},
    {0.3150426796961634, 0.12167047292780339}, {0.4337935076260451, 0.1155056680537256},
    {0.5454214713888396, 0.10744427011596563}, {0.6480936519369755, 0.09761865210411388},
    {0.7401241915785544, 0.08619016153195327}, {0.820001985973903, 0.0733464814110803},
    {0.8864155270044011, 0.05929858491543678}, {0.9382745520027328, 0.04427743881741981},
    {0.9747285559713095, 0.028531388628933663}, {0.9951872199970213, 0.0123412297999872},
    {0.09501250983763744, 0.1894506104550685}, {0.2816035507792589, 0.18260341504492358},
    {0.45801677765722737, 0.16915651939500254}, {0.6178762444026438, 0.14959598881657674},
    {0.755404408355003, 0.12462897125553388}, {0.8656312023878318, 0.09515851168249279},
    {0.9445750230732326, 0.062253523938647894}, {0.9894009349916499, 0.027152459411754096},
    {0.1252334085114689, 0.24914704581340277}, {0.3678314989981802, 0.2334925365383548},
    {0.5873179542866175, 0.20316742672306592}, {0.7699026741943047, 0.16007832854334622},
    {0.9041172563704749, 0.10693932599531843}, {0.9815606342467192, 0.04717533638651183},
    {0.1834346424956498, 0.362683783378362}, {0.525532409916329, 0.31370664587788727},
    {0.7966664774136267, 0.22238103445337448}, {0.9602898564975362, 0.10122853629037626},
};

// Below this eccentricity a prolate spheroid's flow is taken as the sphere's
// (the two differ by O(e^2)).
constexpr double E_LINE = 1e-4;
constexpr int UF = 4;  // doubles per node of the staged free field: velocity, pressure
constexpr int MC = 8;  // doubles per mode: (re, im) of velocity and pressure
constexpr int MODE_HALF = (2 * WK + 1) * (WK + 1) * UF;   // (n_x, n_y >= 0, component) of a slab's sums
constexpr int SLAB = MODE_HALF * (2 * WK + 1) * 2;         // doubles per slab: for each n_z, (re, im)
constexpr int NPART = 8;  // partial sums per tile of k_stokes_sum

__device__ __forceinline__ bool loaded(const PartDev& P) {
    return P.Fext[0] != 0.0 || P.Fext[1] != 0.0 || P.Fext[2] != 0.0 || P.Text[0] != 0.0 || P.Text[1] != 0.0 ||
           P.Text[2] != 0.0;
}

// Free-space creeping flow that the load of particle P drives, added to
// (u[0..2], u[3]) = (velocity, pressure) at offset d from its centre; rigid
// motion and no pressure inside the body.  The pressure is that of the
// Stokeslets, 2 mu (s.r) / R^3, and of the stresslets, 2 mu (r.p)(r.m) / R^5
// times theirs; the potential singularities and the rotlets carry none
// (the sphere: 3 mu R (U.d) / (2 r^3) = F.d / (4 pi r^3)).
//
// Prolate spheroid (a > b = c): the exact solution of Chwang & Wu (J. Fluid
// Mech. 63, 1974; 67, 1975) as singularities on the focal segment |xi| <= f,
// f = a e, axis p, g(xi) = f^2 - xi^2, r = d - xi p, R = |r|; with
// s = F / (16 pi mu f) and t = T / (8 pi mu (4/3) f^3), t_c its part across p:
//   Stokeslets s / R + (s.r) r / R^3 (uniform: they carry the force),
//   potential dipoles -(1 - e^2) / (2 e^2) g [-s / R^3 + 3 (s.r) r / R^5],
//   rotlets g t x r / R^3 (they carry the torque),
//   stresslets 3 e^2 / (2 - e^2) g r (r.p)(r.m) / R^5, m = t_c x p,
//   potential quadrupoles (1 - e^2) / (4 (2 - e^2)) g^2 (p.grad) of the
//   dipole of m: 3 (m (r.p) + (r.m) p) / R^5 - 15 (r.m)(r.p) r / R^7.
// The body moves with the velocities of eq. drag4's X^A, Y^A, X^C, Y^C:
// V = F_p / (16 pi mu f alpha_p) + F_c / (16 pi mu f alpha_c), alpha_p =
// e^2 / D1, alpha_c = 2 e^2 / D2; Omega = t_p D3 / (1 - e^2) + t_c D1 /
// (2 - e^2); D1 = -2e + (1 + e^2) L, D2 = 2e + (3e^2 - 1) L, D3 = 2e -
// (1 - e^2) L, L = ln((1 + e) / (1 - e)) (power series below e = 1/2, where
// they cancel).
//
// With d = z p + n, n across the axis, and zeta = z - xi, r = zeta p + n, so
// (s.r) = s.n + zeta s.p, (r.m) = n.m (m is across p), and the flow is
//   s A + n B + p (B_zeta + E) + (t x n) C + (t x p) C_zeta + m D
// of eight scalar integrals over the segment (the eighth is the pressure).
// The points of the integrals depend on delta, the distance from d to
// the segment.  From 0.8 f on the integrands are smooth and plain
// Gauss-Legendre over the whole segment converges: 32 points, 24 from
// 1.15 f, 16 from 1.95 f, 12 from 3.2 f, 8 from 9 f (truncation below 1e-16 of
// the velocity at these lines for aspect ratios 1.02 to 5, measured in
// extended precision).  Nearer, the substitution xi = x0 -+ delta sinh(t) about
// the point x0 of the segment nearest d smooths the peak, with
// 24 points on each side of x0 within f / 2 and 16 beyond (within ~2e-15 of
// the integral); the nodes +-x of a rule share one exponential,
// e^t = e^(tm/2) e^(+-tm x/2).
// Every other shape: the sphere of radius Req = (abc)^(1/3) moving with
// F / (6 pi mu Req) and turning with T / (8 pi mu Req^3) (Stokes' solution
// and the rotlet), rigid inside Req.
//
// FlowConst: everything above that does not depend on the node, once per
// particle (k_stokes_prep).
struct FlowConst {
    double xc[3], p[3], S[3], Sp, G[3], Gp[3], m[3], U[3], W[3];
    double f, if_, bfac, dl, ka, ia2, ib2, mu2, R;
    int line, torque;
};
constexpr int FLOW_DOUBLES = (int)(sizeof(FlowConst) / sizeof(double));
static_assert(sizeof(FlowConst) % sizeof(double) == 0, "FlowConst is stored in a scratch of doubles");

__device__ void flow_const(const PartDev& P, double mu, FlowConst& C) {
    const double a = P.axes[0], b = P.axes[1];
    const double e2 = a > b && b == P.axes[2] ? 1.0 - (b / a) * (b / a) : 0.0;
    for (int k = 0; k < 3; ++k) C.xc[k] = P.xc[k];
    C.line = e2 >= E_LINE * E_LINE;
    C.torque = P.Text[0] != 0.0 || P.Text[1] != 0.0 || P.Text[2] != 0.0;
    C.mu2 = 2.0 * mu;
    C.R = eq_radius(P);
    if (!C.line) {
        const double R = C.R;
        const double cu = 1.0 / (6.0 * M_PI * mu * R), cw = 1.0 / (8.0 * M_PI * mu * R * R * R);
        for (int k = 0; k < 3; ++k) {
            C.U[k] = P.Fext[k] * cu;
            C.W[k] = P.Text[k] * cw;
        }
        return;
    }
    const double e = sqrt(e2), f = a * e;
    double D1 = 0.0, D2 = 0.0, D3 = 0.0;
    if (e < 0.5) {  // D1 = sum 8k e^(2k+1) / (4k^2 - 1), D2 = sum 8(k+1) ..., D3 = sum 4 ... (k >= 1)
        double ek = e * e2;
        for (int k = 1; k <= 30; ++k) {
            const double den = 4.0 * k * k - 1.0;
            D1 += 8.0 * k * ek / den;
            D2 += 8.0 * (k + 1) * ek / den;
            D3 += 4.0 * ek / den;
            ek *= e2;
        }
    } else {
        const double L = log((1.0 + e) / (1.0 - e));
        D1 = -2.0 * e + (1.0 + e2) * L;
        D2 = 2.0 * e + (3.0 * e2 - 1.0) * L;
        D3 = 2.0 * e - (1.0 - e2) * L;
    }
    C.f = f;
    C.if_ = 1.0 / f;
    C.bfac = -(1.0 - e2) / (2.0 * e2);
    C.dl = 3.0 * e2 / (2.0 - e2);
    C.ka = (1.0 - e2) / (4.0 * (2.0 - e2));
    C.ia2 = 1.0 / (a * a);
    C.ib2 = 1.0 / (b * b);
    double Rm[3][3];
    body_to_lab(P.q, Rm);
    const double p[3] = {Rm[0][0], Rm[1][0], Rm[2][0]};
    const double Fp = P.Fext[0] * p[0] + P.Fext[1] * p[1] + P.Fext[2] * p[2];
    const double Tp = P.Text[0] * p[0] + P.Text[1] * p[1] + P.Text[2] * p[2];
    const double cf = 1.0 / (16.0 * M_PI * mu * f), ct = 1.0 / (8.0 * M_PI * mu * (4.0 / 3.0) * f * f * f);
    double Gc[3];
    for (int k = 0; k < 3; ++k) {
        C.p[k] = p[k];
        C.S[k] = P.Fext[k] * cf;
        C.G[k] = P.Text[k] * ct;
        Gc[k] = (P.Text[k] - Tp * p[k]) * ct;
        C.U[k] = Fp * p[k] * cf * D1 / e2 + (P.Fext[k] - Fp * p[k]) * cf * D2 / (2.0 * e2);
        C.W[k] = Tp * p[k] * ct * D3 / (1.0 - e2) + Gc[k] * D1 / (2.0 - e2);
    }
    C.Sp = Fp * cf;
    const double* G = C.G;
    const double m[3] = {Gc[1] * p[2] - Gc[2] * p[1], Gc[2] * p[0] - Gc[0] * p[2], Gc[0] * p[1] - Gc[1] * p[0]};
    const double Gp[3] = {G[1] * p[2] - G[2] * p[1], G[2] * p[0] - G[0] * p[2], G[0] * p[1] - G[1] * p[0]};
    for (int k = 0; k < 3; ++k) {
        C.m[k] = m[k];
        C.Gp[k] = Gp[k];
    }
}

// One thread per particle: its constants, and the box it loads (-1: none).
__global__ void k_stokes_prep(const PartDev* __restrict__ parts, int np, double mu, FlowConst* __restrict__ fc,
                              int* __restrict__ pbox) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    const bool use = loaded(parts[p]);
    pbox[p] = use ? parts[p].box : -1;
    if (use) flow_const(parts[p], mu, fc[p]);
}

// x^(-1/2) of a normal x > 0: the instruction's estimate and one third-order
// step, y (1 + e (1/2 + 3 e / 8)), e = 1 - x y^2, without the library's
// selects for zero and infinity (R2 is a squared distance outside the body).
__device__ __forceinline__ double inv_sqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// The eight integrals of particle_flow, a point at a time.
struct LineSums {
    double A, B, Bz, C, Cz, D, E, pr;
};
template <bool TORQUE>
__device__ __forceinline__ void line_point(const FlowConst& K, double n2, double Sn, double nm, double zeta, double g,
                                           double wq, LineSums& I) {
    const double R2 = n2 + zeta * zeta;
    const double iR = inv_sqrt(R2), iR2 = iR * iR, iR3 = iR * iR2;
    const double Sr = Sn + K.Sp * zeta, cS3 = K.bfac * g * iR2;  // cS3 / R: the dipoles' weight over R^3
    double B = Sr * iR3 * (1.0 + 3.0 * cS3), pr = Sr * iR3;
    I.A += wq * (iR * (1.0 - cS3));
    if constexpr (TORQUE) {
        const double iR5 = iR3 * iR2, cQ = K.ka * g * g, rpm = zeta * nm * iR5, st = K.dl * g * rpm;
        B += st - 15.0 * cQ * iR2 * rpm;
        pr += st;
        const double c = wq * g * iR3, q = 3.0 * wq * cQ * iR5;
        I.C += c;
        I.Cz += c * zeta;
        I.D += q * zeta;
        I.E += q * nm;
    }
    I.B += wq * B;
    I.Bz += wq * B * zeta;
    I.pr += wq * pr;
}

template <bool TORQUE>
__device__ __forceinline__ void line_sums(const FlowConst& K, double z, double n2, double Sn, double nm, LineSums& I) {
    const double f = K.f;
    const double x0 = fmin(fmax(z, -f), f), zx = z - x0;
    const double d2 = n2 + zx * zx;  // delta^2 > 0: the segment lies inside the body
    const double q2 = d2 * (K.if_ * K.if_);
    // (delta / f)^2 below the square of a line
    auto below = [&](double line) { return q2 < line * line; };
    // the rule is the wave's: the one its nearest node on this side of 0.8 f
    // needs (so the table is read with scalar loads and no lane waits for a
    // longer rule than its own row of nodes)
    if (!below(0.8)) {
        const bool b1 = __any(below(1.15)), b2 = __any(below(1.95)), b3 = __any(below(3.2)), b4 = __any(below(9.0));
        const int row = b1 ? GL32 : (b2 ? GL24 : (b3 ? GL16 : (b4 ? GL12 : GL8)));
        const int half = b1 ? 16 : (b2 ? 12 : (b3 ? 8 : (b4 ? 6 : 4)));
#pragma unroll 2
        for (int j = 0; j < half; ++j) {
            const double xi = f * GLTAB[row + j][0], wq = f * GLTAB[row + j][1], g = (f - xi) * (f + xi);
            line_point<TORQUE>(K, n2, Sn, nm, z - xi, g, wq, I);
            line_point<TORQUE>(K, n2, Sn, nm, z + xi, g, wq, I);
        }
        return;
    }
    const bool near = __any(below(0.5));
    const int row = near ? GL24 : GL16, half = near ? 12 : 8;
    const double idel = inv_sqrt(d2), delta = d2 * idel;
    for (int side = 0; side < 2; ++side) {
        const double sgn = side ? 1.0 : -1.0, len = side ? f - x0 : x0 + f;
        if (len <= 0.0) continue;
        const double sl = len * idel, tm = asinh(sl), et = sqrt(sl + sqrt(1.0 + sl * sl)), it = 1.0 / et;
        const double wh = 0.25 * tm * delta, hd = 0.5 * delta;
        for (int j = 0; j < half; ++j) {
            const double eh = exp(0.5 * tm * GLTAB[row + j][0]), ih = 1.0 / eh, w = wh * GLTAB[row + j][1];
#pragma unroll
            for (int v = 0; v < 2; ++v) {  // e^t and e^-t of the two nodes
                const double ep = v ? et * eh : et * ih, em = v ? it * ih : it * eh;
                const double off = sgn * hd * (ep - em);  // xi = x0 + off
                line_point<TORQUE>(K, n2, Sn, nm, zx - off, ((f - x0) - off) * ((f + x0) + off), w * (ep + em), I);
            }
        }
    }
}

__device__ __forceinline__ void particle_flow(const FlowConst& K, const double d[3], double u[4]) {
    const double *U = K.U, *W = K.W;
    if (!K.line) {
        const double r = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        const double R = K.R, mu = 0.5 * K.mu2;
        const double wx[3] = {W[1] * d[2] - W[2] * d[1], W[2] * d[0] - W[0] * d[2], W[0] * d[1] - W[1] * d[0]};
        if (r < R) {
            for (int k = 0; k < 3; ++k) u[k] += U[k] + wx[k];
            return;
        }
        const double ex[3] = {d[0] / r, d[1] / r, d[2] / r};
        const double Ue = U[0] * ex[0] + U[1] * ex[1] + U[2] * ex[2];
        const double a1 = 0.75 * R / r, a3 = 0.25 * R * R * R / (r * r * r), rr = (R / r) * (R / r) * (R / r);
        for (int k = 0; k < 3; ++k)
            u[k] += a1 * (U[k] + Ue * ex[k]) + a3 * (U[k] - 3.0 * Ue * ex[k]) + rr * wx[k];
        u[3] += 1.5 * mu * R * Ue / (r * r);
        return;
    }
    const double* p = K.p;
    const double z = d[0] * p[0] + d[1] * p[1] + d[2] * p[2];
    const double n[3] = {d[0] - z * p[0], d[1] - z * p[1], d[2] - z * p[2]};
    const double n2 = n[0] * n[0] + n[1] * n[1] + n[2] * n[2];
    if (z * z * K.ia2 + n2 * K.ib2 < 1.0) {  // inside: rigid motion
        u[0] += U[0] + W[1] * d[2] - W[2] * d[1];
        u[1] += U[1] + W[2] * d[0] - W[0] * d[2];
        u[2] += U[2] + W[0] * d[1] - W[1] * d[0];
        return;
    }
    const double *S = K.S, *G = K.G;
    const double Sn = S[0] * n[0] + S[1] * n[1] + S[2] * n[2];
    LineSums I = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (K.torque) {  // the same for every node of the particle
        line_sums<true>(K, z, n2, Sn, n[0] * K.m[0] + n[1] * K.m[1] + n[2] * K.m[2], I);
        const double Gn[3] = {G[1] * n[2] - G[2] * n[1], G[2] * n[0] - G[0] * n[2], G[0] * n[1] - G[1] * n[0]};
        for (int k = 0; k < 3; ++k) u[k] += Gn[k] * I.C + K.Gp[k] * I.Cz + K.m[k] * I.D;
    } else {
        line_sums<false>(K, z, n2, Sn, 0.0, I);
    }
    for (int k = 0; k < 3; ++k) u[k] += S[k] * I.A + n[k] * I.B + p[k] * (I.Bz + I.E);
    u[3] += K.mu2 * I.pr;
}

// Free-space flow and pressure of every node of the started boxes (the sum
// over each box's loaded particles of particle_flow), node-major into uf at
// UF * (ooff + site - base).  A work-group per tile; the box's loaded particles
// are listed in index order, TILE at a time, in LDS.
// Bound by FP64 arithmetic (84 % of the issue slots; 28 operations a point);
// four waves to a SIMD at the price of 29 spilled values beat two without, and
// three are no better.  64 boxes, 7.7 M nodes: 412 us (461 with the library's
// rsqrt, a square root for the rule and divisions for the node's place; 1507
// with the constants per node, two-sided rules everywhere and the vector terms
// inside the quadrature).  Waves of 4 x 4 x 4 nodes in place of rows would need
// 5 to 10 % fewer points.
__global__ __launch_bounds__(TILE, 4) void k_stokes_free(const BoxDesc* __restrict__ boxes,
                                                      const int* __restrict__ tile_box,
                                                      const FlowConst* __restrict__ fc,
                                                      const int* __restrict__ pbox, int np, int only_box,
                                                      long long base, double* __restrict__ uf) {
    __shared__ int list[TILE];
    __shared__ int wcnt[TILE / 64];
    const int tile = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int bi = tile_box[tile];
    if (only_box >= 0 && bi != only_box) return;  // uniform over the block
    const BoxDesc& B = boxes[bi];
    const int s = (tile - B.tile0) * TILE + tid;
    int x, y;
    const int z = div_magic(div_magic(s, B.nx, B.mnx, B.lnx, x), B.ny, B.mny, B.lny, y);
    double u[UF] = {0.0, 0.0, 0.0, 0.0};
    for (int p0 = 0; p0 < np; p0 += TILE) {
        const int p = p0 + tid;
        const bool take = p < np && pbox[p] == bi;
        const unsigned long long bal = __ballot(take);
        if (lane == 0) wcnt[wv] = __popcll(bal);
        __syncthreads();
        int off = 0, cnt = 0;
        for (int w = 0; w < TILE / 64; ++w) {
            off += w < wv ? wcnt[w] : 0;
            cnt += wcnt[w];
        }
        if (take) list[off + __popcll(bal & ((1ull << lane) - 1ull))] = p;
        __syncthreads();
        if (s < B.n)
            for (int j = 0; j < cnt; ++j) {
                // one particle for the whole wave: its constants are scalar loads
                const FlowConst& K = fc[__builtin_amdgcn_readfirstlane(list[j])];
                double d[3];
                offset(K.xc, B, x, y, z, d);
                particle_flow(K, d, u);
            }
        __syncthreads();
    }
    if (s < B.n) {
        double2* o = reinterpret_cast<double2*>(uf + UF * (B.ooff + s - base));
        o[0] = double2{u[0], u[1]};
        o[1] = double2{u[2], u[3]};
    }
}

// exp(i 2 pi n x / L) for n = -WK..WK (WK = 2) into e[n + WK] (re, im):
// powers of the n = 1 term, the negative ones conjugate.
static_assert(WK == 2, "twiddles() builds the modes |n| <= 2");
__device__ __forceinline__ void powers(double c1, double s1, double e[2 * WK + 1][2]) {
    const double c2 = c1 * c1 - s1 * s1, s2 = 2.0 * s1 * c1;
    e[WK][0] = 1.0;
    e[WK][1] = 0.0;
    e[WK + 1][0] = c1;
    e[WK + 1][1] = s1;
    e[WK - 1][0] = c1;
    e[WK - 1][1] = -s1;
    e[WK + 2][0] = c2;
    e[WK + 2][1] = s2;
    e[WK - 2][0] = c2;
    e[WK - 2][1] = -s2;
}

__device__ __forceinline__ void twiddles(int x, int L, double e[2 * WK + 1][2]) {
    double s1, c1;
    sincospi(2.0 * x / L, &s1, &c1);
    powers(c1, s1, e);
}

// The periodic correction Re sum_m c_m exp(i k_m . x) at the nodes of one
// tile, an axis at a time (row_coefs, called by every thread of the
// work-group): for each plane z the tile touches, Z[a][b][k] = sum over n_z of
// c_(a, b, n_z)[k] exp(i kz z); for each of its rows (y, z), R[a][k] = sum over
// n_y of Z[a][b][k] exp(i ky y); then a node's correction is
// Re sum_a R[a][k] exp(i kx x).  The corrected field is real, so the
// coefficients of -n are the conjugates of those of n: a = 0..WK only, the terms
// a > 0 counted twice.  c: the box's WM x MC coefficients (slots outside the
// box's mode set hold 0).  5 + 5 products for each of 12 row coefficients
// (25 for each of 20 when both axes were summed at once over all a).
// The work-group's LDS is sized for the launch's boxes (plane_doubles for each plane
// and row_doubles for each row a tile can touch), so that it does not bound
// how many work-groups a compute unit holds.
constexpr int PLANE_DOUBLES = (WK + 1) * (2 * WK + 1) * UF * 2, ROW_DOUBLES = (WK + 1) * UF * 2;
// planes and rows a tile of an nx x ny x nz box can touch
inline int tile_rows(int nx) { return (TILE - 2) / nx + 2; }
inline int tile_planes(int nx, int ny) { return (tile_rows(nx) - 2) / ny + 2; }

// Fills Z (planes of the tile) and R (its rows); returns the tile's first row.
__device__ int row_coefs(const BoxDesc& B, const double* __restrict__ c, int s0, double* Z, double* R) {
    const int tid = threadIdx.x, nt = blockDim.x;
    const int row0 = s0 / B.nx, row1 = (min(s0 + TILE, B.n) - 1) / B.nx;
    const int z0 = row0 / B.ny, nplanes = row1 / B.ny - z0 + 1, nrows = row1 - row0 + 1;
    constexpr int NB = 2 * WK + 1, PER_Z = PLANE_DOUBLES / 2, PER_ROW = ROW_DOUBLES / 2;
    for (int t = tid; t < nplanes * PER_Z; t += nt) {  // item (plane, a, b, k)
        const int zi = t / PER_Z, a = (t / (NB * UF)) % (WK + 1), b = (t / UF) % NB, k = t % UF;
        double e[NB][2], re = 0.0, im = 0.0;
        twiddles(z0 + zi, B.nz, e);
#pragma unroll
        for (int iz = 0; iz < NB; ++iz) {
            const double* cm = c + MC * ((WK + a) + NB * (b + NB * iz)) + 2 * k;
            re += cm[0] * e[iz][0] - cm[1] * e[iz][1];
            im += cm[0] * e[iz][1] + cm[1] * e[iz][0];
        }
        Z[2 * t] = re;
        Z[2 * t + 1] = im;
    }
    __syncthreads();
    for (int t = tid; t < nrows * PER_ROW; t += nt) {  // item (row, a, k)
        const int r = t / PER_ROW, a = (t / UF) % (WK + 1), k = t % UF, row = row0 + r, zi = row / B.ny - z0;
        double e[NB][2], re = 0.0, im = 0.0;
        twiddles(row % B.ny, B.ny, e);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const double* zz = Z + 2 * (((zi * (WK + 1) + a) * NB + b) * UF + k);
            re += zz[0] * e[b][0] - zz[1] * e[b][1];
            im += zz[0] * e[b][1] + zz[1] * e[b][0];
        }
        R[2 * t] = a ? 2.0 * re : re;
        R[2 * t + 1] = a ? 2.0 * im : im;
    }
    __syncthreads();
    return row0;
}

__device__ __forceinline__ double wave_sum(double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// The wave's sums of eight values, value (lane >> 3) returned to each lane: the
// lanes share out the values at the first three levels (10 exchanges; wave_sum
// of each takes 48), the additions are wave_sum's.
__device__ __forceinline__ double wave_sum8(const double (&v)[8], int lane) {
    double a[4], b[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool up = lane & 32;
        a[k] = (up ? v[k + 4] : v[k]) + __shfl_xor(up ? v[k] : v[k + 4], 32);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const bool up = lane & 16;
        b[k] = (up ? a[k + 2] : a[k]) + __shfl_xor(up ? a[k] : a[k + 2], 16);
    }
    const bool up = lane & 8;
    double w = (up ? b[1] : b[0]) + __shfl_xor(up ? b[0] : b[1], 8);
    for (int off = 4; off > 0; off >>= 1) w += __shfl_xor(w, off);
    return w;
}

// Discrete Fourier sums S_n = sum_x (u, p)_free(x) exp(-i k_n . x), |n_i| <= WK,
// over the planes z = slab, slab + nslab, ... of a box, an axis at a time (the
// field is real, so n_y >= 0 suffices: the others are conjugates).  Along y:
// a thread keeps one x and sums its rows of the plane for n_y = 0..WK (20 sums,
// 20 multiply-adds per node; consecutive threads read consecutive nodes).
// Along x: 60 outputs (n_x, n_y, component) from those sums in LDS, four threads to
// an output.  Along z: the plane's outputs times exp(-i kz z) for the five n_z,
// kept in registers over the slab's planes.  The field is read once, about 60
// operations a node; a work-group per (n_y, n_z) pair read it 25 times over and
// spent 400 a node in all.  Bound by the chain of a plane's four phases; three
// work-groups fit a compute unit (LDS, registers: a fourth would need less of
// both).  One 96^3 box 1500 -> 22 us (25 -> 96 work-groups), 64 boxes of edges
// 32-64 (7.7 M nodes) 1108 -> 84 us (165 with a serial x sum over one bank and
// slabs twice and four times the size, the last of which ran on few compute
// units).
constexpr int YT = 128;  // rows of the phase table held in LDS at a time
__global__ __launch_bounds__(256) void k_stokes_modes(const BoxDesc* __restrict__ boxes,
                                                      const int* __restrict__ slab_box,
                                                      const double* __restrict__ uf, long long base, int only_box,
                                                      double* __restrict__ S) {
    __shared__ double Bs[(2 * WK + 1) * UF][257];  // odd rows: the x sum reads a column of them
    __shared__ double ty[YT][4], tx[256][4];  // (cos, sin) of n = 1 and of n = 2
    const int bi = slab_box[blockIdx.x], tid = threadIdx.x;
    if (only_box >= 0 && bi != only_box) return;  // uniform over the block
    const BoxDesc& B = boxes[bi];
    const int slab = (int)blockIdx.x - B.slab0;
    const int nx = B.nx, ny = B.ny, nz = B.nz;
    auto phase = [](double (&t)[4], int i, int n) {
        double c, s;
        sincospi(2.0 * i / n, &s, &c);
        t[0] = c;
        t[1] = s;
        t[2] = c * c - s * s;
        t[3] = 2.0 * s * c;
    };
    const int o = tid % MODE_HALF, seg = tid / MODE_HALF;  // output and its share of the x sum
    const int ok = o % UF, oy = (o / UF) % (WK + 1), ox = o / (UF * (WK + 1)) - WK;
    constexpr int NSEG = 256 / MODE_HALF;
    double Zr[2 * WK + 1], Zi[2 * WK + 1];
#pragma unroll
    for (int k = 0; k < 2 * WK + 1; ++k) Zr[k] = Zi[k] = 0.0;
    for (int z = slab; z < nz; z += B.nslab) {
        double pr = 0.0, pi = 0.0;
        for (int x0 = 0; x0 < nx; x0 += 256) {
            const int cw = min(256, nx - x0), ng = 256 / cw, g = tid / cw, x = x0 + tid % cw;
            if (tid < cw && (nx > 256 || z == slab)) phase(tx[tid], x0 + tid, nx);
            double acc[UF][2 * WK + 1];
#pragma unroll
            for (int k = 0; k < UF; ++k)
#pragma unroll
                for (int j = 0; j < 2 * WK + 1; ++j) acc[k][j] = 0.0;
            for (int y0 = 0; y0 < ny; y0 += YT) {
                const int y1 = min(ny, y0 + YT);
                if (ny > YT || (x0 == 0 && z == slab)) {
                    __syncthreads();
                    if (tid < y1 - y0) phase(ty[tid], y0 + tid, ny);
                    __syncthreads();
                }
                if (g < ng) {
                    const double* row = uf + UF * (B.ooff + x + (long long)nx * ny * z - base);
#pragma unroll 8
                    for (int y = y0 + g; y < y1; y += ng) {
                        const double2* q = reinterpret_cast<const double2*>(row + (long long)UF * nx * y);
                        const double2 q0 = q[0], q1 = q[1];
                        const double u[UF] = {q0.x, q0.y, q1.x, q1.y};
                        const double* e = ty[y - y0];
#pragma unroll
                        for (int k = 0; k < UF; ++k) {
                            acc[k][0] += u[k];
#pragma unroll
                            for (int j = 0; j < WK; ++j) {
                                acc[k][1 + 2 * j] += u[k] * e[2 * j];
                                acc[k][2 + 2 * j] -= u[k] * e[2 * j + 1];
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < UF; ++k)
#pragma unroll
                for (int j = 0; j < 2 * WK + 1; ++j) Bs[k * (2 * WK + 1) + j][tid] = acc[k][j];
            __syncthreads();
            if (ng > 1) {  // the thread groups' sums of each x, into the first group's place
                for (int i = tid; i < (2 * WK + 1) * UF * cw; i += 256) {
                    const int j = i / cw, xx = i % cw;
                    double v = Bs[j][xx];
#pragma unroll 4
                    for (int h = 1; h < ng; ++h) v += Bs[j][h * cw + xx];
                    Bs[j][xx] = v;
                }
                __syncthreads();
            }
            if (seg < NSEG) {
                const double* br = Bs[ok * (2 * WK + 1) + (oy ? 2 * oy - 1 : 0)];
                const double* bm = Bs[ok * (2 * WK + 1) + (oy ? 2 * oy : 0)];
                const double* tn = &tx[0][ox ? 2 * abs(ox) - 2 : 0];
                // n_x = 0: (1, 0) for (c, sn); n_y = 0: no imaginary sum
                const double cf = ox ? 1.0 : 0.0, sf = ox < 0 ? -1.0 : cf, mf = oy ? 1.0 : 0.0;
#pragma unroll 4
                for (int xx = seg; xx < cw; xx += NSEG) {
                    const double c = cf * tn[4 * xx] + (1.0 - cf), sn = sf * tn[4 * xx + 1], r = br[xx], m = mf * bm[xx];
                    pr += r * c + m * sn;  // (r + i m) (c - i sn)
                    pi += m * c - r * sn;
                }
            }
            __syncthreads();
        }
        double e[2 * WK + 1][2];
        twiddles(z, nz, e);
#pragma unroll
        for (int k = 0; k < 2 * WK + 1; ++k) {  // exp(-i kz z)
            Zr[k] += pr * e[k][0] + pi * e[k][1];
            Zi[k] += pi * e[k][0] - pr * e[k][1];
        }
    }
    double* red = &Bs[0][0];  // NSEG x SLAB
    if (seg < NSEG)
#pragma unroll
        for (int k = 0; k < 2 * WK + 1; ++k) {
            red[seg * SLAB + (o * (2 * WK + 1) + k) * 2] = Zr[k];
            red[seg * SLAB + (o * (2 * WK + 1) + k) * 2 + 1] = Zi[k];
        }
    __syncthreads();
    for (int i = tid; i < SLAB; i += 256) {
        double v = red[i];
        for (int h = 1; h < NSEG; ++h) v += red[h * SLAB + i];
        S[(long long)(B.slab0 + slab) * SLAB + i] = v;
    }
}
static_assert((256 / MODE_HALF) * SLAB <= (2 * WK + 1) * UF * 256, "the slab's sums are reduced in the place of Bs");

// Correction coefficients, a work-group per box and a thread per mode slot:
// the periodic solution's coefficient of every loaded particle of the box
// minus the free flow's DFT coefficient S_m / N (its slabs summed in order);
// zero for slots outside the box's mode set.  The pressure's is -i (k.f) / k^2
// of the force density f (the torque's has no divergence and drives none).
__global__ __launch_bounds__(128) void k_stokes_coef(const BoxDesc* __restrict__ boxes,
                                                     const PartDev* __restrict__ parts,
                                                     const int* __restrict__ pbox, int np, double mu, int only_box,
                                                     const double* __restrict__ S, double* __restrict__ C) {
    __shared__ int list[128];
    __shared__ int wcnt[2];
    const int bi = blockIdx.x, m = threadIdx.x, lane = m & 63, wv = m >> 6;
    if (only_box >= 0 && bi != only_box) return;  // uniform over the block
    const BoxDesc& B = boxes[bi];
    const int n[3] = {m % (2 * WK + 1) - WK, (m / (2 * WK + 1)) % (2 * WK + 1) - WK, m / ((2 * WK + 1) * (2 * WK + 1)) - WK};
    const int L[3] = {B.nx, B.ny, B.nz};
    bool use = m < WM && !(n[0] == 0 && n[1] == 0 && n[2] == 0);
    for (int a = 0; a < 3; ++a) use = use && abs(n[a]) <= wk_axis(L[a]);
    double c[MC] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const double V = (double)B.n;
    double k[3];
    for (int a = 0; a < 3; ++a) k[a] = 2.0 * M_PI * n[a] / L[a];
    const double k2 = k[0] * k[0] + k[1] * k[1] + k[2] * k[2];
    for (int p0 = 0; p0 < np; p0 += 128) {
      const int pt = p0 + m;
      const bool take = pt < np && pbox[pt] == bi;
      const unsigned long long bal = __ballot(take);
      if (lane == 0) wcnt[wv] = __popcll(bal);
      __syncthreads();
      if (take) list[(wv ? wcnt[0] : 0) + __popcll(bal & ((1ull << lane) - 1ull))] = pt;
      __syncthreads();
      const int cnt = use ? wcnt[0] + wcnt[1] : 0;
      for (int j = 0; j < cnt; ++j) {
        const PartDev& P = parts[list[j]];
        // The traction of a body in rigid motion is sigma(x) (F + C x), sigma
        // the unit sphere's uniform layer mapped onto the surface: for an
        // ellipsoid (diag(a, b, c) in the body frame) its transform is
        // F sinc(kappa) - 3 i (Q^T k) j1(kappa) / kappa, kappa = |diag(a, b, c)
        // R^T k|, Q = integral of x f^T the first moment: the torque's
        // antisymmetric part, Q^T k = -(k x T) / 2, and for a prolate spheroid
        // the line solution's stresslet e^2 / (2 - e^2) sym(p (T_c x p)).
        // The force is spread on every ellipsoid so; the torque on the
        // prolate spheroid so and on any other body over the sphere of
        // radius Req (kappa = |k| Req, no stresslet).
        double Rm[3][3];
        body_to_lab(P.q, Rm);
        double ka2 = 0.0;
        for (int j = 0; j < 3; ++j) {
            const double kb = (k[0] * Rm[0][j] + k[1] * Rm[1][j] + k[2] * Rm[2][j]) * P.axes[j];
            ka2 += kb * kb;
        }
        const double xa = sqrt(ka2), sinc = sin(xa) / xa;
        const double kF = k[0] * P.Fext[0] + k[1] * P.Fext[1] + k[2] * P.Fext[2];
        double g[3] = {-0.5 * (k[1] * P.Text[2] - k[2] * P.Text[1]), -0.5 * (k[2] * P.Text[0] - k[0] * P.Text[2]),
                       -0.5 * (k[0] * P.Text[1] - k[1] * P.Text[0])};  // Q^T k
        const double a_ = P.axes[0], b_ = P.axes[1];
        const double e2 = a_ > b_ && b_ == P.axes[2] ? 1.0 - (b_ / a_) * (b_ / a_) : 0.0;
        double xk = sqrt(k2) * eq_radius(P);
        if (e2 >= E_LINE * E_LINE) {
            const double p[3] = {Rm[0][0], Rm[1][0], Rm[2][0]};
            const double Tp = P.Text[0] * p[0] + P.Text[1] * p[1] + P.Text[2] * p[2];
            const double Tc[3] = {P.Text[0] - Tp * p[0], P.Text[1] - Tp * p[1], P.Text[2] - Tp * p[2]};
            const double m[3] = {Tc[1] * p[2] - Tc[2] * p[1], Tc[2] * p[0] - Tc[0] * p[2], Tc[0] * p[1] - Tc[1] * p[0]};
            const double cs = 0.5 * e2 / (2.0 - e2);
            const double km = k[0] * m[0] + k[1] * m[1] + k[2] * m[2], kp = k[0] * p[0] + k[1] * p[1] + k[2] * p[2];
            for (int j = 0; j < 3; ++j) g[j] += cs * (km * p[j] + kp * m[j]);
            xk = xa;
        }
        const double j1k = (sin(xk) - xk * cos(xk)) / (xk * xk * xk);  // j1(kappa) / kappa
        const double kg = k[0] * g[0] + k[1] * g[1] + k[2] * g[2];
        double sp, cp;
        sincos(-(k[0] * P.xc[0] + k[1] * P.xc[1] + k[2] * P.xc[2]), &sp, &cp);  // exp(-i k . x_c)
        for (int a = 0; a < 3; ++a) {
            // u_hat / V = (I - k k / k^2) f_hat / (mu k^2 V), f_hat = F sinc - 3 i g j1k
            const double re = (P.Fext[a] - k[a] * kF / k2) * sinc / (mu * k2) / V;
            const double im = -3.0 * (g[a] - k[a] * kg / k2) * j1k / (mu * k2) / V;
            c[2 * a] += re * cp - im * sp;
            c[2 * a + 1] += re * sp + im * cp;
        }
        // p_hat / V = -i (k . f_hat) / (k^2 V) = pre + i pim
        const double pre = -3.0 * kg * j1k / k2 / V, pim = -kF * sinc / k2 / V;
        c[6] += pre * cp - pim * sp;
        c[7] += pre * sp + pim * cp;
      }
      __syncthreads();
    }
    if (use) {
        // the slab sums hold n_y >= 0; a slot below it is the conjugate of -n
        const int sg = n[1] < 0 ? -1 : 1;
        const int o = ((sg * n[0] + WK) * (WK + 1) + sg * n[1]) * UF, iz = sg * n[2] + WK;
        double d[MC] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int h = 0; h < B.nslab; ++h) {
            const double* q = S + (long long)(B.slab0 + h) * SLAB;
#pragma unroll
            for (int a = 0; a < UF; ++a) {
                d[2 * a] += q[((o + a) * (2 * WK + 1) + iz) * 2];
                d[2 * a + 1] += q[((o + a) * (2 * WK + 1) + iz) * 2 + 1];
            }
        }
#pragma unroll
        for (int a = 0; a < UF; ++a) {
            c[2 * a] -= d[2 * a] / V;
            c[2 * a + 1] -= sg * d[2 * a + 1] / V;
        }
    }
    if (m < WM)
        for (int a = 0; a < MC; ++a) C[((long long)bi * WM + m) * MC + a] = c[a];
}

// The periodic correction added to the staged field at every fluid node, in
// place, and the tile's partial sums over its fluid nodes: of u (3), of p u
// (3), of p and the count.  Writing the corrected field back costs 32 bytes a
// node and spares k_stokes_write the correction.  Bound by the rows' coefficients
// and the sums beside 66 bytes a node: 64 boxes, 7.7 M nodes, 143 us (82 at the
// copy rate; 411 with the correction unfactored, 197 with the node loaded after
// the coefficients and a full exchange for each of the eight sums).
__global__ __launch_bounds__(TILE) void k_stokes_sum(const BoxDesc* __restrict__ boxes,
                                                     const int* __restrict__ tile_box,
                                                     const uint16_t* __restrict__ omap,
                                                     double* __restrict__ uf, long long base, int only_box,
                                                     const double* __restrict__ coef, int planes,
                                                     double* __restrict__ partial) {
    extern __shared__ double zr[];  // planes x PLANE_DOUBLES, then the rows
    __shared__ double red[TILE / 64][NPART];
    double *Z = zr, *R = zr + planes * PLANE_DOUBLES;
    const int tile = blockIdx.x, tid = threadIdx.x;
    const int bi = tile_box[tile];
    const BoxDesc& B = boxes[bi];
    const int s = (tile - B.tile0) * TILE + tid;
    double v[NPART] = {0, 0, 0, 0, 0, 0, 0, 0};
    const bool started = only_box < 0 || bi == only_box;  // uniform over the block
    int row0 = 0;
    // the node's loads are under way while the rows' coefficients are formed
    double2* o = reinterpret_cast<double2*>(uf + UF * (B.ooff + s - base));
    double2 q0 = {0.0, 0.0}, q1 = {0.0, 0.0};
    uint16_t owner = 0xFFFF;
    if (started && s < B.n) {
        owner = omap[B.ooff + s];
        q0 = o[0];
        q1 = o[1];
    }
    if (started) row0 = row_coefs(B, coef + (long long)bi * WM * MC, (tile - B.tile0) * TILE, Z, R);
    if (owner == 0) {
        double u[UF] = {q0.x, q0.y, q1.x, q1.y};
        int x;
        const int row = div_magic(s, B.nx, B.mnx, B.lnx, x);
        const double* Rr = R + (row - row0) * ROW_DOUBLES;  // [a][k] (re, im)
        double ex[2 * WK + 1][2];
        twiddles(x, B.nx, ex);
#pragma unroll
        for (int k = 0; k < UF; ++k) {
            u[k] += Rr[2 * k];
#pragma unroll
            for (int a = 1; a <= WK; ++a)
                u[k] += Rr[2 * (a * UF + k)] * ex[WK + a][0] - Rr[2 * (a * UF + k) + 1] * ex[WK + a][1];
        }
        o[0] = double2{u[0], u[1]};
        o[1] = double2{u[2], u[3]};
        for (int k = 0; k < 3; ++k) {
            v[k] = u[k];
            v[3 + k] = u[3] * u[k];
        }
        v[6] = u[3];
        v[7] = 1.0;
    }
    const double w8 = wave_sum8(v, tid & 63);
    if ((tid & 7) == 0) red[tid >> 6][(tid >> 3) & 7] = w8;
    __syncthreads();
    if (tid < NPART) {
        double w = 0.0;
        for (int h = 0; h < TILE / 64; ++h) w += red[h][tid];
        partial[(long long)tile * NPART + tid] = w;
    }
}

// A work-group per box: the mean pressure pbar of its fluid nodes and the
// uniform velocity ubar removed from them.  A fluid node gets the density
// rho = rho0 + 3 (p - pbar) (p = c_s^2 (rho - rho0)), so the fluid's mass is
// unchanged, and ubar = (sum rho u + sum_p M U) / (N rho0) makes the box's
// momentum sum rho (u - ubar) + sum_p M U zero.
__global__ __launch_bounds__(256) void k_stokes_mean(const BoxDesc* __restrict__ boxes,
                                                    const PartDev* __restrict__ parts, int np,
                                                    const double* __restrict__ partial, double rho0,
                                                    double* __restrict__ ubar) {
    __shared__ double red[4][NPART + 3];
    const int b = blockIdx.x, tid = threadIdx.x;
    const BoxDesc& B = boxes[b];
    double S[NPART] = {0, 0, 0, 0, 0, 0, 0, 0}, MU[3] = {0, 0, 0};
    for (int t = B.tile0 + tid; t < B.tile0 + B.ntiles; t += 256)
        for (int k = 0; k < NPART; ++k) S[k] += partial[(long long)t * NPART + k];
    for (int p = tid; p < np; p += 256)
        if (parts[p].box == b)
            for (int k = 0; k < 3; ++k) MU[k] += parts[p].M * parts[p].U[k];
#pragma unroll
    for (int k = 0; k < NPART + 3; ++k) {
        const double v = wave_sum(k < NPART ? S[k] : MU[k - NPART]);
        if ((tid & 63) == 0) red[tid >> 6][k] = v;
    }
    __syncthreads();
    if (tid != 0) return;
    for (int k = 0; k < NPART; ++k) S[k] = (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
    for (int k = 0; k < 3; ++k) MU[k] = (red[0][NPART + k] + red[1][NPART + k]) + (red[2][NPART + k] + red[3][NPART + k]);
    const double N = S[7], pbar = N > 0 ? S[6] / N : 0.0;
    double J[3];
    for (int k = 0; k < 3; ++k) J[k] = rho0 * S[k] + 3.0 * (S[3 + k] - pbar * S[k]) + MU[k];
    for (int k = 0; k < 3; ++k) ubar[4 * b + k] = N > 0 ? J[k] / (N * rho0) : 0.0;
    ubar[4 * b + 3] = pbar;
}

// Bound by memory (a staged node read, Q populations written: in FP16 70 bytes
// a node, 64 boxes 123 us, 86 at the copy rate, 463 with the correction here
// too); the storage convention is a template parameter so that a slot costs an
// addition, and the two directions of a pair share their products.
template <int ST, int Q, int CV>
__global__ __launch_bounds__(TILE) void k_stokes_write(const BoxDesc* __restrict__ boxes,
                                                       const int* __restrict__ tile_box,
                                                       const uint16_t* __restrict__ omap,
                                                       const PartDev* __restrict__ parts,
                                                       const double* __restrict__ uf, long long base,
                                                       const double* __restrict__ ubar,
                                                       typename Store<ST>::T* __restrict__ f, KParams kp,
                                                       int only_box) {
    using S = Store<ST>;
    const int tile = blockIdx.x;
    const int bi = tile_box[tile];
    if (only_box >= 0 && bi != only_box) return;  // uniform over the block
    const BoxDesc& B = boxes[bi];
    const int s = (tile - B.tile0) * TILE + (int)threadIdx.x;
    if (s >= B.n) return;
    // the staged node comes with its owner, not after it
    const double2* o = reinterpret_cast<const double2*>(uf + UF * (B.ooff + s - base));
    const double2 q0 = o[0], q1 = o[1];
    const uint16_t owner = omap[B.ooff + s];
    if (owner == 0xFFFF) return;
    const int nx = B.nx, ny = B.ny, nz = B.nz;
    int x, y;
    const int z = div_magic(div_magic(s, nx, B.mnx, B.lnx, x), ny, B.mny, B.lny, y);
    const double rho0 = kp.rho0;
    double rho = rho0, u[3];
    if (owner == 0) {
        u[0] = q0.x - ubar[4 * bi];
        u[1] = q0.y - ubar[4 * bi + 1];
        u[2] = q1.x - ubar[4 * bi + 2];
        rho = rho0 + 3.0 * (q1.y - ubar[4 * bi + 3]);
    } else {  // rigid motion at the rest density inside a particle
        const PartDev& P = parts[owner - 1];
        double d[3];
        offset(P.xc, B, x, y, z, d);
        u[0] = P.U[0] + P.W[1] * d[2] - P.W[2] * d[1];
        u[1] = P.U[1] + P.W[2] * d[0] - P.W[0] * d[2];
        u[2] = P.U[2] + P.W[0] * d[1] - P.W[1] * d[0];
    }
    const double e0 = (rho - rho0) - 1.5 * rho * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
    // site offsets of the neighbours at +1 and -1 along each axis
    const int dx[2] = {x == nx - 1 ? 1 - nx : 1, x == 0 ? nx - 1 : -1};
    const int dy[2] = {(y == ny - 1 ? 1 - ny : 1) * nx, (y == 0 ? ny - 1 : -1) * nx};
    const int dz[2] = {(z == nz - 1 ? 1 - nz : 1) * nx * ny, (z == 0 ? nz - 1 : -1) * nx * ny};
    typename S::T* fb = f + B.foff;
    auto put = [&](int i, double dev) {
        // the slot this node reads f_i from at the next step (no walls here)
        const int to = CV == CV_ODD ? 0 : (cx(i) ? dx[cx(i) > 0] : 0) + (cy(i) ? dy[cy(i) > 0] : 0) +
                                              (cz(i) ? dz[cz(i) > 0] : 0);
        S::st64(fb + (long long)(CV == CV_EVEN ? opp(i) : i) * B.stride + (s + to), dev, kp.scale);
    };
    put(0, wgt<Q>(0) * e0);
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const double cu = cx(i) * u[0] + cy(i) * u[1] + cz(i) * u[2];
        const double ev = wgt<Q>(i) * (e0 + 4.5 * rho * cu * cu), od = wgt<Q>(i) * (3.0 * rho * cu);
        put(i, ev + od);
        put(i + 1, ev - od);
    }
}

// ---------------------------------------------------------------------------
// Fallback monitor of warm-started boxes, one work-group per box, run every
// monitor period.  W0, the viscous time 2 a^2 / nu of the box's largest
// particle (a its largest semi-axis), is the time in which a particle sheds
// the error of its start.  The first check at least Wref = W0 / 4 steps after
// the warm start takes the reference: the flow energy E = sum |j|^2 over the
// box's fluid and every particle's V = (U, a Omega).  The first check at
// least W0 steps after it decides from the residuals (the relative changes
// since the reference: |E - E_ref| / (2 E), E being quadratic in the velocity,
// and the largest |V - V_ref| / |V| over the box's particles) and the
// prediction.  The box misses when more than a quarter of its particles
// (MON_MISS_SHARE) are further than tol from their predictions: a lone
// particle on its own miss, while in a crowded box the interactions can
// carry a few particles away from any one-particle prediction without the
// start being wrong.
//   no miss   accepted;
//   a miss while a residual exceeds tol (the run moves away from the
//     prediction)   fallback: the box restarts from the plain start (fluid and
//     particles at rest, pending transition book-keeping dropped), its steps
//     so far spent;
//   a miss with both residuals below tol (the run has settled elsewhere)
//     kept, its sample to be added to the training data.
constexpr double MON_MISS_SHARE = 0.25;
__global__ __launch_bounds__(256) void k_warm_monitor(const BoxDesc* __restrict__ boxes, BoxMon* __restrict__ mon,
                                                      const double* __restrict__ partial, PartDev* __restrict__ parts,
                                                      int np, const double* __restrict__ pred,
                                                      double* __restrict__ vref, long long step) {
    const int b = blockIdx.x, tid = threadIdx.x;
    BoxMon& M = mon[b];
    __shared__ double red[4][4];
    __shared__ int phase;  // 0 nothing, 1 take the reference, 2 decide
    __shared__ int decide;
    if (M.status != MON_PENDING) {
        if (tid == 0) M.reset = 0;
        return;
    }
    if (tid == 0) {
        const long long age = step - M.t0;
        phase = M.t_ref < 0 ? (age >= M.Wref ? 1 : 0) : (age >= M.W0 && step > M.t_ref ? 2 : 0);
        M.reset = 0;
    }
    __syncthreads();
    if (phase == 0) return;  // uniform over the block
    const BoxDesc& B = boxes[b];
    // the box's flow energy, tile partials summed in a fixed order
    double e = 0.0;
    for (int t = B.tile0 + tid; t < B.tile0 + B.ntiles; t += blockDim.x) e += partial[t];
    // the box's particles: the largest relative change since the reference,
    // and how many of them miss their prediction
    double dv = 0.0, miss = 0.0, cnt = 0.0;
    for (int p = tid; p < np; p += blockDim.x) {
        const PartDev& P = parts[p];
        if (P.box != b) continue;
        const double a = fmax(P.axes[0], fmax(P.axes[1], P.axes[2]));
        const double V[6] = {P.U[0], P.U[1], P.U[2], a * P.W[0], a * P.W[1], a * P.W[2]};
        double* vr = vref + 6 * (long long)p;
        const double* pr = pred + 6 * (long long)p;
        if (phase == 1) {
            for (int k = 0; k < 6; ++k) vr[k] = V[k];
            continue;
        }
        double d2 = 0, v2 = 0, m2 = 0, p2 = 0;
        for (int k = 0; k < 6; ++k) {
            const double pk = k < 3 ? pr[k] : a * pr[k];
            d2 += (V[k] - vr[k]) * (V[k] - vr[k]);
            v2 += V[k] * V[k];
            m2 += (V[k] - pk) * (V[k] - pk);
            p2 += pk * pk;
        }
        dv = fmax(dv, v2 > 0 ? sqrt(d2 / v2) : 0.0);
        if (m2 > M.tol * M.tol * p2) miss += 1.0;
        cnt += 1.0;
    }
    for (int o = 32; o > 0; o >>= 1) {
        e += __shfl_xor(e, o);
        dv = fmax(dv, __shfl_xor(dv, o));
        miss += __shfl_xor(miss, o);
        cnt += __shfl_xor(cnt, o);
    }
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = e;
        red[1][tid >> 6] = dv;
        red[2][tid >> 6] = miss;
        red[3][tid >> 6] = cnt;
    }
    __syncthreads();
    if (tid == 0) {
        double E = 0, DV = 0, MISS = 0, N = 0;
        for (int k = 0; k < 4; ++k) {
            E += red[0][k];
            DV = fmax(DV, red[1][k]);
            MISS += red[2][k];
            N += red[3][k];
        }
        int dec = 0;
        if (phase == 1) {
            M.E_ref = E;
            M.t_ref = step;
        } else {
            M.res_flow = E > 0 ? 0.5 * fabs(E - M.E_ref) / E : 0.0;
            M.res_part = DV;
            const bool conv = M.res_flow < M.tol && M.res_part < M.tol;
            dec = MISS <= MON_MISS_SHARE * N ? MON_ACCEPTED : (conv ? MON_STEADY_MISS : MON_FALLBACK);
            M.status = dec;
            M.t_decided = step;
        }
        M.reset = dec == MON_FALLBACK ? 1 : 0;
        decide = dec;
    }
    __syncthreads();
    if (decide != MON_FALLBACK) return;
    for (int p = tid; p < np; p += blockDim.x) {  // the box's particles to rest
        PartDev& P = parts[p];
        if (P.box != b) continue;
        for (int k = 0; k < 3; ++k) {
            P.U[k] = P.W[k] = 0.0;
            P.Pp[k] = P.Lp[k] = 0.0;
        }
        P.dm = 0.0;
    }
}

// Every population slot of a box whose check fell back is set to rest
// (deviation 0 in every storage format and layout).
template <typename T>
__global__ __launch_bounds__(TILE) void k_box_reset(const BoxDesc* __restrict__ boxes, const int* __restrict__ tile_box,
                                                    const BoxMon* __restrict__ mon, T* __restrict__ f, int q) {
    const int tile = blockIdx.x;
    const int bi = tile_box[tile];
    if (!mon[bi].reset) return;
    const BoxDesc& B = boxes[bi];
    const int s = (tile - B.tile0) * TILE + (int)threadIdx.x;
    if (s >= B.n) return;
    for (int i = 0; i < q; ++i) f[B.foff + (long long)i * B.stride + s] = T(0);
}

hipError_t launch_warm_monitor(const BoxDesc* boxes, int nboxes, const int* tile_box, int ntiles, BoxMon* mon,
                               const double* partial, PartDev* parts, int np, const double* pred, double* vref,
                               long long step, void* f, int storage, int q, hipStream_t st) {
    hipLaunchKernelGGL(k_warm_monitor, dim3(nboxes), dim3(256), 0, st, boxes, mon, partial, parts, np, pred, vref,
                       step);
    const int es = storage_bytes(storage);
    if (es == 8)
        hipLaunchKernelGGL((k_box_reset<unsigned long long>), dim3(ntiles), dim3(TILE), 0, st, boxes, tile_box, mon,
                           (unsigned long long*)f, q);
    else if (es == 4)
        hipLaunchKernelGGL((k_box_reset<uint32_t>), dim3(ntiles), dim3(TILE), 0, st, boxes, tile_box, mon,
                           (uint32_t*)f, q);
    else
        hipLaunchKernelGGL((k_box_reset<uint16_t>), dim3(ntiles), dim3(TILE), 0, st, boxes, tile_box, mon,
                           (uint16_t*)f, q);
    return hipGetLastError();
}

hipError_t launch_warm_features(const BoxDesc* boxes, const PartDev* parts, int np, double mu, float* X, double* s,
                                hipStream_t st) {
    if (np <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_warm_features, dim3((np + 63) / 64), dim3(64), 0, st, boxes, parts, np, mu, X, s);
    return hipGetLastError();
}

hipError_t launch_warm_apply(PartDev* parts, int np, const float* Y, const double* s, double mu, double* pred,
                             int only_box, hipStream_t st) {
    if (np <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_warm_apply, dim3((np + 63) / 64), dim3(64), 0, st, parts, np, Y, s, mu, pred, only_box);
    return hipGetLastError();
}

hipError_t launch_warm_targets(const PartDev* parts, int np, const double* s, double mu, float* Y, hipStream_t st) {
    if (np <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_warm_targets, dim3((np + 63) / 64), dim3(64), 0, st, parts, np, s, mu, Y);
    return hipGetLastError();
}

// Planes of a box are dealt to slabs of about 2048 nodes (1 to 512 of them, no
// more than planes): enough work-groups for one large box, and for many small
// ones several rounds of them, so that the last is not a large part of the time (64
// boxes, 7.7 M nodes: 165 us with 8192 nodes, 111 with 4096, 84 with
// 2048; a slab's sums are 4.8 KB).  A function of the box alone, so a box's sums do not depend on
// what else is started.
int stokes_slabs(int nx, int ny, int nz) {
    const long long n = (long long)nx * ny * nz;
    return (int)std::max<long long>(1, std::min<long long>(std::min<long long>(nz, 512), n / 2048));
}

void stokes_tile(int nx, int ny, int& rows, int& planes) {
    rows = std::max(rows, tile_rows(nx));
    planes = std::max(planes, tile_planes(nx, ny));
}

namespace {
struct StokesScratch {  // offsets in doubles
    size_t S, C, partial, ubar, fc, pbox, total;
};
StokesScratch stokes_layout(int nboxes, int ntiles, int nslabs, int max_particles) {
    StokesScratch L{};
    size_t at = 0;
    auto take = [&](size_t n) {
        const size_t o = at;
        at += n;
        return o;
    };
    L.S = take((size_t)nslabs * SLAB);
    L.C = take((size_t)nboxes * WM * MC);
    L.partial = take((size_t)ntiles * NPART);
    L.ubar = take(4 * (size_t)nboxes);
    L.fc = take((size_t)max_particles * FLOW_DOUBLES);
    L.pbox = take(((size_t)max_particles + 1) / 2);
    L.total = at;
    return L;
}
}  // namespace

size_t stokes_scratch_doubles(int nboxes, int ntiles, int nslabs, int max_particles) {
    return stokes_layout(nboxes, ntiles, nslabs, max_particles).total;
}
int stokes_free_doubles() { return UF; }

hipError_t launch_stokes_start(const BoxDesc* boxes, int nboxes, const int* tile_box, int ntiles, int nslabs,
                               const int* slab_box, int rows, int planes, int max_particles, const uint16_t* omap,
                               const PartDev* parts, int np, double mu, double* scratch, double* uf, long long base,
                               void* f, const KParams& kp, int only_box, hipStream_t st) {
    const StokesScratch L = stokes_layout(nboxes, ntiles, nslabs, max_particles);
    double *S = scratch + L.S, *C = scratch + L.C, *partial = scratch + L.partial, *ubar = scratch + L.ubar;
    FlowConst* fc = reinterpret_cast<FlowConst*>(scratch + L.fc);
    int* pbox = reinterpret_cast<int*>(scratch + L.pbox);
    if (np > 0)
        hipLaunchKernelGGL(k_stokes_prep, dim3((np + 63) / 64), dim3(64), 0, st, parts, np, mu, fc, pbox);
    hipLaunchKernelGGL(k_stokes_free, dim3(ntiles), dim3(TILE), 0, st, boxes, tile_box, fc, pbox, np, only_box, base,
                       uf);
    hipLaunchKernelGGL(k_stokes_modes, dim3(nslabs), dim3(256), 0, st, boxes, slab_box, uf, base, only_box, S);
    hipLaunchKernelGGL(k_stokes_coef, dim3(nboxes), dim3(128), 0, st, boxes, parts, pbox, np, mu, only_box, S, C);
    hipLaunchKernelGGL(k_stokes_sum, dim3(ntiles), dim3(TILE),
                       sizeof(double) * ((size_t)planes * PLANE_DOUBLES + (size_t)rows * ROW_DOUBLES), st, boxes,
                       tile_box, omap, uf, base, only_box, C, planes, partial);
    hipLaunchKernelGGL(k_stokes_mean, dim3(nboxes), dim3(256), 0, st, boxes, parts, np, partial, kp.rho0, ubar);
    auto write = [&](auto st_, auto q_, auto cv_) {
        constexpr int ST = decltype(st_)::value, Q = decltype(q_)::value, CV = decltype(cv_)::value;
        hipLaunchKernelGGL((k_stokes_write<ST, Q, CV>), dim3(ntiles), dim3(TILE), 0, st, boxes, tile_box, omap, parts,
                           uf, base, ubar, (typename Store<ST>::T*)f, kp, only_box);
    };
    auto by_cv = [&](auto st_, auto q_) {
        if (kp.conv == CV_ODD) write(st_, q_, std::integral_constant<int, CV_ODD>{});
        else if (kp.conv == CV_EVEN) write(st_, q_, std::integral_constant<int, CV_EVEN>{});
        else write(st_, q_, std::integral_constant<int, CV_PULL>{});
    };
    auto by_q = [&](auto st_) {
        if (kp.q == 27) by_cv(st_, std::integral_constant<int, 27>{});
        else by_cv(st_, std::integral_constant<int, 19>{});
    };
    switch (kp.storage) {
        case ST_F64: by_q(std::integral_constant<int, ST_F64>{}); break;
        case ST_F32: by_q(std::integral_constant<int, ST_F32>{}); break;
        case ST_F16: by_q(std::integral_constant<int, ST_F16>{}); break;
        default: by_q(std::integral_constant<int, ST_BF16>{});
    }
    return hipGetLastError();
}

}  // namespace lbd
