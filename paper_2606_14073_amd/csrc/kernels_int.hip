// kernels_int.hip -- the spin-lattice step on the device: velocity and
// position half-steps, the lattice Langevin step, the spin sweep over a fixed
// colouring of the spin carriers, and fixed-order per-replica reductions.
// Positions, velocities, spins and all sums are FP64.
#include "engine.h"

namespace nep {

namespace {

inline int nblk(int n, int b) { return (n + b - 1) / b; }

__global__ void k_kick(Sys S) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S.N) return;
    const RepDev &R = S.rep[S.rid[i]];
    if (!R.active) return;
    const double c = 0.5 * R.dt * KAPPA / R.mass[i < S.N_fe ? 0 : 1];
    d4 v = S.vel[i];
    const d4 f = S.force[i];
    v.x += c * f.x;
    v.y += c * f.y;
    v.z += c * f.z;
    S.vel[i] = v;
}

// The single-precision copy of a position, for the cutoff tests that are not
// close: their error bound takes periodic coordinates to lie in the box, and
// folding them to cost no more than rounding. A coordinate for which that does
// not hold becomes NaN, which leaves its tests undecided.
constexpr double FOLD_MAX = 1.0e7;   // A; beyond it a coordinate's own rounding (1e-9 A) enters the bound
__device__ inline float fold4(const RepDev &R, int a, double x) {
    return !R.pbc[a] || (x >= -1.0 && x <= R.box[a] + 1.0) ? (float)x : __int_as_float(0x7fc00000);
}
__device__ inline float4 pos4_of(const RepDev &R, const d4 &p) {
    return make_float4(fold4(R, 0, p.x), fold4(R, 1, p.y), fold4(R, 2, p.z), 0.0f);
}

__device__ inline void fold(const RepDev &R, d4 &p) {
    if (R.pbc[0]) p.x -= R.box[0] * floor(p.x / R.box[0]);
    if (R.pbc[1]) p.y -= R.box[1] * floor(p.y / R.box[1]);
    if (R.pbc[2]) p.z -= R.box[2] * floor(p.z / R.box[2]);
}

__global__ void k_drift(Sys S) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S.N) return;
    const RepDev &R = S.rep[S.rid[i]];
    if (!R.active) return;
    const double h = 0.5 * R.dt;
    d4 p = S.pos[i];
    const d4 v = S.vel[i];
    p.x += h * v.x;
    p.y += h * v.y;
    p.z += h * v.z;
    fold(R, p);
    S.pos[i] = p;
    S.pos4[i] = pos4_of(R, p);
}

__global__ void k_pos4(Sys S) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S.N) return;
    const RepDev &R = S.rep[S.rid[i]];
    d4 p = S.pos[i];   // the caller's, in any image
    const bool far = fmax(fabs(p.x), fmax(fabs(p.y), fabs(p.z))) > FOLD_MAX && (R.pbc[0] || R.pbc[1] || R.pbc[2]);
    fold(R, p);
    float4 q = pos4_of(R, p);
    if (far) q.x = __int_as_float(0x7fc00000);
    S.pos4[i] = q;
}

__device__ inline double temperature(const RepDev &R) { return R.T0 + (R.T1 - R.T0) * ramp_frac(R); }

__global__ void k_langevin(Sys S) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S.N) return;
    const RepDev &R = S.rep[S.rid[i]];
    if (!R.active || R.ensemble != 1) return;
    const double c1 = exp(-R.gammaL * R.dt);
    const double sig = sqrt((1.0 - c1 * c1) * KAPPA * KB * temperature(R) / R.mass[i < S.N_fe ? 0 : 1]);
    double xi[3];
    gauss3(R.seed, (uint32_t)S.orig[i], (unsigned long long)R.step, 0u, xi);
    d4 v = S.vel[i];
    v.x = c1 * v.x + sig * xi[0];
    v.y = c1 * v.y + sig * xi[1];
    v.z = c1 * v.z + sig * xi[2];
    S.vel[i] = v;
}

// noise field of the step and the reference copies S^n, S_hat
__global__ void k_spin_prep(Sys S) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S.N_fe) return;
    const RepDev &R = S.rep[S.rid[i]];
    if (!R.active) return;
    const double T = temperature(R);
    d4 e = {0, 0, 0, 0};
    if (!R.lsf && R.alpha > 0 && T > 0) {
        const double sig = sqrt(2.0 * R.alpha * KB * T * HBAR / R.dt);
        double xi[3];
        gauss3(R.seed, (uint32_t)S.orig[i], (unsigned long long)R.step, 1u, xi);
        e.x = sig * xi[0];
        e.y = sig * xi[1];
        e.z = sig * xi[2];
    }
    S.eta[i] = e;
    const d4 s = S.spin[i];
    S.spin_n[i] = s;
    S.spin_hat[i] = s;
}

// replicas whose self-consistent iteration has converged keep their spins
__device__ inline bool spin_pass_on(const RepDev &R) { return R.active && !R.sc_done; }

__global__ void k_spin_restore(Sys S) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S.N_fe) return;
    if (!spin_pass_on(S.rep[S.rid[i]])) return;
    S.spin[i] = S.spin_n[i];
}

__global__ void k_spin_mid(Sys S) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S.N_fe) return;
    if (!spin_pass_on(S.rep[S.rid[i]])) return;
    const d4 a = S.spin_n[i], b = S.spin[i];
    const double x = 0.5 * (a.x + b.x), y = 0.5 * (a.y + b.y), z = 0.5 * (a.z + b.z);
    // unit spins: the normalised average; spins of variable length: the average
    const double n = S.rep[S.rid[i]].lsf ? 1.0 : sqrt(x * x + y * y + z * z);
    d4 h = {x / n, y / n, z / n, 0.0};
    S.spin_hat[i] = h;
}

// sin(t) and 1 - cos(t) from their Taylor series (coefficients +-1/n!) through
// t^19 and t^20, for |t| <= 1 where the truncation error is below 1e-19; no
// cancellation in 1 - cos. Both are polynomials of degree 9 in u = t^2,
// evaluated in Estrin's form (pairs, then u^2, u^4, u^8): five dependent
// steps instead of nine, since the midpoint iteration is latency bound.
__device__ inline void sin_omc_taylor(double t, double &sn, double &omc) {
    const double u = t * t, u2 = u * u, u4 = u2 * u2, u8 = u4 * u4;
    // sin(t)/t = sum_k (-1)^k u^k / (2k+1)!
    const double s01 = fma(u, -1.0 / 6.0, 1.0);
    const double s23 = fma(u, -1.0 / 5040.0, 1.0 / 120.0);
    const double s45 = fma(u, -1.0 / 39916800.0, 1.0 / 362880.0);
    const double s67 = fma(u, -1.0 / 1307674368000.0, 1.0 / 6227020800.0);
    const double s89 = fma(u, -1.0 / 121645100408832000.0, 1.0 / 355687428096000.0);
    const double ps = fma(u8, s89, fma(u4, fma(u2, s67, s45), fma(u2, s23, s01)));
    // (1 - cos t)/t^2 = sum_k (-1)^k u^k / (2k+2)!
    const double c01 = fma(u, -1.0 / 24.0, 0.5);
    const double c23 = fma(u, -1.0 / 40320.0, 1.0 / 720.0);
    const double c45 = fma(u, -1.0 / 479001600.0, 1.0 / 3628800.0);
    const double c67 = fma(u, -1.0 / 20922789888000.0, 1.0 / 87178291200.0);
    const double c89 = fma(u, -1.0 / 2432902008176640000.0, 1.0 / 6402373705728000.0);
    const double pc = fma(u8, c89, fma(u4, fma(u2, c67, c45), fma(u2, c23, c01)));
    sn = t * ps;
    omc = u * pc;
}

// 1/sqrt(x) for x > 0 in FP64: the hardware estimate y (relative error e0
// about 5e-8 on gfx950) refined by one third-order step,
// y (1 + e/2 + 3 e^2/8) with e = 1 - x y^2, whose truncation error
// 5 e0^3 / 16 is far below rounding: the result is within 1 ulp.
__device__ inline double rsqrt_nr(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Value of lane K of this lane's quad (lanes 4q..4q+3), by DPP.
template <int K>
__device__ inline double quad_bcast(double v) {
    constexpr int ctrl = K | (K << 2) | (K << 4) | (K << 6);   // quad_perm [K, K, K, K]
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

template <int K>
__device__ inline float quad_bcast(float v) {
    constexpr int ctrl = K | (K << 2) | (K << 4) | (K << 6);
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), ctrl, 0xF, 0xF, false));
}

// Value of the lane that differs in bit M of its number within sixteen, for a
// butterfly sum over M = 1, 2, 4, 8 in turn (DPP; M = 4 and 8 read the mirrored
// lane, which by then holds the same sum).
template <int M>
__device__ inline double row_partner(double v) {
    constexpr int ctrl = M == 1 ? 0xB1 : M == 2 ? 0x4E : M == 4 ? 0x141 : 0x140;   // quad_perm, row_half_mirror, row_mirror
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// One coupling's contribution to the field on a spin: exchange J s_j, DMI
// D s_j x r, anisotropic exchange K (s_j . r) r, subtracted from h, with
// explicit fused multiply-adds and no other contraction.
__device__ inline void coupling_field(double J, double D, double K, double rx, double ry, double rz, double sx,
                                      double sy, double sz, double &hx, double &hy, double &hz) {
#pragma clang fp contract(off)
    const double sr = fma(sz, rz, fma(sy, ry, sx * rx));
    const double ks = K * sr;
    hx -= fma(J, sx, fma(D, fma(sy, rz, -(sz * ry)), ks * rx));
    hy -= fma(J, sy, fma(D, fma(sz, rx, -(sx * rz)), ks * ry));
    hz -= fma(J, sz, fma(D, fma(sx, ry, -(sy * rx)), ks * rz));
}

// The sweep over a colour class: every spin takes an implicit-midpoint
// Rodrigues rotation over tau = dt/2 in the field of its (other-colour)
// neighbours, its own anisotropy/onsite terms at the midpoint, the Zeeman field
// and the noise. L lanes share a spin (L = 4, 8 or 16): they split the neighbour
// gather (couplings stored in colour-list order, so a wavefront reads contiguous
// records), reduce, and then solve the midpoint equation together (each quad
// of lanes evaluates the rotation at four points per Newton step); lane 0
// stores the result.
// The field sum has one order whatever L is: sixteen virtual lanes v each
// add the couplings in slots v, v + 16, v + 32, ... in turn, and a butterfly
// over v (xor 1, 2, 4, 8) adds the sixteen partial sums. Lane l of L carries
// the virtual lanes l + L k, k < 16 / L; the butterfly levels below L run
// across lanes and the others inside the lane. A spin's result thus has the
// same bits with any L, so each launch takes the L that suits the size of its
// colour class (fewer, fuller waves for large classes, more workgroups for small
// ones) and a replica still gives the same bits alone and in any batch.
// The arithmetic is not contracted: the compiler would fuse multiplies and adds
// differently in the instances (their code is scheduled apart), and their
// results would then differ in the last bit; where a fused multiply-add is
// wanted it is written out.
constexpr int SWEEP_V = 16;              // virtual lanes of the field sum
constexpr int SWEEP_WIDE_MIN = 8192;     // classes of at least this many spins take 8 lanes per spin
constexpr int SWEEP_WIDER_MIN = 32768;   // and of at least this many 4
constexpr int SWEEP_LDS_THREADS = 512;   // workgroup of a replica whose spins stay in LDS

// what a visit needs that does not depend on the neighbours' spins: everything
// indexed by the colour-list position p (atom, coupling count, self terms, the
// first 32 coupling slots, read whether or not they are in use and masked
// afterwards), then the atom's noise and spin
template <typename real, int L>
struct SweepSpin {
    static constexpr int P = SWEEP_V / L;   // virtual lanes per lane
    static constexpr int R0 = 2 * P;        // coupling slots per lane loaded up front: u = 2 k + w is lane + L k + 16 w
    int p, i, nc, cj[R0];
    real cv[R0][6], A[7];
    d4 e, s4, sj[R0];
    __device__ void load(const Sys &S, const Work<real> &W, int lane, int p_) {
        p = p_;
        const size_t lf = S.N_fe;
        i = S.col_idx[p];
        nc = W.cpl_n[p];
        const real *o = W.selfc + (size_t)p * 8;
#pragma unroll
        for (int x = 0; x < 7; x++) A[x] = o[x];
#pragma unroll
        for (int u = 0; u < R0; u++) {
            const size_t q = (size_t)(lane + L * (u >> 1) + SWEEP_V * (u & 1)) * lf + p;
            cj[u] = W.cpl_j[q];
            const real *c = W.cpl + q * 6;
#pragma unroll
            for (int x = 0; x < 6; x++) cv[u][x] = c[x];
        }
    }
    __device__ void load_atom(const Sys &S) {
        e = S.eta[i];
        s4 = S.spin[i];
    }
    // the partners' spins of the slots in use; at(j) is spin j
    template <typename At>
    __device__ void load_partners(int lane, At at) {
#pragma unroll
        for (int u = 0; u < R0; u++) sj[u] = at(lane + L * (u >> 1) + SWEEP_V * (u & 1) < nc ? cj[u] : i);
    }
};

// the field of the neighbours on the spin, summed over its lanes; at(j) is spin j
template <typename real, int L, typename At>
__device__ inline void sweep_field(const Sys &S, const Work<real> &W, const SweepSpin<real, L> &q, int lane, At at,
                                   double &hx, double &hy, double &hz) {
#pragma clang fp contract(off)
    constexpr int P = SweepSpin<real, L>::P, R0 = SweepSpin<real, L>::R0;
    const size_t lf = S.N_fe;
    double px[P], py[P], pz[P];
#pragma unroll
    for (int k = 0; k < P; k++) px[k] = py[k] = pz[k] = 0;
#pragma unroll
    for (int u = 0; u < R0; u++) {
        const int k = u >> 1;
        if (lane + L * k + SWEEP_V * (u & 1) >= q.nc) continue;
        coupling_field(q.cv[u][0], q.cv[u][1], q.cv[u][2], q.cv[u][3], q.cv[u][4], q.cv[u][5], q.sj[u].x, q.sj[u].y,
                       q.sj[u].z, px[k], py[k], pz[k]);
    }
    // spins with more than 32 couplings
#pragma unroll
    for (int k = 0; k < P; k++)
        for (int s = lane + L * k + 2 * SWEEP_V; s < q.nc; s += SWEEP_V) {
            const int j = W.cpl_j[(size_t)s * lf + q.p];
            const real *c = W.cpl + ((size_t)s * lf + q.p) * 6;
            const d4 v = at(j);
            coupling_field(c[0], c[1], c[2], c[3], c[4], c[5], v.x, v.y, v.z, px[k], py[k], pz[k]);
        }
    // butterfly: levels 1 .. L/2 across the lanes, then L .. 8 inside them
    static_for<4>([&](auto B) {
        constexpr int m = 1 << decltype(B)::value;
        if constexpr (m < L) {
#pragma unroll
            for (int k = 0; k < P; k++) {
                px[k] += row_partner<m>(px[k]);
                py[k] += row_partner<m>(py[k]);
                pz[k] += row_partner<m>(pz[k]);
            }
        }
    });
#pragma unroll
    for (int b = 1; b < P; b <<= 1)
#pragma unroll
        for (int k = 0; k < P; k += 2 * b) {
            px[k] += px[k + b];
            py[k] += py[k + b];
            pz[k] += pz[k + b];
        }
    hx = px[0];
    hy = py[0];
    hz = pz[0];
}

// the replica's constants of the spin step
struct SweepConst {
    double zs, B[3], al, inv, tau, tol, la2, lb4;
    int cap;
};
__device__ inline SweepConst sweep_const(const RepDev &R) {
    SweepConst c;
    const double fr = ramp_frac(R);
    c.zs = R.mu_s * MUB;
#pragma unroll
    for (int a = 0; a < 3; a++) c.B[a] = fma(R.B1[a] - R.B0[a], fr, R.B0[a]);
    c.al = R.alpha;
    c.inv = 1.0 / fma(R.alpha, R.alpha, 1.0);
    c.tau = 0.5 * R.dt / HBAR;
    c.tol = R.mid_tol;
    c.cap = R.mid_cap;
    c.la2 = 2.0 * R.landau_a;   // onsite moment-length term
    c.lb4 = 4.0 * R.landau_b;
    return c;
}

// The spin after its visit, from the neighbours' field h, and the number of its
// rotations that stopped at the cap; every lane gets the same. turns = 2 takes
// the colour twice in a row (the end of the ascending and the start of the
// descending pass): the neighbour field is the same for both rotations, the
// second starts from the first one's result.
template <typename real, int L>
__device__ inline int sweep_solve(const RepDev &R, const SweepConst &c, const SweepSpin<real, L> &q, uint32_t orig,
                                  int lane, int turns, int visit0, double hx, double hy, double hz, double &yx, double &yy,
                                  double &yz) {
#pragma clang fp contract(off)
    const double Axx = q.A[0], Ayy = q.A[1], Azz = q.A[2], Axy = q.A[3], Axz = q.A[4], Ayz = q.A[5], os = q.A[6];
    const d4 e = q.e, s4 = q.s4;
    hx += fma(c.zs, c.B[0], e.x);
    hy += fma(c.zs, c.B[1], e.y);
    hz += fma(c.zs, c.B[2], e.z);
    const double al = c.al, inv = c.inv, tau = c.tau, tol = c.tol, la2 = c.la2, lb4 = c.lb4;
    const int cap = c.cap;
    const double Dxx = Axx + os, Dyy = Ayy + os, Dzz = Azz + os;   // A_i + o_i I
    double sx = s4.x, sy = s4.y, sz = s4.z;
    double len = 1.0;    // length of the midpoint vector: 1, or |s| for spins of variable length
    // G(y): the spin rotated about the precession vector taken at the
    // midpoint m = len (s + y)/|s + y| (field, damping, anisotropy, onsite
    // and moment-length terms evaluated at m), by the angle |w| tau (Rodrigues)
    auto rotate = [&](double px, double py, double pz, double &nx, double &ny, double &nz) {
        double mx = sx + px, my = sy + py, mz = sz + pz;
        const double mn = rsqrt_nr(fma(mz, mz, fma(my, my, mx * mx))) * len;
        mx *= mn;
        my *= mn;
        mz *= mn;
        const double kl = fma(lb4, fma(mz, mz, fma(my, my, mx * mx)), la2);
        const double h0 = fma(-kl, mx, fma(-2.0, fma(Axz, mz, fma(Axy, my, Dxx * mx)), hx));
        const double h1 = fma(-kl, my, fma(-2.0, fma(Ayz, mz, fma(Dyy, my, Axy * mx)), hy));
        const double h2 = fma(-kl, mz, fma(-2.0, fma(Dzz, mz, fma(Ayz, my, Axz * mx)), hz));
        const double wx = fma(al, fma(my, h2, -(mz * h1)), h0) * inv;
        const double wy = fma(al, fma(mz, h0, -(mx * h2)), h1) * inv;
        const double wz = fma(al, fma(mx, h1, -(my * h0)), h2) * inv;
        const double w2 = fma(wz, wz, fma(wy, wy, wx * wx));
        if (w2 == 0.0) {
            nx = sx;
            ny = sy;
            nz = sz;
            return;
        }
        const double iw = rsqrt_nr(w2);
        const double th = w2 * iw * tau, ath = fabs(th);   // negative for a backward step
        double sn, cs, omc;
        if (ath <= 1.0) {
            sin_omc_taylor(th, sn, omc);
            cs = 1.0 - omc;
        } else {
            sincos(th, &sn, &cs);
            omc = 1.0 - cs;
        }
        const double ux = wx * iw, uy = wy * iw, uz = wz * iw;
        const double us = fma(uz, sz, fma(uy, sy, ux * sx)), uo = us * omc;
        nx = fma(ux, uo, fma(fma(uy, sz, -(uz * sy)), sn, sx * cs));
        ny = fma(uy, uo, fma(fma(uz, sx, -(ux * sz)), sn, sy * cs));
        nz = fma(uz, uo, fma(fma(ux, sy, -(uy * sx)), sn, sz * cs));
    };
    // the same in single precision, for a starting point only
    const float fhx = (float)hx, fhy = (float)hy, fhz = (float)hz, fal = (float)al, finv = (float)inv, ftau = (float)tau;
    const float gxx = (float)Dxx, gyy = (float)Dyy, gzz = (float)Dzz, gxy = (float)Axy, gxz = (float)Axz, gyz = (float)Ayz;
    const float fla2 = (float)la2, flb4 = (float)lb4;
    auto rotate_f = [&](float sx, float sy, float sz, float ln, float px, float py, float pz, float &nx, float &ny,
                        float &nz) {
        float mx = sx + px, my = sy + py, mz = sz + pz;
        const float mn = __builtin_amdgcn_rsqf(fmaf(mz, mz, fmaf(my, my, mx * mx))) * ln;
        mx *= mn;
        my *= mn;
        mz *= mn;
        const float kl = fmaf(flb4, ln * ln, fla2);
        const float h0 = fmaf(-kl, mx, fmaf(-2.0f, fmaf(gxz, mz, fmaf(gxy, my, gxx * mx)), fhx));
        const float h1 = fmaf(-kl, my, fmaf(-2.0f, fmaf(gyz, mz, fmaf(gyy, my, gxy * mx)), fhy));
        const float h2 = fmaf(-kl, mz, fmaf(-2.0f, fmaf(gzz, mz, fmaf(gyz, my, gxz * mx)), fhz));
        const float wx = fmaf(fal, fmaf(my, h2, -(mz * h1)), h0) * finv;
        const float wy = fmaf(fal, fmaf(mz, h0, -(mx * h2)), h1) * finv;
        const float wz = fmaf(fal, fmaf(mx, h1, -(my * h0)), h2) * finv;
        const float w2 = fmaxf(fmaf(wz, wz, fmaf(wy, wy, wx * wx)), 1.0e-30f);
        const float iw = __builtin_amdgcn_rsqf(w2);
        const float rev = w2 * iw * ftau * 0.15915494f;   // |w| tau in revolutions
        const float sn = __builtin_amdgcn_sinf(rev), cs = __builtin_amdgcn_cosf(rev);
        const float ux = wx * iw, uy = wy * iw, uz = wz * iw;
        const float uo = fmaf(uz, sz, fmaf(uy, sy, ux * sx)) * (1.0f - cs);
        nx = fmaf(ux, uo, fmaf(fmaf(uy, sz, -(uz * sy)), sn, sx * cs));
        ny = fmaf(uy, uo, fmaf(fmaf(uz, sx, -(ux * sz)), sn, sy * cs));
        nz = fmaf(uz, uo, fmaf(fmaf(ux, sy, -(uy * sx)), sn, sz * cs));
    };
    // The midpoint equation y = G(y) is solved by Newton's method on
    // G(y) - y with a forward-difference Jacobian: the four lanes of each
    // quad evaluate G at y and at y + h e_x, y + h e_y, y + h e_z at once
    // (the spin's other lanes are otherwise idle here), exchange the results by
    // quad broadcasts and take the same step. The iteration stops, as the
    // plain fixed-point one, when |G(y) - y| <= tol, and returns G(y): a
    // rotation of the spin, so its length is kept. The Jacobian's relative
    // error (about 1e-9 from the step h = 2^-23) only slows the final
    // convergence to linear with that ratio.
    // The chain of dependent FP64 operations is what a visit costs (about 1,650
    // cycles an iteration), so the first two iterations, which only have to come
    // near, run in FP32 (step 2^-11): from about 1e-7 one FP64 iteration reaches
    // the tolerance and the next one finds that it did, where from y = s it took
    // three and that one. Per colour launch, without and with it: 11,520 atoms FP64
    // 7.0 -> 6.5 us; 262,144 8.1 -> 7.6, FP32 7.3 -> 6.8; 1,048,576 FP32 13.0 -> 12.1;
    // 2,097,152 FP64 21.9 -> 21.3.
    const int sub = lane & 3;
    constexpr double FD_H = 0x1p-23, FD_IH = 0x1p23;
    constexpr float FF_H = 0x1p-11f, FF_IH = 0x1p11f;
    constexpr int PRE = 2;   // FP32 iterations, counted as iterations
    // Spins of variable length with damping: the rotation sits between two
    // longitudinal half steps of the Langevin dynamics over dt/4 each,
    // x += (gamma t/hbar) h(x) + sqrt(2 gamma kB T t/hbar) xi, h the full
    // field at x (neighbours, Zeeman, anisotropy, onsite and moment-length
    // terms), xi the Philox normals of streams 2 + 2 visit and 3 + 2 visit
    // (visit 0 ascending, 1 descending); every lane of the spin takes them
    // alike.
    const bool lsf = R.lsf != 0, lsf_damp = lsf && R.lsf_gamma > 0;
    const double T = lsf_damp ? temperature(R) : 0.0;
    auto lsf_half = [&](double &x, double &y, double &z, uint32_t stream) {
        const double t = 0.25 * R.dt;
        const double kl = la2 + lb4 * (x * x + y * y + z * z);
        const double f0 = hx - 2.0 * (Dxx * x + Axy * y + Axz * z) - kl * x;
        const double f1 = hy - 2.0 * (Axy * x + Dyy * y + Ayz * z) - kl * y;
        const double f2 = hz - 2.0 * (Axz * x + Ayz * y + Dzz * z) - kl * z;
        double xi[3] = {0.0, 0.0, 0.0};
        if (T > 0) gauss3(R.seed, orig, (unsigned long long)R.step, stream, xi);
        const double k = R.lsf_gamma * t / HBAR, sig = sqrt(2.0 * R.lsf_gamma * KB * T * t / HBAR);
        x += k * f0 + sig * xi[0];
        y += k * f1 + sig * xi[1];
        z += k * f2 + sig * xi[2];
    };
    yx = sx;
    yy = sy;
    yz = sz;
    int ncapped = 0;
    for (int turn = 0; turn < turns; turn++) {
        if (turn) {
            sx = yx;
            sy = yy;
            sz = yz;
        }
        const uint32_t visit = (uint32_t)(visit0 + turn);
        if (lsf_damp) lsf_half(sx, sy, sz, 2u + 2u * visit);
        if (lsf) len = sqrt(sx * sx + sy * sy + sz * sz);
        yx = sx;
        yy = sy;
        yz = sz;
        int it0 = 0;
        if (cap > 2 * PRE) {
            const float fx = (float)sx, fy = (float)sy, fz = (float)sz, ln = (float)len;
            float zx = fx, zy = fy, zz = fz, first = 0, last = 0;
#pragma unroll
            for (int k = 0; k < PRE; k++) {
                float nx, ny, nz;
                rotate_f(fx, fy, fz, ln, zx + (sub == 1 ? FF_H : 0.0f), zy + (sub == 2 ? FF_H : 0.0f),
                         zz + (sub == 3 ? FF_H : 0.0f), nx, ny, nz);
                const float g0x = quad_bcast<0>(nx), g0y = quad_bcast<0>(ny), g0z = quad_bcast<0>(nz);
                const float rx = g0x - zx, ry = g0y - zy, rz = g0z - zz;
                last = fmaxf(fabsf(rx), fmaxf(fabsf(ry), fabsf(rz)));
                if (k == 0) first = last;
                const float a00 = 1.0f - (quad_bcast<1>(nx) - g0x) * FF_IH, a10 = -(quad_bcast<1>(ny) - g0y) * FF_IH,
                            a20 = -(quad_bcast<1>(nz) - g0z) * FF_IH;
                const float a01 = -(quad_bcast<2>(nx) - g0x) * FF_IH, a11 = 1.0f - (quad_bcast<2>(ny) - g0y) * FF_IH,
                            a21 = -(quad_bcast<2>(nz) - g0z) * FF_IH;
                const float a02 = -(quad_bcast<3>(nx) - g0x) * FF_IH, a12 = -(quad_bcast<3>(ny) - g0y) * FF_IH,
                            a22 = 1.0f - (quad_bcast<3>(nz) - g0z) * FF_IH;
                auto det2 = [](float a, float b, float c, float d) { return fmaf(a, b, -(c * d)); };
                const float c00 = det2(a11, a22, a12, a21), c01 = det2(a12, a20, a10, a22),
                            c02 = det2(a10, a21, a11, a20);
                const float id = __builtin_amdgcn_rcpf(fmaf(a02, c02, fmaf(a01, c01, a00 * c00)));
                zx = fmaf(fmaf(det2(a01, a12, a02, a11), rz, fmaf(det2(a02, a21, a01, a22), ry, c00 * rx)), id, zx);
                zy = fmaf(fmaf(det2(a02, a10, a00, a12), rz, fmaf(det2(a00, a22, a02, a20), ry, c01 * rx)), id, zy);
                zz = fmaf(fmaf(det2(a00, a11, a01, a10), rz, fmaf(det2(a01, a20, a00, a21), ry, c02 * rx)), id, zz);
            }
            // taken only where it converges (also false for NaN)
            if (last < 0.01f && last <= 0.1f * first && fabsf(zx) + fabsf(zy) + fabsf(zz) < 1.0e4f) {
                yx = zx;
                yy = zy;
                yz = zz;
                it0 = PRE;
            }
        }
        for (int it = it0; it < cap; it++) {
            double nx, ny, nz;
            rotate(yx + (sub == 1 ? FD_H : 0.0), yy + (sub == 2 ? FD_H : 0.0), yz + (sub == 3 ? FD_H : 0.0), nx, ny,
                   nz);
            const double g0x = quad_bcast<0>(nx), g0y = quad_bcast<0>(ny), g0z = quad_bcast<0>(nz);
            const double rx = g0x - yx, ry = g0y - yy, rz = g0z - yz;
            const double diff = fmax(fabs(rx), fmax(fabs(ry), fabs(rz)));
            if (diff <= tol || it + 1 == cap) {
                yx = g0x;
                yy = g0y;
                yz = g0z;
                ncapped += diff > tol;
                break;
            }
            // A = I - J, J columns (G(y + h e_c) - G(y)) / h
            const double a00 = 1.0 - (quad_bcast<1>(nx) - g0x) * FD_IH, a10 = -(quad_bcast<1>(ny) - g0y) * FD_IH,
                         a20 = -(quad_bcast<1>(nz) - g0z) * FD_IH;
            const double a01 = -(quad_bcast<2>(nx) - g0x) * FD_IH, a11 = 1.0 - (quad_bcast<2>(ny) - g0y) * FD_IH,
                         a21 = -(quad_bcast<2>(nz) - g0z) * FD_IH;
            const double a02 = -(quad_bcast<3>(nx) - g0x) * FD_IH, a12 = -(quad_bcast<3>(ny) - g0y) * FD_IH,
                         a22 = 1.0 - (quad_bcast<3>(nz) - g0z) * FD_IH;
            // y += A^-1 r (Cramer's rule); a plain fixed-point step if A is not
            // safely invertible (never for a contracting map)
            auto det2 = [](double a, double b, double c, double d) { return fma(a, b, -(c * d)); };   // ab - cd
            const double c00 = det2(a11, a22, a12, a21), c01 = det2(a12, a20, a10, a22), c02 = det2(a10, a21, a11, a20);
            const double det = fma(a02, c02, fma(a01, c01, a00 * c00));
            if (fabs(det) > 0.25) {
                double id = __builtin_amdgcn_rcp(det);   // refined once: a step needs no more
                id = fma(fma(-det, id, 1.0), id, id);
                yx += fma(det2(a01, a12, a02, a11), rz, fma(det2(a02, a21, a01, a22), ry, c00 * rx)) * id;
                yy += fma(det2(a02, a10, a00, a12), rz, fma(det2(a00, a22, a02, a20), ry, c01 * rx)) * id;
                yz += fma(det2(a00, a11, a01, a10), rz, fma(det2(a01, a20, a00, a21), ry, c02 * rx)) * id;
            } else {
                yx = g0x;
                yy = g0y;
                yz = g0z;
            }
        }
        if (lsf_damp) lsf_half(yx, yy, yz, 3u + 2u * visit);
    }
    return ncapped;
}

// One colour class per launch. Latency is what bounds a class: list position ->
// couplings -> neighbour spins -> midpoint solve -> store. With the spins loaded
// beside the replica's state instead of after it: 11,520 atoms FP64 6.8 -> 6.5 us
// per launch; 262,144 7.9 -> 7.6, FP32 7.2 -> 6.8; 1,048,576 FP32 12.3 -> 12.1;
// 2,097,152 FP64 22.1 -> 21.3.
template <typename real, int L>
__global__ void __launch_bounds__(256) k_sweep(Sys S, Work<real> W, int base, int count, int turns, int visit0) {
    const int lane = threadIdx.x & (L - 1);
    const int t = blockIdx.x * (256 / L) + threadIdx.x / L;
    if (t >= count) return;
    SweepSpin<real, L> q;
    q.load(S, W, lane, base + t);
    const int r = S.col_rid[base + t];
    q.load_atom(S);
    const RepDev &R = S.rep[r];
    // The partners' spins and the replica's constants are loaded beside its
    // state, not after it; a replica whose pass is off may hold couplings of an
    // earlier layout, so that their indices are bounded here.
    const int n = S.N_fe;
    q.load_partners(lane, [&](int j) { return S.spin[(unsigned)j < (unsigned)n ? j : q.i]; });
    const SweepConst k = sweep_const(R);
    asm volatile("" ::: "memory");   // keeps those loads before the branch
    if (!spin_pass_on(R)) return;
    double hx, hy, hz, yx, yy, yz;
    sweep_field<real, L>(S, W, q, lane, [&](int j) { return S.spin[j]; }, hx, hy, hz);
    const int ncapped = sweep_solve(R, k, q, (uint32_t)S.orig[q.i], lane, turns, visit0, hx, hy, hz, yx, yy, yz);
    if (lane == 0) {
        S.spin[q.i] = d4{yx, yy, yz, 0.0};
        if (ncapped) atomicAdd(&S.rep[r].capped, ncapped);
    }
}

// The whole sweep of a replica in one workgroup, its spins in LDS: the colour
// classes follow each other after a barrier, and the couplings of the next
// class's first spins are loaded while this one's are solved, so that a class
// costs its field sum and its solve, 3.3 us, without the launch, the loads and
// the spins' way through memory (5.1 us and the gap to the next launch). What
// bounds it is the chain of about 1,200 dependent instructions of a visit.
// FP64 takes 16 lanes per spin; FP32 couplings leave registers for the eight
// that suit more spins per class. 512 atoms, whole step, FP64 986 -> 756 us,
// FP32 929 -> 665; 1,728 atoms 1,104 -> 1,009 and 1,021 -> 771. A larger replica
// needs several rounds of spins per class in its one workgroup and is slower
// than by class launches: FP64 2,744 atoms 999 -> 1,265 us; FP32 2,744 atoms
// 908 -> 902, 4,096 atoms 1,048 -> 1,080.
template <typename real>
__global__ void __launch_bounds__(SWEEP_LDS_THREADS) k_sweep_lds(Sys S, Work<real> W) {
    constexpr int L = sizeof(real) == 8 ? 16 : 8;
    extern __shared__ double sp[];   // [n_fe][3]
    __shared__ int c0[SWEEP_LDS_COLOURS], c1[SWEEP_LDS_COLOURS], sn[2];   // a colour's list positions; colours, capped
    constexpr int PER = SWEEP_LDS_THREADS / L;
    const int tid = threadIdx.x, lane = tid & (L - 1), t = tid / L, rid = blockIdx.x;
    const RepDev &R = S.rep[rid];
    if (!spin_pass_on(R)) return;
    const int n = R.n_fe, off = R.fe_off;
    for (int c = tid; c < SWEEP_LDS_COLOURS; c += SWEEP_LDS_THREADS) c0[c] = c1[c] = 0;
    if (tid < 2) sn[tid] = 0;
    __syncthreads();
    // inside a colour the list holds the replica's spins one after the other
    for (int a = tid; a < n; a += SWEEP_LDS_THREADS) {
        const int p = S.colpos[off + a], c = S.colour[off + a];
        const d4 v = S.spin[off + a];
        sp[3 * a] = v.x;
        sp[3 * a + 1] = v.y;
        sp[3 * a + 2] = v.z;
        if (p == 0 || S.col_rid[p - 1] != rid || S.colour[S.col_idx[p - 1]] != c) {
            c0[c] = p;
            atomicMax(&sn[0], c + 1);
        }
        if (p + 1 == S.N_fe || S.col_rid[p + 1] != rid || S.colour[S.col_idx[p + 1]] != c) c1[c] = p + 1;
    }
    __syncthreads();
    const int ncol = sn[0], steps = 2 * ncol - 1;
    const SweepConst k = sweep_const(R);
    const auto class_of = [&](int step) { return step < ncol ? step : 2 * ncol - 2 - step; };
    const auto at = [&](int j) {
        const double *v = sp + 3 * (j - off);
        return d4{v[0], v[1], v[2], 0.0};
    };
    SweepSpin<real, L> nx;
    nx.i = off;
    if (steps > 0 && c0[0] + t < c1[0]) {
        nx.load(S, W, lane, c0[0] + t);
        nx.e = S.eta[nx.i];
    }
    int ncapped = 0;
    for (int step = 0; step < steps; step++) {
        const int c = class_of(step), cn = class_of(min(step + 1, steps - 1));
        const int turns = step == ncol - 1 ? 2 : 1, visit0 = step < ncol ? 0 : 1, p1 = c1[c];
        for (int p = c0[c] + t; p < p1; p += PER) {
            SweepSpin<real, L> q = nx;
            if (p + PER < p1) nx.load(S, W, lane, p + PER);
            else if (c0[cn] + t < c1[cn]) nx.load(S, W, lane, c0[cn] + t);
            q.s4 = at(q.i);
            q.load_partners(lane, at);
            double hx, hy, hz, yx, yy, yz;
            sweep_field<real, L>(S, W, q, lane, at, hx, hy, hz);
            ncapped += sweep_solve(R, k, q, (uint32_t)S.orig[q.i], lane, turns, visit0, hx, hy, hz, yx, yy, yz);
            nx.e = S.eta[nx.i];
            if (lane == 0) {
                double *v = sp + 3 * (q.i - off);
                v[0] = yx;
                v[1] = yy;
                v[2] = yz;
            }
        }
        // a lane group without a spin in this class
        if (c0[c] + t >= p1 && c0[cn] + t < c1[cn]) {
            nx.load(S, W, lane, c0[cn] + t);
            nx.e = S.eta[nx.i];
        }
        __syncthreads();
    }
    if (lane == 0 && ncapped) atomicAdd(&sn[1], ncapped);
    for (int a = tid; a < n; a += SWEEP_LDS_THREADS) S.spin[off + a] = d4{sp[3 * a], sp[3 * a + 1], sp[3 * a + 2], 0.0};
    __syncthreads();
    if (tid == 0 && sn[1]) atomicAdd(&S.rep[rid].capped, sn[1]);
}

// Re-layout of the resident replicas: atom k of the new layout takes the state
// rows of atom src[k] of the old one, whose five arrays were copied whole to
// the staging buffer; src[k] = -1 marks atoms of replicas new to the device.
__global__ void __launch_bounds__(256) k_gather_state(const d4 *stage, size_t n_old, const int *src, int n, d4 *pos,
                                                      d4 *vel, d4 *spin, d4 *force, d4 *field) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int s = src[k];
    if (s < 0 || (size_t)s >= n_old) return;
    pos[k] = stage[s];
    vel[k] = stage[n_old + s];
    spin[k] = stage[2 * n_old + s];
    force[k] = stage[3 * n_old + s];
    field[k] = stage[4 * n_old + s];
}

__global__ void k_set_active(RepDev *rep, const int *act, int n) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < n && act[r] >= 0) rep[r].active = act[r];
}

__global__ void k_step_end(Sys S) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= S.n_rep) return;
    RepDev &R = S.rep[r];
    if (!R.active) return;
    if (R.failed & 3) {      // list overflow or coupled same-colour spins: the step is void
        R.active = 0;
        return;
    }
    R.step += 1;
    R.sc_done = 0;
    R.capped = 0;
    // a replica waiting for a new colouring stops after this (exact) step
    if (R.step >= R.step_end || (R.failed & 4)) R.active = 0;
}

// Self-consistent midpoint (Sec. 5.1): the corrector is a fixed-point
// iteration x -> g(x) on the end-of-step spins, g being the sweep at the
// midpoint normalise((S^n + x)/2); x^(0) = S^n. After each sweep, per spin
// carrier of an iterating replica: the residual f = g - x and its max norm
// (non-negative doubles order like their bit patterns, so an integer max over
// the bits is the max; a wave reduces first and issues one atomic when all its
// lanes belong to one replica). Plain iteration keeps x = g for the next pass.
// The accelerated variant (depth > 0, one replica) stores the differences
// dF = f - f_prev, dG = g - g_prev in a ring of depth slots and sums, per
// workgroup in a fixed order, the Gram entries dF_a . dF_b and dF_a . f of
// the mk newest columns.
__device__ inline int sc_slot(int pass, int age, int depth) {   // ring slot of the column made `age` passes ago
    return ((pass - 1 - age) % depth + depth) % depth;
}

__global__ void __launch_bounds__(256) k_sc_check(Sys S, int pass, int depth, int mk) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    int r = -1;
    double d = 0;
    double3 f = {0, 0, 0};
    bool on = false;
    const size_t lf = S.N_fe;
    if (i < S.N_fe) {
        const int ri = S.rid[i];
        const RepDev &R = S.rep[ri];
        if (spin_pass_on(R) && R.sc_tol > 0) {
            on = true;
            const d4 g = S.spin[i];
            const d4 x = pass == 0 ? S.spin_n[i] : S.sc_x[i];
            f = make_double3(g.x - x.x, g.y - x.y, g.z - x.z);
            d = fmax(fabs(f.x), fmax(fabs(f.y), fabs(f.z)));
            r = pass > 0 ? ri : -1;
            if (depth == 0) {
                S.sc_x[i] = g;
            } else {
                if (pass > 0) {
                    const int sl = sc_slot(pass, 0, depth);
                    const d4 fp = S.sc_f[i], gp = S.sc_g[i];
                    S.sc_dF[sl * lf + i] = d4{f.x - fp.x, f.y - fp.y, f.z - fp.z, 0.0};
                    S.sc_dG[sl * lf + i] = d4{g.x - gp.x, g.y - gp.y, g.z - gp.z, 0.0};
                }
                S.sc_f[i] = d4{f.x, f.y, f.z, 0.0};
                S.sc_g[i] = g;
            }
        }
    }
    const int r0 = __shfl(r, 0);
    if (__all(r == r0)) {
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) d = fmax(d, __shfl_xor(d, m));
        if ((threadIdx.x & 63) == 0 && r0 >= 0)
            atomicMax(&S.rep[r0].sc_delta, (unsigned long long)__double_as_longlong(d));
    } else if (r >= 0) {
        atomicMax(&S.rep[r].sc_delta, (unsigned long long)__double_as_longlong(d));
    }
    if (mk == 0) return;   // uniform over the grid
    // Gram entries of the mk newest columns (age order), this workgroup's atoms
    __shared__ double red[4][SC_NK];
    double3 c[SC_MAXD];
#pragma unroll
    for (int a = 0; a < SC_MAXD; a++) {
        c[a] = make_double3(0, 0, 0);
        if (a < mk && on) {
            const d4 v = S.sc_dF[sc_slot(pass, a, depth) * lf + i];
            c[a] = make_double3(v.x, v.y, v.z);
        }
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int k = 0;
#pragma unroll
    for (int a = 0; a < SC_MAXD; a++) {
        if (a >= mk) break;
#pragma unroll
        for (int b = 0; b <= a; b++) {
            double v = c[a].x * c[b].x + c[a].y * c[b].y + c[a].z * c[b].z;
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m);
            if (lane == 0) red[wv][k] = v;
            k++;
        }
        double v = c[a].x * f.x + c[a].y * f.y + c[a].z * f.z;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m);
        if (lane == 0) red[wv][k] = v;
        k++;
    }
    __syncthreads();
    const int nk = mk * (mk + 1) / 2 + mk;
    if (threadIdx.x < nk) {
        const int t = threadIdx.x;
        S.sc_part[(size_t)blockIdx.x * SC_NK + t] = ((red[0][t] + red[1][t]) + red[2][t]) + red[3][t];
    }
}

// One workgroup: converged or capped replicas stop; count the others. A
// replica with a fixed number of correctors (sc_tol 0) iterating beside
// others stops after its k_corr corrector passes, as it would alone; every
// replica records its pass count and last change when it stops. With
// mixing, the Gram matrix is summed over the workgroups in order and the
// regularised normal equations (G + lam I) gam = r, lam = reg * trace(G) / mk,
// are solved by Cholesky; a pivot below 1e-13 of its diagonal entry (a column
// in the span of the others) gives the plain step. sc_out: pending replicas,
// largest change of this pass, used columns, gam[mk].
__global__ void __launch_bounds__(256) k_sc_decide(Sys S, int pass, int mk, int nblocks, double reg, int k_corr) {
    __shared__ int cnt;
    __shared__ unsigned long long dmax;
    __shared__ double sum[SC_NK];
    if (threadIdx.x == 0) {
        cnt = 0;
        dmax = 0;
    }
    __syncthreads();
    int mine = 0;
    for (int r = threadIdx.x; r < S.n_rep; r += blockDim.x) {
        RepDev &R = S.rep[r];
        if (!R.active || R.sc_done) continue;
        if (R.sc_tol <= 0) {
            if (pass >= k_corr) {
                R.sc_done = 1;
                R.sc_passes = pass + 1;
                R.sc_last = 0;
            } else {
                mine++;
            }
            continue;
        }
        const double dl = __longlong_as_double((long long)R.sc_delta);
        if (pass >= 1) atomicMax(&dmax, R.sc_delta);
        if (pass >= 1 && (dl <= R.sc_tol || pass >= R.sc_max)) {
            R.sc_done = 1;
            R.sc_passes = pass + 1;
            R.sc_last = dl;
        }
        R.sc_delta = 0;
        mine += !R.sc_done;
    }
    if (mine) atomicAdd(&cnt, mine);
    const int nk = mk * (mk + 1) / 2 + mk;
    if (threadIdx.x < nk) {
        double v = 0;
        for (int b = 0; b < nblocks; b++) v += S.sc_part[(size_t)b * SC_NK + threadIdx.x];
        sum[threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double *out = S.sc_out;
    out[0] = cnt;
    out[1] = __longlong_as_double((long long)dmax);
    out[2] = 0;
    if (mk == 0 || cnt == 0) return;
    double G[SC_MAXD][SC_MAXD], rh[SC_MAXD], L[SC_MAXD][SC_MAXD], y[SC_MAXD], gam[SC_MAXD];
    int k = 0;
    for (int a = 0; a < mk; a++) {
        for (int b = 0; b <= a; b++) G[a][b] = G[b][a] = sum[k++];
        rh[a] = sum[k++];
    }
    double tr = 0;
    for (int a = 0; a < mk; a++) tr += G[a][a];
    if (!(tr > 0)) return;
    const double lam = reg * tr / mk;
    for (int a = 0; a < mk; a++) {
        for (int b = 0; b <= a; b++) {
            double v = G[a][b] + (a == b ? lam : 0.0);
            for (int c = 0; c < b; c++) v -= L[a][c] * L[b][c];
            if (a == b) {
                if (!(v > 1e-13 * (G[a][a] + lam))) return;
                L[a][a] = sqrt(v);
            } else {
                L[a][b] = v / L[b][b];
            }
        }
    }
    for (int a = 0; a < mk; a++) {
        double v = rh[a];
        for (int c = 0; c < a; c++) v -= L[a][c] * y[c];
        y[a] = v / L[a][a];
    }
    for (int a = mk - 1; a >= 0; a--) {
        double v = y[a];
        for (int c = a + 1; c < mk; c++) v -= L[c][a] * gam[c];
        gam[a] = v / L[a][a];
    }
    for (int a = 0; a < mk; a++) out[3 + a] = gam[a];
    out[2] = mk;
}

// mixed iterate x = g - sum_a gam_a dG_a (the plain x = g when no columns are
// used) and the midpoint spins normalise((S^n + x)/2) of the next pass
__global__ void __launch_bounds__(256) k_sc_mix(Sys S, int pass, int depth) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S.N_fe) return;
    if (!spin_pass_on(S.rep[S.rid[i]])) return;
    const size_t lf = S.N_fe;
    const int used = (int)S.sc_out[2];
    const d4 g = S.spin[i];
    double x = g.x, y = g.y, z = g.z;
    for (int a = 0; a < used; a++) {
        const double ga = S.sc_out[3 + a];
        const d4 v = S.sc_dG[sc_slot(pass, a, depth) * lf + i];
        x -= ga * v.x;
        y -= ga * v.y;
        z -= ga * v.z;
    }
    S.sc_x[i] = d4{x, y, z, 0.0};
    const d4 a = S.spin_n[i];
    const double mx = 0.5 * (a.x + x), my = 0.5 * (a.y + y), mz = 0.5 * (a.z + z);
    const double n = S.rep[S.rid[i]].lsf ? 1.0 : sqrt(mx * mx + my * my + mz * mz);
    S.spin_hat[i] = d4{mx / n, my / n, mz / n, 0.0};
}

// per-chunk partial sums of the observables (fixed tree), then per replica
template <typename real>
__global__ void __launch_bounds__(256) k_obs_partial(Sys S, Work<real> W, const Chunk *chunks, double *partial) {
    __shared__ double red[NOBS][256];
    const Chunk c = chunks[blockIdx.x];
    const int t = threadIdx.x;
    double v[NOBS];
#pragma unroll
    for (int k = 0; k < NOBS; k++) v[k] = 0;
    const int i = c.begin + t;
    if (i < c.end) {
        const RepDev &R = S.rep[c.rid];
        const int fe = i < S.N_fe;
        const d4 vel = S.vel[i], s = S.spin[i], H = S.field[i], p = S.pos[i], F = S.force[i];
        const double m = R.mass[fe ? 0 : 1];
        v[0] = (double)W.Ei[i];
        v[1] = 0.5 * m * (vel.x * vel.x + vel.y * vel.y + vel.z * vel.z) / KAPPA;
        if (fe) {
            const double fr = ramp_frac(R), zs = R.mu_s * MUB;
            v[2] = -zs * ((R.B0[0] + (R.B1[0] - R.B0[0]) * fr) * s.x + (R.B0[1] + (R.B1[1] - R.B0[1]) * fr) * s.y +
                          (R.B0[2] + (R.B1[2] - R.B0[2]) * fr) * s.z);
            const double cx = s.y * H.z - s.z * H.y, cy = s.z * H.x - s.x * H.z, cz = s.x * H.y - s.y * H.x;
            v[3] = cx * cx + cy * cy + cz * cz;
            v[4] = s.x * H.x + s.y * H.y + s.z * H.z;
            v[5] = s.x;
            v[6] = s.y;
            v[7] = s.z;
            v[8] = sqrt(s.x * s.x + s.y * s.y + s.z * s.z);
        }
        const double chk = p.x + p.y + p.z + vel.x + vel.y + vel.z + s.x + s.y + s.z + F.x + F.y + F.z + v[0];
        v[NOBS - 1] = isfinite(chk) ? 0.0 : 1.0;
    }
#pragma unroll
    for (int k = 0; k < NOBS; k++) red[k][t] = v[k];
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (t < off)
#pragma unroll
            for (int k = 0; k < NOBS; k++) red[k][t] += red[k][t + off];
        __syncthreads();
    }
    if (t < NOBS) partial[(size_t)blockIdx.x * NOBS + t] = red[t][0];
}

// one workgroup per replica: thread t sums chunks t, t+256, ... in order,
// then a fixed tree; the result depends only on the replica's own chunks
__global__ void __launch_bounds__(256) k_obs_final(Sys S, const int *chunk_ptr, const double *partial, double *out) {
    __shared__ double red[NOBS][256];
    const int r = blockIdx.x, t = threadIdx.x;
    double v[NOBS];
#pragma unroll
    for (int k = 0; k < NOBS; k++) v[k] = 0;
    for (int c = chunk_ptr[r] + t; c < chunk_ptr[r + 1]; c += 256)
#pragma unroll
        for (int k = 0; k < NOBS; k++) v[k] += partial[(size_t)c * NOBS + k];
#pragma unroll
    for (int k = 0; k < NOBS; k++) red[k][t] = v[k];
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (t < off)
#pragma unroll
            for (int k = 0; k < NOBS; k++) red[k][t] += red[k][t + off];
        __syncthreads();
    }
    // slot 9: the replica's capped rotations (a counter, not a sum); slot
    // NOBS-1 counts non-finite atoms
    if (t < NOBS) out[(size_t)r * NOBS + t] = t == 9 ? (double)S.rep[r].capped : red[t][0];
}

}  // namespace

void launch_kick(const Sys &S, hipStream_t st) {
    if (S.N) hipLaunchKernelGGL(k_kick, dim3(nblk(S.N, 256)), dim3(256), 0, st, S);
}
void launch_drift(const Sys &S, hipStream_t st) {
    if (S.N) hipLaunchKernelGGL(k_drift, dim3(nblk(S.N, 256)), dim3(256), 0, st, S);
}
void launch_pos4(const Sys &S, hipStream_t st) {
    if (S.N) hipLaunchKernelGGL(k_pos4, dim3(nblk(S.N, 256)), dim3(256), 0, st, S);
}
void launch_langevin(const Sys &S, hipStream_t st) {
    if (S.N) hipLaunchKernelGGL(k_langevin, dim3(nblk(S.N, 256)), dim3(256), 0, st, S);
}
void launch_spin_prep(const Sys &S, hipStream_t st) {
    if (S.N_fe) hipLaunchKernelGGL(k_spin_prep, dim3(nblk(S.N_fe, 256)), dim3(256), 0, st, S);
}
void launch_spin_restore(const Sys &S, hipStream_t st) {
    if (S.N_fe) hipLaunchKernelGGL(k_spin_restore, dim3(nblk(S.N_fe, 256)), dim3(256), 0, st, S);
}
void launch_spin_mid(const Sys &S, hipStream_t st) {
    if (S.N_fe) hipLaunchKernelGGL(k_spin_mid, dim3(nblk(S.N_fe, 256)), dim3(256), 0, st, S);
}
void launch_step_end(const Sys &S, hipStream_t st) {
    if (S.n_rep) hipLaunchKernelGGL(k_step_end, dim3(nblk(S.n_rep, 64)), dim3(64), 0, st, S);
}
void launch_set_active(RepDev *rep, const int *act, int n, hipStream_t st) {
    if (n) hipLaunchKernelGGL(k_set_active, dim3(nblk(n, 64)), dim3(64), 0, st, rep, act, n);
}
void launch_gather_state(const d4 *stage, size_t n_old, const int *src, int n, d4 *pos, d4 *vel, d4 *spin, d4 *force,
                         d4 *field, hipStream_t st) {
    if (n) hipLaunchKernelGGL(k_gather_state, dim3(nblk(n, 256)), dim3(256), 0, st, stage, n_old, src, n, pos, vel,
                              spin, force, field);
}
int sc_part_blocks(int n_fe) { return nblk(n_fe, 256); }
void launch_sc_check(const Sys &S, int pass, int depth, double reg, int k_corr, hipStream_t st) {
    const int mk = depth > 0 ? (pass < depth ? pass : depth) : 0;
    const int nb = nblk(S.N_fe, 256);
    if (S.N_fe) hipLaunchKernelGGL(k_sc_check, dim3(nb), dim3(256), 0, st, S, pass, depth, mk);
    hipLaunchKernelGGL(k_sc_decide, dim3(1), dim3(256), 0, st, S, pass, S.N_fe ? mk : 0, nb, reg, k_corr);
}
void launch_sc_mix(const Sys &S, int pass, int depth, hipStream_t st) {
    if (S.N_fe) hipLaunchKernelGGL(k_sc_mix, dim3(nblk(S.N_fe, 256)), dim3(256), 0, st, S, pass, depth);
}

// colours 0, 1, .., C-1 and then C-1, .., 0; the two visits of colour C-1 are
// one launch
template <typename real>
void launch_sweep(const Sys &S, const Work<real> &W, const int *col_ptr_host, int n_colours, int lds_spins,
                  hipStream_t st) {
    if (lds_spins > 0) {
        hipLaunchKernelGGL(k_sweep_lds<real>, dim3(S.n_rep), dim3(SWEEP_LDS_THREADS), 3 * sizeof(double) * lds_spins, st, S,
                           W);
        return;
    }
    for (int pass = 0; pass < 2; pass++)
        for (int cc = 0; cc < n_colours; cc++) {
            if (pass == 1 && cc == 0) continue;       // done as the second turn of the last ascending launch
            const int c = pass == 0 ? cc : n_colours - 1 - cc;
            const int turns = (pass == 0 && cc == n_colours - 1) ? 2 : 1;
            const int b = col_ptr_host[c], n = col_ptr_host[c + 1] - b;
            if (n >= SWEEP_WIDER_MIN)
                hipLaunchKernelGGL((k_sweep<real, 4>), dim3(nblk(n, 256 / 4)), dim3(256), 0, st, S, W, b, n, turns,
                                   pass);
            else if (n >= SWEEP_WIDE_MIN)
                hipLaunchKernelGGL((k_sweep<real, 8>), dim3(nblk(n, 256 / 8)), dim3(256), 0, st, S, W, b, n, turns,
                                   pass);
            else if (n > 0)
                hipLaunchKernelGGL((k_sweep<real, 16>), dim3(nblk(n, 256 / 16)), dim3(256), 0, st, S, W, b, n, turns,
                                   pass);
        }
}

template <typename real>
void launch_observe(const Sys &S, const Work<real> &W, const Chunk *chunks, int n_chunks,
                    const int *chunk_ptr, double *partial, double *out, hipStream_t st) {
    if (n_chunks == 0) return;
    hipLaunchKernelGGL(k_obs_partial<real>, dim3(n_chunks), dim3(256), 0, st, S, W, chunks, partial);
    hipLaunchKernelGGL(k_obs_final, dim3(S.n_rep), dim3(256), 0, st, S, chunk_ptr, partial, out);
}

template void launch_sweep<double>(const Sys &, const Work<double> &, const int *, int, int, hipStream_t);
template void launch_sweep<float>(const Sys &, const Work<float> &, const int *, int, int, hipStream_t);
template void launch_observe<double>(const Sys &, const Work<double> &, const Chunk *, int, const int *, double *,
                                     double *, hipStream_t);
template void launch_observe<float>(const Sys &, const Work<float> &, const Chunk *, int, const int *, double *,
                                    double *, hipStream_t);

}  // namespace nep
