// kernels_nep.hip -- the spin-aware NEP on the device: descriptor, per-species
// read-out, backward pass (forces and effective fields) and the bilinear spin
// couplings of the frozen-Fp magnetic energy.
//
// Mapping. Every kernel walks lists of the neighbours inside the cutoffs, put
// together from the Verlet rows by k_active for each new set of positions.
// Radial-set work (radial, exchange, DMI, anisotropic, single-ion channels
// inside 6 A) runs one lane per atom, or eight in small replicas. Angular-set
// work (angular and spin-angular channels inside 4.5 A) takes eight atoms per
// wavefront: the descriptor eight lanes per atom, each with a tile of the
// accumulators A_nlm and B_nlm, the backward pass and the coupling assembly a
// lane per pair. Spin-carrying atoms occupy the leading index range and every grid
// is split so that a wavefront never mixes species; the lists hold spin
// carriers first, so the pair type tau, and with it every coefficient address,
// is uniform across the wavefront inside each loop. Sums over neighbours follow
// the in-cutoff ranks (ascending atom index): results are deterministic and
// independent of how replicas are batched.
//
// Gather without atomics: the backward pass writes, per listed pair (i,j),
// dE_i/dd_ij and dE_i/ds_j into a pair record; a gather kernel then forms
// F_k = sum_j dE_k/dd_kj - sum_j dE_j/dd_jk and H_k = -(dE_k/ds_k + sum_j dE_j/ds_k)
// by reading the partner's record at the reverse slot.
#include "engine.h"

namespace nep {

namespace {

// grid split: blocks b in [0, nbFe) take spin carriers, the rest the others
__device__ inline int atom_of_block(const Sys &S, int b, int per_block, int nbFe, int local, bool &fe) {
    if (b < nbFe) {
        fe = true;
        const int i = b * per_block + local;
        return i < S.N_fe ? i : -1;
    }
    fe = false;
    const int i = S.N_fe + (b - nbFe) * per_block + local;
    return i < S.N ? i : -1;
}

// i, or -1 when its replica is not advancing (paused for a new colouring,
// finished, or its step void): the force-field kernels leave such atoms alone
__device__ inline int live(const Sys &S, int i) { return i >= 0 && S.rep[S.rid[i]].active ? i : -1; }
// the same for the radial-set sums over L lanes per atom
template <int L>
__device__ inline int live_lanes(const Sys &S, int i) {
    if (i < 0) return -1;
    const RepDev &R = S.rep[S.rid[i]];
    return R.active && (R.wide != 0) == (L > 1) ? i : -1;
}

// v summed over the L = 1 or 8 neighbouring lanes of an atom, every lane with
// the result: xor 1, 2 and (the mirrored lane, whose quad holds the same sum) 4
template <int CTRL>
__device__ inline double dpp(double v) {
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ inline float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int L, typename real>
__device__ inline real lane_sum(real v) {
    if constexpr (L > 1) {
        v += dpp<0xB1>(v);    // quad_perm [1, 0, 3, 2]
        v += dpp<0x4E>(v);    // quad_perm [2, 3, 0, 1]
        v += dpp<0x141>(v);   // row_half_mirror
    }
    return v;
}

template <typename real>
__device__ inline void load_spin(const d4 *sp, int j, real s[3]) {
    const d4 v = sp[j];
    s[0] = (real)v.x;
    s[1] = (real)v.y;
    s[2] = (real)v.z;
}

// displacement to an already loaded neighbour position, in FP64, then cast
template <typename real>
__device__ inline real geom_p(const Img &R, const d4 &pi, const d4 &pj, real d[3]) {
    double dx, dy, dz;
    min_image(R, pi, pj, dx, dy, dz);
    d[0] = (real)dx;
    d[1] = (real)dy;
    d[2] = (real)dz;
    return d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
}

// C[k] = sum_n Fp[n] c[n][k]  (coefficients wave-uniform)
template <typename real>
__device__ inline void contract(const real *c, const real *Fp, int nn, real C[NB]) {
#pragma unroll
    for (int k = 0; k < NB; k++) C[k] = 0;
    // once per atom: rolled, so the coefficients are loaded nine at a time
#pragma unroll 1
    for (int n = 0; n < nn; n++) {
        const real f = Fp[n];
#pragma unroll
        for (int k = 0; k < NB; k++) C[k] += f * c[n * NB + k];
    }
}

template <typename real>
__device__ inline real dotk(const real C[NB], const real f[NB]) {
    real s = 0;
#pragma unroll
    for (int k = 0; k < NB; k++) s += C[k] * f[k];
    return s;
}

// -------------------------------------------------------------------------
// Neighbours inside the cutoffs at the present positions, compacted in row
// order: the Verlet rows hold a third more (the skin), at places that differ
// from atom to atom, so every pair kernel that walked them spent that share of
// its lanes on nothing. One pass per set of positions, eight lanes per atom
// (ranks by ballot); the lists depend on the positions alone and not on which
// farther atoms the rows happen to hold.
// What bounds it is the gather of the neighbours' positions, one L1 access per
// 16 bytes and lane: the test runs on the single-precision positions (one
// access), and the few pairs that lie within its rounding error of a cutoff
// are tested as the pair kernels compute r^2.
// 2,097,152 atoms, FP64: 1.4 ms of a step for its two passes, against 6.8 ms
// that the pair kernels no longer spend on the skin.
// -------------------------------------------------------------------------

// the cutoff tests of one atom
template <typename real>
struct CutTest {
    static constexpr real rc = (real)RC_R, rca = (real)RC_A;
    float px, py, pz, bx, by, bz, ix, iy, iz, tol;
    __device__ void set(const Img &R, const float4 &p) {
        px = p.x, py = p.y, pz = p.z;
        bx = (float)R.b[0], by = (float)R.b[1], bz = (float)R.b[2];
        ix = (float)R.ib[0], iy = (float)R.ib[1], iz = (float)R.ib[2];
        // Rounding of r^2 near a cutoff: with periodic coordinates folded into
        // the box (pos4), both atoms' coordinates, the box edge, its multiple
        // (0 or +-1 edges) and the differences are at most M, each rounded by
        // 2^-24 M or less, five of them per component; r below 7 A, so
        // 2 sqrt(3) r e + 3 e^2 for the components and 1e-5 for the sum.
        float M = fmaxf(fmaxf(fabsf(px), fabsf(py)), fabsf(pz));
        M = fmaxf(M, fmaxf(fmaxf(bx, by), bz)) + 7.0f;
        const float e = M * 3.0e-7f;
        tol = 25.0f * e + 3.0f * e * e + 1.0e-5f;
    }
    __device__ float r2(const float4 &q) const {
        float dx = q.x - px, dy = q.y - py, dz = q.z - pz;
        dx -= bx * rintf(dx * ix);
        dy -= by * rintf(dy * iy);
        dz -= bz * rintf(dz * iz);
        return dx * dx + dy * dy + dz * dz;
    }
    // inside rc_R, inside rc_A
    __device__ void operator()(const Sys &S, const Img &R, int i, int j, const float4 &q, bool &in, bool &inA) const {
        const float c2 = (float)(RC_R * RC_R), ca2 = (float)(RC_A * RC_A);
        const float f2 = r2(q);
        in = f2 < c2;
        inA = f2 < ca2;
        if (!(fabsf(f2 - c2) >= tol && fabsf(f2 - ca2) >= tol)) {   // also for NaN
            real d[3];
            const real x2 = geom_p(R, S.pos[i], S.pos[j], d);
            in = x2 < rc * rc;
            inA = x2 < rca * rca;
        }
    }
};

// The lists are put together in LDS and written in whole lines: stored by each
// lane as it went along (its ranks differ from its neighbours') they left L2 in
// parts, 3.8 times their bytes. Latency bounds it, so LDS holds the ranks that a
// crystal or a liquid has (62 and 29 in FeGe, 84 and 41 in water, in the mean) and
// any further ones are stored one by one: six workgroups fit in a CU's LDS instead
// of three; and the partner's slot is used a round after its load. Mean of a
// step's two passes: 2,097,152 atoms 1.06 -> 0.72 ms; 1,048,576 in a slab, FP32
// 0.52 -> 0.36; 262,144 128 -> 85 us; 375,000 water atoms 304 -> 202 (one pass).
constexpr int ACT_R = 96, ACT_A = 48;
template <typename real>
__global__ void __launch_bounds__(256) k_active(Sys S, int n) {
    constexpr int ATOMS = 32;
    __shared__ int sR[ACT_R * ATOMS];                       // [rank][atom]
    __shared__ __align__(16) int sA[ATOMS * ACT_A];         // [atom][rank]
    __shared__ __align__(8) uint16_t sS[ATOMS * ACT_A];
    __shared__ uint16_t sX[MAXFE * ATOMS];                  // [rank][atom]
    __shared__ int sn[2 * ATOMS];                           // entries of sR and sX
    const int lane = threadIdx.x & 7, gbase = threadIdx.x & 56, at = threadIdx.x >> 3;
    const int first = blockIdx.x * ATOMS;
    const size_t ld = S.N, lf = S.N_fe;
    int nR = 0, nA = 0, nX = 0;
    // the loads of the prologue together; the first two row entries are read
    // before the row's length is known, and bounded in case they lie beyond it
    const int ii = min(first + at, n - 1);
    const RepDev &rep = S.rep[S.rid[ii]];
    const int len = S.lenR[ii], lenfe = S.lenFeR[ii];
    const float4 pi = S.pos4[ii];
    int vn = S.rowR[(size_t)lane * ld + ii], vm = S.rowR[(size_t)(lane + 8) * ld + ii];
    if ((vn & ~ANG_BIT) >= S.N) vn = ii;
    float4 qn = S.pos4[vn & ~ANG_BIT];
    const int i = first + at < n && rep.active ? ii : -1;
    if (i >= 0) {
        const Img R = img_of(rep);
        CutTest<real> cut;
        cut.set(R, pi);
        const int mx = S.mag && i < S.N_fe ? MAXFE : 0;
        const unsigned below = (1u << lane) - 1u;
        int nL = 0, nFeR = 0, nFeA = 0;
        // the row entry two rounds ahead, its position one round ahead; the
        // partner's slot is used one round after its load was started
        if (lane + 8 >= len) vm = i;
        int po = -1, px = -1, pa = 0, prev = 0;   // the pair's angular rank, its place in sX, and its slots
        const auto put_slots = [&]() {
            const uint16_t sr = (uint16_t)(pa | prev << 8);
            if (po >= ACT_A) S.actS[(size_t)i * MAXA + po] = sr;
            else if (po >= 0) sS[at * ACT_A + po] = sr;
            if (px >= 0) sX[px] = po >= 0 && pa < MAXFE && prev < MAXFE ? sr : NO_RECORD;
        };
        for (int s0 = 0; s0 < len; s0 += 8) {
            const int s = s0 + lane, v = vn, j = v & ~ANG_BIT;
            const float4 q = qn;
            vn = vm;
            qn = S.pos4[vn & ~ANG_BIT];
            vm = s + 16 < len ? S.rowR[(size_t)(s + 16) * ld + i] : i;
            const bool listed = s < len, ang = listed && (v & ANG_BIT);
            bool in = false, inA = false;
            if (listed) cut(S, R, i, j, q, in, inA);
            inA = inA && ang;
            const unsigned mL = (unsigned)(__ballot(ang) >> gbase) & 0xffu;   // an entry's angular slot: the flagged ones before it
            const unsigned mR = (unsigned)(__ballot(in) >> gbase) & 0xffu;
            const unsigned mA = (unsigned)(__ballot(inA) >> gbase) & 0xffu;
            const int kR = nR + __popc(mR & below);
            put_slots();
            po = px = -1;
            if (inA) {
                pa = nL + __popc(mL & below);
                po = nA + __popc(mA & below);
                prev = S.revA[(size_t)pa * ld + i];
                if (po < ACT_A) sA[at * ACT_A + po] = j;
                else S.actA[(size_t)i * MAXA + po] = j;
            }
            if (in) {
                if (kR < ACT_R) sR[kR * ATOMS + at] = j;
                else S.actR[(size_t)kR * ld + i] = j;
                if (s < lenfe && kR < mx) px = kR * ATOMS + at;
            }
            nL += __popc(mL);
            nR += __popc(mR);
            nA += __popc(mA);
            if (s0 < lenfe) {
                const unsigned mf = lenfe - s0 < 8 ? (1u << (lenfe - s0)) - 1u : 0xffu;
                nFeR += __popc(mR & mf);
                nFeA += __popc(mA & mf);
            }
        }
        put_slots();
        nX = min(nFeR, mx);
        if (lane == 0) {
            S.cntR[i] = nR;
            S.cntFeR[i] = nFeR;
            S.cntA[i] = nA;
            S.cntFeA[i] = nFeA;
        }
    }
    if (lane == 0) {
        sn[at] = min(nR, ACT_R);
        sn[ATOMS + at] = nX;
    }
    __syncthreads();
    const int a2 = threadIdx.x & (ATOMS - 1), r0 = threadIdx.x / ATOMS;
    for (int r = r0; r < sn[a2]; r += 256 / ATOMS) S.actR[(size_t)r * ld + first + a2] = sR[r * ATOMS + a2];
    for (int r = r0; r < sn[ATOMS + a2]; r += 256 / ATOMS) S.xS[(size_t)r * lf + first + a2] = sX[r * ATOMS + a2];
    for (int k = 4 * lane; k < min(nA, ACT_A); k += 32) {
        *reinterpret_cast<int4 *>(S.actA + (size_t)i * MAXA + k) = *reinterpret_cast<const int4 *>(sA + at * ACT_A + k);
        *reinterpret_cast<ushort4 *>(S.actS + (size_t)i * MAXA + k) =
            *reinterpret_cast<const ushort4 *>(sS + at * ACT_A + k);
    }
}

// -------------------------------------------------------------------------
// forward: radial set, L lanes per atom: lane l takes the in-cutoff pairs of
// rank l modulo L
// -------------------------------------------------------------------------

template <typename real, int L, int THREADS>
__device__ __forceinline__ void desc_radial(const Sys &S, const real *__restrict__ C, const Work<real> &W, const d4 *spin,
                                            int block, int nbFe) {
    bool fe;
    const int l = threadIdx.x % L;
    const int i = live_lanes<L>(S, atom_of_block(S, block, THREADS / L, nbFe, threadIdx.x / L, fe));
    if (i < 0) return;
    const Img R = img_of(S.rep[S.rid[i]]);
    const d4 pi = S.pos[i];
    const real rc = (real)RC_R;
    const int cnt = S.cntR[i], nfe = S.cntFeR[i];
    const size_t ld = S.N;
    const int *row = S.actR + i;
    real *q = W.q + (size_t)i * DP;
    real qR[NR], qE[NR], qD[NR], qA[NR], qS[NR];
#pragma unroll
    for (int n = 0; n < NR; n++) qR[n] = qE[n] = qD[n] = qA[n] = qS[n] = 0;
    real si[3];
    load_spin(spin, i, si);
    if (fe && S.mag) {
        real FR[NB], FE[NB], FD[NB], FA[NB], FS[NB];
#pragma unroll
        for (int k = 0; k < NB; k++) FR[k] = FE[k] = FD[k] = FA[k] = FS[k] = 0;
        // neighbour index two slots ahead, position and spin one slot ahead
        int j1 = l < nfe ? row[(size_t)l * ld] : 0;
        int j2 = l + L < nfe ? row[(size_t)(l + L) * ld] : j1;
        d4 p1 = S.pos[j1], v1 = spin[j1];
        for (int s = l; s < nfe; s += L) {
            const d4 pj = p1, vj = v1;
            j1 = j2;
            p1 = S.pos[j1];
            v1 = spin[j1];
            if (s + 2 * L < nfe) j2 = row[(size_t)(s + 2 * L) * ld];
            real d[3];
            const real r2 = geom_p(R, pi, pj, d);
            real r, ir;
            r_and_inv(r2, r, ir);
            const real rh[3] = {d[0] * ir, d[1] * ir, d[2] * ir};
            real f[NB];
            radial_basis(r, rc, f);
            const real sj[3] = {(real)vj.x, (real)vj.y, (real)vj.z};
            const real ss = si[0] * sj[0] + si[1] * sj[1] + si[2] * sj[2];
            const real cx = si[1] * sj[2] - si[2] * sj[1], cy = si[2] * sj[0] - si[0] * sj[2],
                       cz = si[0] * sj[1] - si[1] * sj[0];
            const real dm = rh[0] * cx + rh[1] * cy + rh[2] * cz;
            const real a = si[0] * rh[0] + si[1] * rh[1] + si[2] * rh[2];
            const real b = sj[0] * rh[0] + sj[1] * rh[1] + sj[2] * rh[2];
            const real ab = a * b, aa = a * a;
#pragma unroll
            for (int k = 0; k < NB; k++) {
                FR[k] += f[k];
                FE[k] += f[k] * ss;
                FD[k] += f[k] * dm;
                FA[k] += f[k] * ab;
                FS[k] += f[k] * aa;
            }
        }
        // contract with tau = (Fe, Fe) coefficients
        for (int n = 0; n < NR; n++) {
            const int o = (0 * NR + n) * NB;
            real r_ = 0, e_ = 0, d_ = 0, a_ = 0, s_ = 0;
#pragma unroll
            for (int k = 0; k < NB; k++) {
                r_ += (C + P_CR)[o + k] * FR[k];
                e_ += (C + P_CEX)[o + k] * FE[k];
                d_ += (C + P_CDM)[o + k] * FD[k];
                a_ += (C + P_CAN)[o + k] * FA[k];
                s_ += (C + P_CSI)[o + k] * FS[k];
            }
            qR[n] = r_;
            qE[n] = e_;
            qD[n] = d_;
            qA[n] = a_;
            qS[n] = s_;
        }
        // non-magnetic neighbours: only the radial and single-ion channels survive
#pragma unroll
        for (int k = 0; k < NB; k++) FR[k] = FS[k] = 0;
        int j1_ = nfe + l < cnt ? row[(size_t)(nfe + l) * ld] : 0;
        int j2_ = nfe + l + L < cnt ? row[(size_t)(nfe + l + L) * ld] : j1_;
        d4 p1_ = S.pos[j1_];
        for (int s = nfe + l; s < cnt; s += L) {
            const d4 pj_ = p1_;
            j1_ = j2_;
            p1_ = S.pos[j1_];
            if (s + 2 * L < cnt) j2_ = row[(size_t)(s + 2 * L) * ld];
            real d[3];
            const real r2 = geom_p(R, pi, pj_, d);
            real r, ir;
            r_and_inv(r2, r, ir);
            real f[NB];
            radial_basis(r, rc, f);
            const real a = (si[0] * d[0] + si[1] * d[1] + si[2] * d[2]) * ir;
            const real aa = a * a;
#pragma unroll
            for (int k = 0; k < NB; k++) {
                FR[k] += f[k];
                FS[k] += f[k] * aa;
            }
        }
        for (int n = 0; n < NR; n++) {
            const int o = (1 * NR + n) * NB;
            real r_ = 0, s_ = 0;
#pragma unroll
            for (int k = 0; k < NB; k++) {
                r_ += (C + P_CR)[o + k] * FR[k];
                s_ += (C + P_CSI)[o + k] * FS[k];
            }
            qR[n] += r_;
            qS[n] += s_;
        }
    } else {
        for (int part = 0; part < 2; part++) {
            real FR[NB];
#pragma unroll
            for (int k = 0; k < NB; k++) FR[k] = 0;
            const int b = (part ? nfe : 0) + l, e = part ? cnt : nfe;
            int j1_ = b < e ? row[(size_t)b * ld] : 0;
            int j2_ = b + L < e ? row[(size_t)(b + L) * ld] : j1_;
            d4 p1_ = S.pos[j1_];
            for (int s = b; s < e; s += L) {
                const d4 pj_ = p1_;
                j1_ = j2_;
                p1_ = S.pos[j1_];
                if (s + 2 * L < e) j2_ = row[(size_t)(s + 2 * L) * ld];
                real d[3];
                const real r2 = geom_p(R, pi, pj_, d);
                real f[NB], r, ir;
                r_and_inv(r2, r, ir);
                radial_basis(r, rc, f);
#pragma unroll
                for (int k = 0; k < NB; k++) FR[k] += f[k];
            }
            const int tau = (fe ? 0 : 2) + part;
            for (int n = 0; n < NR; n++) {
                const int o = (tau * NR + n) * NB;
                real r_ = 0;
#pragma unroll
                for (int k = 0; k < NB; k++) r_ += (C + P_CR)[o + k] * FR[k];
                qR[n] += r_;
            }
        }
    }
#pragma unroll
    for (int n = 0; n < NR; n++) {
        qR[n] = lane_sum<L>(qR[n]);
        if (fe && S.mag) {
            qE[n] = lane_sum<L>(qE[n]);
            qD[n] = lane_sum<L>(qD[n]);
            qA[n] = lane_sum<L>(qA[n]);
            qS[n] = lane_sum<L>(qS[n]);
        }
    }
    if (l) return;
    q[D_OS] = fe && S.mag ? si[0] * si[0] + si[1] * si[1] + si[2] * si[2] : real(0);
#pragma unroll
    for (int n = 0; n < NR; n++) {
        q[D_R + n] = qR[n];
        q[D_EX + n] = qE[n];
    }
    // The structural-only read-out contracts over the first 40 entries (the
    // zero onsite and exchange entries 37-39 included): it never reads the
    // later magnetic channels, which stay unwritten there.
    if (S.mag) {
#pragma unroll
        for (int n = 0; n < NR; n++) {
            q[D_DM + n] = qD[n];
            q[D_AN + n] = qA[n];
            q[D_SI + n] = qS[n];
        }
    }
}

template <typename real>
__global__ void __launch_bounds__(256) k_desc_radial(Sys S, const real *__restrict__ C, Work<real> W,
                                                     const d4 *spin, int nbFe) {
    desc_radial<real, 1, 256>(S, C, W, spin, blockIdx.x, nbFe);
}

// -------------------------------------------------------------------------
// angular-set kernels: one wavefront = 8 atoms x 8 lanes
// Every neighbour loop runs in two phases, spin-carrying neighbours first
// (they lead each list) and then the others, so within a phase the pair type
// tau and thus every coefficient address is uniform across the wavefront and
// the coefficients are scalar operands.
// -------------------------------------------------------------------------

constexpr int ANG_ATOMS = 8;             // atoms per workgroup
constexpr int ANG_TW = 2 * NA + NLM;     // staged values per neighbour
constexpr int ANG_TS = 8 * ANG_TW + 1;   // per-atom stride (shifts LDS banks)

// What the lanes of other atoms need of an atom: position, spin, box and
// inverse box (zero on free axes), as doubles in LDS. Filled by its eight lanes.
// A wavefront of these kernels lives for two to five rounds of pairs, two to four
// wavefronts share a SIMD, and the latency of each dependent load of its
// prologue (replica, counts, list entries, positions) costs about a round: so
// all loads that do not depend on each other are issued before the first is
// used, from the atom's own rows whether or not it turns out to be live.
constexpr int AT_W = 12;
struct AtomStage {
    d4 v;             // position (lane 0), spin (lane 1)
    double b;         // lanes 2-7: one component of the box or inverse box
    bool active;
    __device__ void load(const Sys &S, const d4 *spin, int i, int lane) {
        const RepDev &R = S.rep[S.rid[i]];
        const int c = max(lane - 2, 0), a = c < 3 ? c : c - 3;
        v = (lane == 1 ? spin : S.pos)[i];
        b = c < 3 ? R.box[a] : R.ibox[a];
        if (!R.pbc[a]) b = 0;
        active = R.active != 0;
    }
    __device__ void put(int lane, double *at) const {
        if (lane < 2) {
            at[3 * lane] = v.x;
            at[3 * lane + 1] = v.y;
            at[3 * lane + 2] = v.z;
        } else {
            at[4 + lane] = b;
        }
    }
};
template <typename real>
__device__ inline real geom_lds(const double *at, const d4 &pj, real d[3]) {
    const Img g = {{at[6], at[7], at[8]}, {at[9], at[10], at[11]}};
    return geom_p(g, d4{at[0], at[1], at[2], 0.0}, pj, d);
}

// The pairs of the eight atoms of a wavefront as one sequence, atom after atom:
// off[k] is the first pair of atom k (wave-uniform), find() the atom of pair p.
struct Flat8 {
    int off[ANG_ATOMS + 1];
    __device__ void set(int n) {   // n: pairs of this lane's atom
        off[0] = 0;
#pragma unroll
        for (int k = 0; k < ANG_ATOMS; k++) off[k + 1] = off[k] + __builtin_amdgcn_readlane(n, 8 * k);
    }
    __device__ int find(int p, int &o) const {
        int a = 0;
        o = 0;
#pragma unroll
        for (int k = 1; k < ANG_ATOMS; k++) {
            const bool g = p >= off[k];
            a += g;
            o = g ? off[k] : o;
        }
        return a;
    }
    __device__ int own(int slot) const {   // first pair of atom `slot`
        int o = 0;
#pragma unroll
        for (int k = 1; k < ANG_ATOMS; k++) o = slot >= k ? off[k] : o;
        return o;
    }
};

template <typename real>
__device__ inline real dotc(const real *c, const real f[NB]) {
    real s = 0;
#pragma unroll
    for (int k = 0; k < NB; k++) s += c[k] * f[k];
    return s;
}

// forward: per round, lanes stage eight neighbours of their atom (radial
// functions g^A_n and (s_i.s_j) g^sa_n for all n, the 24 harmonics) in LDS,
// then the lanes accumulate A_nlm and B_nlm over the staged neighbours. B only
// has spin-carrying pairs (spin-carrying centre, first phase).
// A lane holds all n of six harmonics, 13 LDS values for 42 products (three
// harmonics of A and B together would take 17). Where both A and B are
// accumulated, lanes 0-3 take A and lanes 4-7 B; where one of them is, lanes
// 0-3 take the even and lanes 4-7 the odd entries, and the two halves are added
// afterwards: so the phase with A alone comes first. Lane 7 - q has the harmonics of lane q, so that the halves meet
// under the mirrored-lane permutation. Lanes without a neighbour stage zeros:
// the trip count is that of the wavefront and the loop unrolls. The rounds of both
// phases form one sequence, loaded ahead across the phases' border.
// FP64 is bound by latency at the two wavefronts per SIMD that the accumulators
// and the tile allow (VALU 49 %, LDS 46 % busy), FP32 by VALU issue.
// 262,144 atoms, mean of the three passes of a step: FP64 236 -> 220 us, FP32
// 143 -> 124; 2,097,152 atoms, FP64: 1.86 -> 1.75 ms.
// Pass modes: PASS_FULL stores A (all atoms) and B (spin carriers) for the
// backward pass; PASS_SPIN (spin carriers only) stores A for the coupling
// assembly; PASS_SPIN_REUSE (same positions as the preceding PASS_SPIN)
// takes A from it and only recomputes B and q^sa.
template <typename real>
__device__ __forceinline__ void desc_angular(const Sys &S, const real *__restrict__ C, const Work<real> &W,
                                             const d4 *spin, int nbFe, int mode) {
    __shared__ real tile[ANG_ATOMS * ANG_TS];
    const int lane = threadIdx.x & 7, slot = threadIdx.x >> 3;
    bool fe;
    const int i0 = atom_of_block(S, blockIdx.x, ANG_ATOMS, nbFe, slot, fe), ii = max(i0, 0);
    const bool reuse = mode == PASS_SPIN_REUSE, mag = S.mag && fe;
    const int *row = S.actA + (size_t)ii * MAXA;
    const d4 pi = S.pos[ii];
    real si[3];
    load_spin(spin, ii, si);
    int cnt = S.cntA[ii], nfe = S.cntFeA[ii];
    const RepDev &rep = S.rep[S.rid[ii]];
    const Img R = img_of(rep);
    const int i = i0 >= 0 && rep.active ? i0 : -1;
    if (i < 0) cnt = nfe = 0;
    // most pairs of an atom of the wavefront, by phase
    int most0 = 0, most1 = 0;
#pragma unroll
    for (int k = 0; k < ANG_ATOMS; k++) {
        const int f = __builtin_amdgcn_readlane(nfe, 8 * k);
        most0 = max(most0, f);
        most1 = max(most1, __builtin_amdgcn_readlane(cnt, 8 * k) - f);
    }
    if (reuse) most1 = 0;
    const int n = lane < NA ? lane : NA - 1;
    const int h = lane >> 2, m0 = 6 * (h ? 7 - lane : lane);
    const real rc = (real)RC_A;
    real acc[NA][6];
#pragma unroll
    for (int x = 0; x < NA; x++)
#pragma unroll
        for (int m = 0; m < 6; m++) acc[x][m] = 0;
    real *my = tile + slot * ANG_TS;
    // rounds of the first phase, then of the second: this lane's neighbour
    // index two rounds ahead, its position and spin one round ahead
    const int rd1 = (most1 + 7) >> 3, rds = rd1 + ((most0 + 7) >> 3);
    const auto slot_of = [&](int rd) { return rd < rd1 ? nfe + 8 * rd + lane : 8 * (rd - rd1) + lane; };
    const auto end_of = [&](int rd) { return rd < rd1 ? cnt : nfe; };
    const auto index_of = [&](int rd, int other) { return slot_of(rd) < end_of(rd) ? row[slot_of(rd)] : other; };
    int jc = index_of(0, ii), jn = index_of(1, jc);
    d4 pc = S.pos[jc], vc = {0, 0, 0, 0};
    if (mag) vc = spin[jc];
    const auto phase = [&](const int part, int rd, const int rd_end, const int most) {
        const int tau = (fe ? 0 : 2) + part;
        const real *cA = C + P_CA + tau * NA * NB, *cS = C + P_CSA + tau * NA * NB;
        const bool spins = mag && part == 0, both = spins && !reuse;
        const int rd0 = rd;
        for (; rd < rd_end; rd++) {
            const bool on = slot_of(rd) < end_of(rd);
            const d4 pj = pc, vj = vc;
            jc = jn;
            pc = S.pos[jc];
            if (mag && rd + 1 >= rd1) vc = spin[jc];
            jn = index_of(rd + 2, jc);
            real *en = my + lane * ANG_TW;
            {
                real d[3];
                real r2 = geom_p(R, pi, pj, d);
                if (!on) {   // any finite geometry; its radial functions are zeroed
                    d[0] = r2 = 1;
                    d[1] = d[2] = 0;
                }
                real r, ir;
                r_and_inv(r2, r, ir);
                real f[NB];
                radial_basis(r, rc, f);
#pragma unroll
                for (int k = 0; k < NB; k++) f[k] = on ? f[k] : real(0);
                if (spins) {
                    const real sj[3] = {(real)vj.x, (real)vj.y, (real)vj.z};
                    const real sig = on ? si[0] * sj[0] + si[1] * sj[1] + si[2] * sj[2] : real(0);
#pragma unroll
                    for (int nn = 0; nn < NA; nn++) en[NA + nn] = sig * dotc(cS + nn * NB, f);
                }
                if (!reuse) {
#pragma unroll
                    for (int nn = 0; nn < NA; nn++) en[nn] = dotc(cA + nn * NB, f);
                }
                real Y[NLM];
                harmonics(d[0] * ir, d[1] * ir, d[2] * ir, Y);
#pragma unroll
                for (int m = 0; m < NLM; m++) en[2 * NA + m] = Y[m];
            }
            __syncthreads();
            // this lane's entries: all, or those of its half
            const real *eg = my + (both ? h * NA : (h ? ANG_TW : 0) + (reuse ? NA : 0));
            const real *ey = my + (both ? 0 : (h ? ANG_TW : 0)) + 2 * NA + m0;
            const int step = both ? ANG_TW : 2 * ANG_TW;
            const int left = min(8, most - 8 * (rd - rd0)), trips = both ? left : (left + 1) >> 1;
#pragma unroll 2
            for (int q = 0; q < trips; q++) {
                real y[6];
#pragma unroll
                for (int m = 0; m < 6; m++) y[m] = ey[q * step + m];
#pragma unroll
                for (int x = 0; x < NA; x++) {
                    const real g = eg[q * step + x];
#pragma unroll
                    for (int m = 0; m < 6; m++) acc[x][m] += g * y[m];
                }
            }
            __syncthreads();
        }
        if (!both) {   // the halves added, the first keeps the sum; the last phase leaves it in both
#pragma unroll
            for (int x = 0; x < NA; x++)
#pragma unroll
                for (int m = 0; m < 6; m++) {
                    acc[x][m] += dpp<0x141>(acc[x][m]);   // row_half_mirror
                    if (part && h) acc[x][m] = 0;
                }
        }
    };
    if (!reuse) phase(1, 0, rd1, most1);
    phase(0, rd1, rds, most0);
    // regroup through LDS: lane n takes A_n and B_n over all 24 harmonics
    real An[NLM], Bn[NLM];
    if (h == 0) {
#pragma unroll
        for (int x = 0; x < NA; x++)
#pragma unroll
            for (int m = 0; m < 6; m++) my[x * NLM + m0 + m] = acc[x][m];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < NLM; m++) An[m] = my[n * NLM + m];
    __syncthreads();
    if (mag && !reuse) {
        if (h) {
#pragma unroll
            for (int x = 0; x < NA; x++)
#pragma unroll
                for (int m = 0; m < 6; m++) my[x * NLM + m0 + m] = acc[x][m];
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < NLM; m++) Bn[m] = my[n * NLM + m];
    } else {
#pragma unroll
        for (int m = 0; m < NLM; m++) Bn[m] = 0;
    }
    if (i < 0 || lane >= NA) return;
    real *ab = W.AB + ((size_t)i * NA + n) * NAB;
    real *q = W.q + (size_t)i * DP;
    if (reuse) {
#pragma unroll
        for (int m = 0; m < NLM; m++) {
            Bn[m] = An[m];
            An[m] = ab[m];
        }
    }
    real qa[4] = {0, 0, 0, 0}, qs[4] = {0, 0, 0, 0};
#pragma unroll
    for (int m = 0; m < NLM; m++) {
        qa[l_of_lm(m) - 1] += An[m] * An[m];
        qs[l_of_lm(m) - 1] += An[m] * Bn[m];
    }
#pragma unroll
    for (int l = 0; l < 4; l++) {
        if (!reuse) q[D_A + 4 * n + l] = qa[l];
        if (S.mag) q[D_SA + 4 * n + l] = qs[l];   // beyond the structural-only read-out's entries
    }
    if (!reuse) {
#pragma unroll
        for (int m = 0; m < NLM; m++) ab[m] = An[m];
    }
    if (mag && mode == PASS_FULL) {   // B only for the spin-carrying backward
#pragma unroll
        for (int m = 0; m < NLM; m++) ab[NLM + m] = Bn[m];
    }
}

template <typename real>
__global__ void __launch_bounds__(64) k_desc_angular(Sys S, const real *__restrict__ C, Work<real> W,
                                                     const d4 *spin, int nbFe, int mode) {
    desc_angular(S, C, W, spin, nbFe, mode);
}

// the same and the radial set of the wide replicas, in blocks of the same eight
// atoms: the two do not depend on each other, and a small system is bound by
// the length of its chain of launches (nb = 0: the radial set alone)
template <typename real>
__global__ void __launch_bounds__(64, 2) k_desc_both(Sys S, const real *__restrict__ C, Work<real> W, const d4 *spin,
                                                  int nbFe, int nb, int mode) {
    if ((int)blockIdx.x < nb) desc_angular(S, C, W, spin, nbFe, mode);
    else desc_radial<real, WIDE_LANES, 64>(S, C, W, spin, blockIdx.x - nb, nbFe);
}

// -------------------------------------------------------------------------
// per-species read-out on the matrix cores
//   Z = Q W0^T + b0 (atoms x 64), E_i = b1 + w1 . tanh(Z_i),
//   Fp = [(1 - tanh^2(Z)) * w1] W0 (atoms x 104)
// One wavefront takes a tile of 16 atoms of one species; W0^T of that species
// is staged in LDS once per workgroup. Operand layout of v_mfma_*_16x16x4:
// A[i][k] in lane i + 16k, B[k][j] in lane j + 16k. Accumulator element r of
// lane l holds column l % 16 and row 4 (l / 16) + r for the FP32
// instruction, row (l / 16) + 4 r for the FP64 one (checked on gfx950).
// Both products run transposed, Z^T = W0 Q^T (hidden x atoms) and Fp^T = W0^T
// G^T: a lane's accumulators of the first are then, element for element, the B
// operands it supplies to the second, whose contraction over the hidden units
// is taken in the order that makes it so (k-step 4 mt + r is hidden unit
// 16 mt + row(kq, r) in lane quarter kq). No transposition, no LDS tile.
// -------------------------------------------------------------------------

template <typename real>
struct MF;
template <>
struct MF<double> {
    typedef double acc_t __attribute__((ext_vector_type(4)));
    __device__ static acc_t mma(double a, double b, acc_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    __device__ static int row(int kq, int r) { return kq + 4 * r; }
};
template <>
struct MF<float> {
    typedef float acc_t __attribute__((ext_vector_type(4)));
    __device__ static acc_t mma(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    __device__ static int row(int kq, int r) { return 4 * kq + r; }
};

constexpr int MLP_WAVES = 8;           // 8 wavefronts x 16 atoms per workgroup
constexpr int MLP_ATOMS = 16 * MLP_WAVES;
// Launches of at most so many 16-atom tiles give a tile to four wavefronts
// (SPLIT): a wavefront with a tile of its own runs 11,700 cycles of matrix
// instructions in a row, and 512 atoms occupied two CUs. Per launch, FP64, the
// former with its coefficient kernel: 512 atoms, full 22 + 13 -> 10 us, spin
// pass 20 + 6 -> 8; 10,648 atoms 25 + 15 -> 23 and 21 + 7.5 -> 13. From about three
// tiles per CU on the split form's staging of W0 for every tile costs as much.
constexpr int MLP_SPLIT_TILES = 704;
// LDS row stride of W0^T. The operand reads walk 16 rows (lanes i16) and 4
// columns (lanes kq); a stride of 2 dwords mod 64 for 8-byte elements puts those
// reads on distinct banks, and of 4 dwords for the 16-byte reads of FP32.
template <typename real>
struct MlpLds;
template <>
struct MlpLds<double> {
    static constexpr int LD = NH + 1;
};
template <>
struct MlpLds<float> {
    static constexpr int LD = NH + 4;
};

// KD: descriptor entries the read-out contracts over (104 for the spin-aware
// model, 40 for the structural-only one, whose 37 entries lead each row).
// SPIN: a spin-step pass, which needs neither E_i nor the gradient of the
// structural entries: the tiles before the one that holds D_OS are left out.
// What bounds it: FP64 shares its units between the matrix and the vector
// instructions, and the library's tanh took as many cycles as the products; FP32
// waited on scattered 4-byte reads and stores and on the LDS transposition of the
// hidden tile. 2,097,152 atoms FP64, full pass 1.9 -> 1.43 ms, spin pass 0.95 ->
// 0.61 (the products alone at the measured 71.8 TFLOP/s: 0.81 and 0.34);
// 1,048,576 atoms FP32 0.60 -> 0.33 and 0.30 -> 0.155. With the descriptor rows
// loaded beside W0 instead of after it: 1.36 and 0.58; 0.27 and 0.134. With the
// radial-set coefficients, formerly 0.54 and 0.22 (FP32 0.16 and 0.08) more: 1.53
// and 0.66; 0.38 and 0.152.

// The radial-set coefficients contracted with the atom's Fp, blocks b of NB
// values: the radial channel's for each neighbour species p (b = p), CR_p[k] =
// sum_n c^R_{2t+p}[n][k] Fp^R_n; on spin carriers the exchange, DMI and
// anisotropic-exchange ones (b = 2, 3, 4; Fe-Fe pairs) and the single-ion ones
// for each neighbour species (b = 5 + p), CS_p[k] = sum_n c^si_p[n][k] Fp^si_n.
// rcoef holds [CR_0 | CR_1 | CS_0 | CS_1][N][NB]: a neighbour reads the NB values
// of its own species (and NB more if it carries a spin), and atoms adjacent in
// memory share cache lines; mcoef [N_fe][CE, CD, CA].
// The accumulators of the second product are, element for element, the B
// operands of this one, K_b Fp^T with a block's coefficients as a 16-row operand
// from LDS, contracted over the block's entries of the descriptor alone: no
// kernel reads Fp back for them.
constexpr int COEF_BLOCKS = 7;
constexpr int coef_entry(int b) { return b < 2 ? D_R : b == 2 ? D_EX : b == 3 ? D_DM : b == 4 ? D_AN : D_SI; }
// does k-step r of descriptor tile x touch block b (over the lane quarters)?
template <typename real>
constexpr bool coef_step(int b, int x, int r) {
    for (int kq = 0; kq < 4; kq++) {
        const int n = 16 * x + (sizeof(real) == 8 ? kq + 4 * r : 4 * kq + r) - coef_entry(b);
        if (n >= 0 && n < NR) return true;
    }
    return false;
}
// the steps of the blocks from b0 on, one after the other: the p-th, and the number of one
struct CoefStep {
    int b, x, r;
};
template <typename real>
constexpr CoefStep coef_nth(int b0, int p) {
    for (int b = b0; b < COEF_BLOCKS; b++)
        for (int x = 0; x < (DP + 15) / 16; x++)
            for (int r = 0; r < 4; r++)
                if (coef_step<real>(b, x, r) && p-- == 0) return {b, x, r};
    return {COEF_BLOCKS, 0, 0};
}
template <typename real>
constexpr int coef_rank(int b0, int b, int x, int r) {
    int p = 0;
    for (CoefStep s = coef_nth<real>(b0, 0); s.b < b || (s.b == b && (s.x < x || (s.x == x && s.r < r)));)
        s = coef_nth<real>(b0, ++p);
    return p;
}
template <int... X>
struct Tiles {
    static constexpr int n = sizeof...(X);
    static constexpr int at(int k) {
        const int t[] = {X...};
        return t[k];
    }
};

// SPLIT: a workgroup of four wavefronts takes 16 atoms. Wavefront w forms hidden
// units 16 w .. 16 w + 15, the activations meet in LDS, and each wavefront
// takes the descriptor tiles of its coefficient blocks and its share of the
// others. Every sum has the order of the other form, so the bits are the same.
template <typename real, int KD, bool SPIN, bool SPLIT>
__global__ void __launch_bounds__(SPLIT ? 256 : 512) k_mlp(Sys S, ModelDev<real> M, Work<real> W, int nbFe) {
    typedef typename MF<real>::acc_t acc_t;
    constexpr int WLD = MlpLds<real>::LD, THREADS = SPLIT ? 256 : 512, ATOMS = SPLIT ? 16 : MLP_ATOMS;
    constexpr bool f64 = sizeof(real) == 8;
    constexpr int KDT = (KD + 15) / 16 * 16, NT = KDT / 16;
    constexpr int B0 = SPIN ? 2 : 0, B1 = KD < DP ? 2 : SPIN ? 5 : COEF_BLOCKS;   // the pass's coefficient blocks
    constexpr int NP = coef_rank<real>(B0, B1, 0, 0);
    __shared__ __align__(16) real sW[KDT * WLD];
    __shared__ real sB[2 * NH];   // b0, w1
    __shared__ real sK[NP * 64];       // [step][lane]
    __shared__ real sA[SPLIT ? 16 * 64 : 1];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const bool fe = (int)blockIdx.x < nbFe;
    const int t = fe ? 0 : 1;
    const int end = fe ? S.N_fe : S.N;
    const int a0 = (fe ? blockIdx.x * ATOMS : S.N_fe + (blockIdx.x - nbFe) * ATOMS) + (SPLIT ? 0 : wave * 16);
    const real *W0 = M.W0 + (size_t)t * DP * NH;
    // Every load of the kernel is issued here, before the first is used. The
    // rows of atoms that are not live are read too: an atom is a column of both
    // products, and what comes of theirs is not stored.
    const int i16 = lane & 15, kq = lane >> 4;
    const int arow = a0 + i16, row_in = min(arow, end - 1);
    const RepDev &rep = S.rep[S.rid[row_in]];
    const real *qrow = W.q + (size_t)row_in * DP;
    // FP32 takes sixteen descriptor entries as four k-steps of four consecutive
    // ones per lane quarter (one 16-byte load), the last eight as two of two.
    auto entry = [&](int ks) {
        if constexpr (f64) return ks * 4 + kq;
        else return ks < KD / 16 * 4 ? (ks >> 2) * 16 + 4 * kq + (ks & 3) : KD / 16 * 16 + 2 * kq + (ks & 1);
    };
    constexpr int SV = KDT * NH / THREADS;
    static_assert(SV * THREADS == KDT * NH, "W0 is staged in whole rounds");
    real w0[SV];
#pragma unroll
    for (int v = 0; v < SV; v++) {
        const int x = v * THREADS + threadIdx.x;
        w0[v] = x < KD * NH ? W0[x] : real(0);
    }
    const real bw = threadIdx.x < NH ? M.b0[t * NH + threadIdx.x] : M.w1[t * NH + threadIdx.x % NH];
    real qa[KD / 4];
    if constexpr (f64) {
#pragma unroll
        for (int ks = 0; ks < KD / 4; ks++) qa[ks] = qrow[ks * 4 + kq];
    } else {
        static_assert(KD % 16 == 8, "two k-steps after the sixteens");
#pragma unroll
        for (int g = 0; g < KD / 16; g++) {
            const float4 v = *reinterpret_cast<const float4 *>(qrow + 16 * g + 4 * kq);
            qa[4 * g] = v.x;
            qa[4 * g + 1] = v.y;
            qa[4 * g + 2] = v.z;
            qa[4 * g + 3] = v.w;
        }
        const float2 v = *reinterpret_cast<const float2 *>(qrow + KD / 16 * 16 + 2 * kq);
        qa[KD / 4 - 2] = v.x;
        qa[KD / 4 - 1] = v.y;
    }
    const bool mag = KD == DP && fe;   // the magnetic and single-ion blocks
    static_for<NP>([&](auto PP) {
        constexpr int p = decltype(PP)::value;
        constexpr CoefStep c = coef_nth<real>(B0, p);
        if (wave != p % (THREADS / 64)) return;
        constexpr int first = coef_entry(c.b);
        const int n = 16 * c.x + MF<real>::row(kq, c.r) - first;
        const real *k = M.cR + (c.b < 2 ? P_CR + (2 * t + c.b) * NR * NB
                                        : c.b == 2 ? P_CEX : c.b == 3 ? P_CDM : c.b == 4 ? P_CAN : P_CSI + (c.b - 5) * NR * NB);
        sK[p * 64 + lane] = n >= 0 && n < NR && i16 < NB && (c.b < 2 || mag) ? k[n * NB + i16] : real(0);
    });
    const bool rv = arow < end && rep.active;
    const real b1 = M.b1[t];
#pragma unroll
    for (int v = 0; v < SV; v++) {
        const int x = v * THREADS + threadIdx.x;
        sW[(x / NH) * WLD + x % NH] = w0[v];
    }
    if (threadIdx.x < 2 * NH) sB[threadIdx.x] = bw;
    __syncthreads();
    // Z^T = W0 Q^T + b0
    real act[4][4];
    if constexpr (SPLIT) {
        acc_t z;
#pragma unroll
        for (int r = 0; r < 4; r++) z[r] = sB[16 * wave + MF<real>::row(kq, r)];
#pragma unroll
        for (int ks = 0; ks < KD / 4; ks++) z = MF<real>::mma(sW[entry(ks) * WLD + wave * 16 + i16], qa[ks], z);
#pragma unroll
        for (int r = 0; r < 4; r++) sA[(4 * wave + r) * 64 + lane] = dtanh<real>(z[r]);
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < 4; mt++)
#pragma unroll
            for (int r = 0; r < 4; r++) act[mt][r] = sA[(4 * mt + r) * 64 + lane];
    } else {
        acc_t z[4];
#pragma unroll
        for (int mt = 0; mt < 4; mt++)
#pragma unroll
            for (int r = 0; r < 4; r++) z[mt][r] = sB[16 * mt + MF<real>::row(kq, r)];
#pragma unroll
        for (int ks = 0; ks < KD / 4; ks++) {
#pragma unroll
            for (int mt = 0; mt < 4; mt++) z[mt] = MF<real>::mma(sW[entry(ks) * WLD + mt * 16 + i16], qa[ks], z[mt]);
        }
#pragma unroll
        for (int mt = 0; mt < 4; mt++)
#pragma unroll
            for (int r = 0; r < 4; r++) act[mt][r] = dtanh<real>(z[mt][r]);
    }
    // energy and the hidden-layer gradient
    real e = 0;
    acc_t g[4];
#pragma unroll
    for (int mt = 0; mt < 4; mt++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const real w = sB[NH + 16 * mt + MF<real>::row(kq, r)];
            const real a = act[mt][r];
            e += w * a;
            g[mt][r] = w * (real(1) - a * a);
        }
    if (!SPIN && (!SPLIT || wave == 0)) {
        e += __shfl_xor(e, 16);
        e += __shfl_xor(e, 32);
        if (kq == 0 && rv) W.Ei[arow] = b1 + e;
    }
    // Fp^T = W0^T G^T: A = W0^T tile from LDS, B = this lane's g; at most four
    // descriptor tiles at once to bound the registers
    real *fp = W.Fp + (size_t)(rv ? arow : 0) * DP;
    acc_t cb[COEF_BLOCKS];
#pragma unroll
    for (int b = 0; b < COEF_BLOCKS; b++) cb[b] = acc_t{0, 0, 0, 0};
    // the tiles of TL, those whose bit is set in `stored` written out, and their
    // part of the blocks [b0, b1)
    const auto tiles = [&](auto TL, auto STORED, auto FIRST, auto LAST) {
        typedef decltype(TL) T;
        constexpr int stored = decltype(STORED)::value;
        acc_t f[T::n];
#pragma unroll
        for (int x = 0; x < T::n; x++) f[x] = acc_t{0, 0, 0, 0};
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
            if constexpr (f64) {
#pragma unroll
                for (int r = 0; r < 4; r++)
#pragma unroll
                    for (int x = 0; x < T::n; x++)
                        f[x] = MF<real>::mma(sW[(T::at(x) * 16 + i16) * WLD + 16 * mt + 4 * r + kq], g[mt][r], f[x]);
            } else {
#pragma unroll
                for (int x = 0; x < T::n; x++) {
                    const float4 w = *reinterpret_cast<const float4 *>(&sW[(T::at(x) * 16 + i16) * WLD + 16 * mt + 4 * kq]);
                    f[x] = MF<real>::mma(w.x, g[mt][0], f[x]);
                    f[x] = MF<real>::mma(w.y, g[mt][1], f[x]);
                    f[x] = MF<real>::mma(w.z, g[mt][2], f[x]);
                    f[x] = MF<real>::mma(w.w, g[mt][3], f[x]);
                }
            }
        }
        static_for<decltype(LAST)::value - decltype(FIRST)::value>([&](auto BB) {
            constexpr int b = decltype(FIRST)::value + decltype(BB)::value;
            static_for<T::n>([&](auto XX) {
                constexpr int x = T::at(decltype(XX)::value);
                static_for<4>([&](auto RR) {
                    constexpr int r = decltype(RR)::value;
                    if constexpr (coef_step<real>(b, x, r)) {
                        constexpr int p = coef_rank<real>(B0, b, x, r);
                        cb[b] = MF<real>::mma(sK[p * 64 + lane], f[decltype(XX)::value][r], cb[b]);
                    }
                });
            });
        });
        if (!rv) return;
        static_for<T::n>([&](auto XX) {
            constexpr int k = decltype(XX)::value, x = T::at(k);
            if constexpr ((stored >> k & 1) != 0) {
                if constexpr (f64) {
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const int d = x * 16 + kq + 4 * r;
                        if (d < KD) fp[d] = f[k][r];
                    }
                } else {
                    const int d = x * 16 + 4 * kq;   // KD is a multiple of four
                    if (d < KD) *reinterpret_cast<float4 *>(fp + d) = make_float4(f[k][0], f[k][1], f[k][2], f[k][3]);
                }
            }
        });
    };
    const auto put = [&](auto FIRST, auto LAST) {
        if (!rv) return;
        static_for<decltype(LAST)::value - decltype(FIRST)::value>([&](auto BB) {
            constexpr int b = decltype(FIRST)::value + decltype(BB)::value;
            if (b >= 2 && !mag) return;
            real *o = b >= 2 && b < 5 ? W.mcoef + (size_t)arow * MCOEF + (b - 2) * NB
                                      : W.rcoef + ((size_t)(b < 2 ? b : b - 3) * S.N + arow) * NB;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int k = MF<real>::row(kq, r);
                if (k < NB) o[k] = cb[b][r];
            }
        });
    };
#define I_(x) std::integral_constant<int, x>{}
    if constexpr (!SPLIT) {
        if constexpr (KD < DP) {
            tiles(Tiles<0, 1, 2>{}, I_(7), I_(0), I_(2));
            put(I_(0), I_(2));
        } else if constexpr (SPIN) {
            tiles(Tiles<2, 3, 4>{}, I_(7), I_(2), I_(5));
            put(I_(2), I_(5));
            tiles(Tiles<5, 6>{}, I_(3), I_(0), I_(0));
        } else {
            tiles(Tiles<0, 1, 2>{}, I_(7), I_(0), I_(4));   // block 3 starts in tile 2
            put(I_(0), I_(3));
            tiles(Tiles<3, 4, 5, 6>{}, I_(15), I_(3), I_(7));
            put(I_(3), I_(7));
        }
    } else if constexpr (KD < DP) {
        if (wave == 0) {
            tiles(Tiles<0>{}, I_(1), I_(0), I_(2));
            put(I_(0), I_(2));
        } else if (wave == 1) {
            tiles(Tiles<1>{}, I_(1), I_(0), I_(0));
        } else if (wave == 2) {
            tiles(Tiles<2>{}, I_(1), I_(0), I_(0));
        }
    } else {
        if (wave == 0) {
            if constexpr (SPIN) {
                tiles(Tiles<6>{}, I_(1), I_(0), I_(0));
            } else {
                tiles(Tiles<0, 1, 6>{}, I_(7), I_(0), I_(2));
                put(I_(0), I_(2));
            }
        } else if (wave == 1) {
            tiles(Tiles<2, 3>{}, I_(3), I_(2), I_(4));
            put(I_(2), I_(4));
        } else if (wave == 2) {
            tiles(Tiles<3, 4>{}, I_(2), I_(4), I_(5));
            put(I_(4), I_(5));
        } else {
            if constexpr (SPIN) {
                tiles(Tiles<5>{}, I_(1), I_(0), I_(0));
            } else {
                tiles(Tiles<4, 5>{}, I_(2), I_(5), I_(7));
                put(I_(5), I_(7));
            }
        }
    }
#undef I_
}

// -------------------------------------------------------------------------
// backward: radial set
// -------------------------------------------------------------------------

template <typename real>
__device__ inline void put_pair(real *pb, size_t idx, const real G[3], const real h[3]) {
    real *p = pb + idx * 6;
    p[0] = G[0];
    p[1] = G[1];
    p[2] = G[2];
    p[3] = h[0];
    p[4] = h[1];
    p[5] = h[2];
}

// Structural part of the radial-set backward pass: the radial channel of
// every pair and the single-ion term of spin-carrying centres, L lanes per atom.
// Both halves of each pair come from this lane: G_ij = dE_i/dd_ij from the
// atom's own coefficients and G_ji = dE_j/dd_ji from the neighbour's
// contracted block (and its spin), so F_i = sum_j (G_ij - G_ji) needs no
// pair records. Own sums: F_i and dE_i/ds_i (single-ion and onsite).
template <typename real>
__device__ inline void partner_radial(const real *cR, const real *cS, bool fe_j, const d4 *spin, int j, real r,
                                      real ir, const real rh[3], const real f[NB], const real df[NB], real Gj[3]) {
    const real dgR = dotc(cR + (size_t)j * NB, df);
    if (fe_j) {
        real sj[3];
        load_spin(spin, j, sj);
        const real gS = dotc(cS + (size_t)j * NB, f), dgS = dotc(cS + (size_t)j * NB, df);
        // rhat_ji = -rhat_ij
        const real a = -(sj[0] * rh[0] + sj[1] * rh[1] + sj[2] * rh[2]);
        const real radial = dgR + dgS * a * a;
        const real ks = real(2) * gS * a * ir;
#pragma unroll
        for (int x = 0; x < 3; x++) Gj[x] = -radial * rh[x] + ks * (sj[x] + a * rh[x]);
    } else {
#pragma unroll
        for (int x = 0; x < 3; x++) Gj[x] = -dgR * rh[x];
    }
}

// Optional short-range repulsion of one pair of type tau at distance r: the
// universal screened-Coulomb (ZBL) potential K Z_i Z_j / r phi(r/a), phi a
// sum of four exponentials of r/a, times the switch
// (1 + cos(pi (r - r_inner)/(r_outer - r_inner)))/2 above r_inner. Z is the
// model's short-range block (products K Z_i Z_j, inverse screening lengths,
// r_inner, r_outer, pi/(r_outer - r_inner)). V and dV/dr of the pair.
template <typename real>
__device__ inline void short_range(const real *Z, int tau, real r, real ir, real &V, real &dV) {
    const real ia = Z[4 + tau];
    const real c0 = real(0.18175) * dexp<real>(real(-3.19980) * ia * r);
    const real c1 = real(0.50986) * dexp<real>(real(-0.94229) * ia * r);
    const real c2 = real(0.28022) * dexp<real>(real(-0.40290) * ia * r);
    const real c3 = real(0.02817) * dexp<real>(real(-0.20162) * ia * r);
    const real phi = c0 + c1 + c2 + c3;
    const real dphi = -ia * (real(3.19980) * c0 + real(0.94229) * c1 + real(0.40290) * c2 + real(0.20162) * c3);
    const real v = Z[tau] * phi * ir;
    const real dv = Z[tau] * (dphi - phi * ir) * ir;
    real s = 1, ds = 0;
    if (r > Z[8]) {
        const real w = Z[10], x = w * (r - Z[8]);
        s = real(0.5) * (real(1) + dcos<real>(x));
        ds = real(-0.5) * w * dsin<real>(x);
    }
    V = v * s;
    dV = dv * s + v * ds;
}

template <typename real, int L, int THREADS>
__device__ __forceinline__ void bwd_radial(const Sys &S, const real *__restrict__ C, const Work<real> &W, int block,
                                           int nbFe) {
    bool fe;
    const int l = threadIdx.x % L;
    const int i = live_lanes<L>(S, atom_of_block(S, block, THREADS / L, nbFe, threadIdx.x / L, fe));
    if (i < 0) return;
    const Img R = img_of(S.rep[S.rid[i]]);
    const d4 pi = S.pos[i];
    const real rc = (real)RC_R;
    const int cnt = S.cntR[i], nfe = S.cntFeR[i];
    const size_t ld = S.N;
    const int *row = S.actR + i;
    const real *Fp = W.Fp + (size_t)i * DP;
    // the neighbours' contracted blocks for this atom's species
    const real *nR = W.rcoef + (size_t)(fe ? 0 : 1) * ld * NB, *nS = W.rcoef + (size_t)(fe ? 2 : 3) * ld * NB;
    real F[3] = {0, 0, 0}, h[3] = {0, 0, 0};
    // short-range term: half of every pair's energy goes to E_i; the force of
    // the pair on i is V'(r) rhat_ij (both halves)
    const real *Z = C + M_ZBL;
    const bool zon = Z[11] != real(0);
    const real zr2 = zon ? Z[9] : real(0);
    real esr = 0;
    if (fe && S.mag) {
        real si[3];
        load_spin(S.spin, i, si);
        const real os2 = real(2) * Fp[D_OS];
        if (l == 0) {   // the atom's own terms, once
            h[0] = os2 * si[0];
            h[1] = os2 * si[1];
            h[2] = os2 * si[2];
        }
        // onsite moment-length term a|s|^2 + b|s|^4: its energy and dE/ds
        const RepDev &Rr = S.rep[S.rid[i]];
        if (l == 0 && (Rr.landau_a != 0.0 || Rr.landau_b != 0.0)) {
            const real la = (real)Rr.landau_a, lb = (real)Rr.landau_b;
            const real s2 = si[0] * si[0] + si[1] * si[1] + si[2] * si[2];
            const real kl = real(2) * la + real(4) * lb * s2;
            h[0] += kl * si[0];
            h[1] += kl * si[1];
            h[2] += kl * si[2];
            esr += la * s2 + lb * s2 * s2;
        }
        for (int part = 0; part < 2; part++) {
            real CR[NB], CS[NB];
            contract((C + P_CR) + part * NR * NB, Fp + D_R, NR, CR);
            contract((C + P_CSI) + part * NR * NB, Fp + D_SI, NR, CS);
            const int b = (part ? nfe : 0) + l, e = part ? cnt : nfe;
            int j1_ = b < e ? row[(size_t)b * ld] : 0;
            int j2_ = b + L < e ? row[(size_t)(b + L) * ld] : j1_;
            d4 p1_ = S.pos[j1_];
            for (int s = b; s < e; s += L) {
                const int j = j1_;
                const d4 pj_ = p1_;
                j1_ = j2_;
                p1_ = S.pos[j1_];
                if (s + 2 * L < e) j2_ = row[(size_t)(s + 2 * L) * ld];
                real d[3];
                const real r2 = geom_p(R, pi, pj_, d);
                real r, ir;
                r_and_inv(r2, r, ir);
                const real rh[3] = {d[0] * ir, d[1] * ir, d[2] * ir};
                real f[NB], df[NB];
                radial_basis_d(r, rc, f, df);
                const real dgR = dotk(CR, df);
                const real gS = dotk(CS, f), dgS = dotk(CS, df);
                const real a = si[0] * rh[0] + si[1] * rh[1] + si[2] * rh[2];
                const real radial = dgR + dgS * a * a;
                const real ks = real(2) * gS * a * ir;
                real Gj[3];
                partner_radial(nR, nS, S.mag && part == 0, S.spin, j, r, ir, rh, f, df, Gj);
#pragma unroll
                for (int x = 0; x < 3; x++) {
                    const real G = radial * rh[x] + ks * (si[x] - a * rh[x]);
                    h[x] += real(2) * gS * a * rh[x];
                    F[x] += G - Gj[x];
                }
                if (r < zr2) {
                    real V, dV;
                    short_range(Z, part, r, ir, V, dV);
                    esr += real(0.5) * V;
#pragma unroll
                    for (int x = 0; x < 3; x++) F[x] += dV * rh[x];
                }
            }
        }
    } else {
        for (int part = 0; part < 2; part++) {
            real CR[NB];
            contract((C + P_CR) + ((fe ? 0 : 2) + part) * NR * NB, Fp + D_R, NR, CR);
            const int b = (part ? nfe : 0) + l, e = part ? cnt : nfe;
            int j1_ = b < e ? row[(size_t)b * ld] : 0;
            int j2_ = b + L < e ? row[(size_t)(b + L) * ld] : j1_;
            d4 p1_ = S.pos[j1_];
            for (int s = b; s < e; s += L) {
                const int j = j1_;
                const d4 pj_ = p1_;
                j1_ = j2_;
                p1_ = S.pos[j1_];
                if (s + 2 * L < e) j2_ = row[(size_t)(s + 2 * L) * ld];
                real d[3];
                const real r2 = geom_p(R, pi, pj_, d);
                real r, ir;
                r_and_inv(r2, r, ir);
                const real rh[3] = {d[0] * ir, d[1] * ir, d[2] * ir};
                real f[NB], df[NB];
                radial_basis_d(r, rc, f, df);
                const real g = dotk(CR, df);
                real Gj[3];
                partner_radial(nR, nS, S.mag && part == 0, S.spin, j, r, ir, rh, f, df, Gj);
#pragma unroll
                for (int x = 0; x < 3; x++) F[x] += g * rh[x] - Gj[x];
                if (r < zr2) {
                    real V, dV;
                    short_range(Z, (fe ? 0 : 2) + part, r, ir, V, dV);
                    esr += real(0.5) * V;
#pragma unroll
                    for (int x = 0; x < 3; x++) F[x] += dV * rh[x];
                }
            }
        }
    }
#pragma unroll
    for (int x = 0; x < 3; x++) {
        F[x] = lane_sum<L>(F[x]);
        h[x] = lane_sum<L>(h[x]);
    }
    esr = lane_sum<L>(esr);
    if (l) return;
    put_pair(W.ownR, (size_t)i, F, h);
    if (esr != real(0)) W.Ei[i] += esr;
}

template <typename real>
__global__ void __launch_bounds__(256) k_bwd_radial(Sys S, const real *__restrict__ C, Work<real> W, int nbFe) {
    bwd_radial<real, 1, 256>(S, C, W, blockIdx.x, nbFe);
}

// Magnetic pair part of the radial-set backward pass: exchange, DMI and
// anisotropic exchange over the spin-carrying neighbours of spin-carrying
// centres, L lanes per atom. The partner's pair energy e_ji has the form of e_ij
// in terms of d_ij (r_hat_ji.(s_j x s_i) = r_hat_ij.(s_i x s_j), and likewise
// for the anisotropic product), so a pair's force on i and field on s_i are
// the formulas of e_ij with the summed coefficients C_i + C_j: no records.
// Sums: F_i and dE/ds_i of these channels.
template <typename real, int L, int THREADS>
__device__ __forceinline__ void bwd_mag(const Sys &S, const Work<real> &W, int block) {
    const int l = threadIdx.x % L;
    const int i0 = block * (THREADS / L) + threadIdx.x / L;
    const int i = live_lanes<L>(S, i0 < S.N_fe ? i0 : -1);
    if (i < 0) return;
    const Img R = img_of(S.rep[S.rid[i]]);
    const d4 pi = S.pos[i];
    const real rc = (real)RC_R;
    const int nfe = min(S.cntFeR[i], MAXFE);
    const size_t ld = S.N;
    const int *row = S.actR + i;
    real F[3] = {0, 0, 0}, h[3] = {0, 0, 0};
    real si[3];
    load_spin(S.spin, i, si);
    real Ci[3 * NB];
    {
        const real *m = W.mcoef + (size_t)i * MCOEF;
#pragma unroll
        for (int k = 0; k < 3 * NB; k++) Ci[k] = m[k];
    }
    // neighbour index two slots ahead, its position and spin one slot ahead
    int j1_ = l < nfe ? row[(size_t)l * ld] : 0;
    int j2_ = l + L < nfe ? row[(size_t)(l + L) * ld] : j1_;
    d4 p1_ = S.pos[j1_], v1_ = S.spin[j1_];
    for (int s = l; s < nfe; s += L) {
        const int j = j1_;
        const d4 pj_ = p1_, vj_ = v1_;
        j1_ = j2_;
        p1_ = S.pos[j1_];
        v1_ = S.spin[j1_];
        if (s + 2 * L < nfe) j2_ = row[(size_t)(s + 2 * L) * ld];
        real d[3];
        const real r2 = geom_p(R, pi, pj_, d);
        real r, ir;
        r_and_inv(r2, r, ir);
        const real rh[3] = {d[0] * ir, d[1] * ir, d[2] * ir};
        real f[NB], df[NB];
        radial_basis_d(r, rc, f, df);
        const real *mj = W.mcoef + (size_t)j * MCOEF;
        real CE[NB], CD[NB], CA[NB];
#pragma unroll
        for (int k = 0; k < NB; k++) {
            CE[k] = Ci[k] + mj[k];
            CD[k] = Ci[NB + k] + mj[NB + k];
            CA[k] = Ci[2 * NB + k] + mj[2 * NB + k];
        }
        const real sj[3] = {(real)vj_.x, (real)vj_.y, (real)vj_.z};
        const real gE = dotk(CE, f), dgE = dotk(CE, df);
        const real gD = dotk(CD, f), dgD = dotk(CD, df);
        const real gA = dotk(CA, f), dgA = dotk(CA, df);
        const real ss = si[0] * sj[0] + si[1] * sj[1] + si[2] * sj[2];
        const real c[3] = {si[1] * sj[2] - si[2] * sj[1], si[2] * sj[0] - si[0] * sj[2],
                           si[0] * sj[1] - si[1] * sj[0]};
        const real w = rh[0] * c[0] + rh[1] * c[1] + rh[2] * c[2];
        const real a = si[0] * rh[0] + si[1] * rh[1] + si[2] * rh[2];
        const real b = sj[0] * rh[0] + sj[1] * rh[1] + sj[2] * rh[2];
        const real radial = dgE * ss + dgD * w + dgA * a * b;
        const real sjxr[3] = {sj[1] * rh[2] - sj[2] * rh[1], sj[2] * rh[0] - sj[0] * rh[2],
                              sj[0] * rh[1] - sj[1] * rh[0]};
        const real kd = gD * ir, ka = gA * ir;
#pragma unroll
        for (int x = 0; x < 3; x++) {
            const real pa = si[x] - a * rh[x], pb = sj[x] - b * rh[x];
            F[x] += radial * rh[x] + kd * (c[x] - w * rh[x]) + ka * (b * pa + a * pb);
            h[x] += gE * sj[x] + gD * sjxr[x] + gA * b * rh[x];
        }
    }
#pragma unroll
    for (int x = 0; x < 3; x++) {
        F[x] = lane_sum<L>(F[x]);
        h[x] = lane_sum<L>(h[x]);
    }
    if (l == 0) put_pair(W.ownM, (size_t)i, F, h);
}

template <typename real>
__global__ void __launch_bounds__(256) k_bwd_mag(Sys S, Work<real> W) {
    bwd_mag<real, 1, 256>(S, W, blockIdx.x);
}

// -------------------------------------------------------------------------
// backward: angular set
//   q^A_nl = sum_m A_nlm^2, q^sa_nl = sum_m A_nlm B_nlm with
//   A_nlm = sum_j g^A_n Y_lm(rhat_ij), B_nlm = sum_j g^sa_n (s_i.s_j) Y_lm(rhat_ij)
//   dE_i/dd_ij = sum_lm [QA_lm d(g^A Y)/dd + (s_i.s_j) QS_lm d(g^sa Y)/dd]
//   with QA_nlm = 2 Fp^A_nl A_nlm + Fp^sa_nl B_nlm, QS_nlm = Fp^sa_nl A_nlm;
//   h_ij = sum_lm Y_lm sum_n QS_nlm g^sa_n, so that dE_i/ds_j = h_ij s_i and
//   the pair adds h_ij s_j to dE_i/ds_i.
// A wavefront takes eight atoms, whose 336 QA/QS values each sit in LDS, and
// their pairs 64 at a time, a lane per pair in full. A pair record holds
// (dE_i/dd_ij, h_ij).
// -------------------------------------------------------------------------

// What bounds it: FP64 issue and the LDS reads of QA/QS (14 per harmonic and
// pair), both per lane slot, and the load latencies at the start. With the
// neighbours dealt eight per atom and round from the Verlet rows only 60 % of the
// slots held a pair inside the cutoff; the flat in-cutoff pairs fill 90 %:
// 2,097,152 atoms, FP64, carriers 4.45 -> 3.49 ms per launch, the others 2.75 -> 2.10;
// 1,048,576 atoms, FP32, 1.23 -> 0.98 and 0.91 -> 0.63 ms. With the prologue's
// loads issued together and the spins loaded a round ahead: 2.82 and 1.78 ms;
// 0.72 and 0.48 ms.

// Each species runs as its own launch over atoms [first, last). Atoms without
// spin work (the second species, or every atom of a structural-only model)
// keep no QS block, so that twice as many of their workgroups fit in a CU's
// LDS.
template <bool FE>
constexpr int qstride() { return (FE ? 2 : 1) * NA * NLM + 1; }

template <typename real, bool FE>
__device__ __forceinline__ void bwd_angular(const Sys &S, const real *__restrict__ C, const Work<real> &W, int first,
                                            int last, int block, real *sQ, double *sAt) {
    constexpr int QSTRIDE = qstride<FE>();
    const int tid = threadIdx.x, lane = tid & 7, slot = tid >> 3;
    const bool fe = first < S.N_fe;    // species 0: the pair types tau = 0, 1
    const int i0 = first + block * ANG_ATOMS;
    // every load of the prologue before the first use of one: a wavefront has
    // four rounds, and the latency of a chain of loads costs as much as one
    const int ii = min(i0 + slot, last - 1);
    const int cnt_i = S.cntA[ii], nfe_i = S.cntFeA[ii];
    AtomStage as;
    as.load(S, S.spin, ii, lane);
    constexpr int QL = NA * NLM / 8;     // this lane's harmonics: 8 (k % 3) + lane of n = k / 3
    real av[QL], bv[FE ? QL : 1];
    {
        const real *ab = W.AB + (size_t)ii * NA * NAB + lane;
#pragma unroll
        for (int k = 0; k < QL; k++) {
            av[k] = ab[k / 3 * NAB + 8 * (k % 3)];
            if (FE) bv[k] = ab[k / 3 * NAB + NLM + 8 * (k % 3)];
        }
    }
    const int i = i0 + slot < last && as.active ? ii : -1;
    const int cnt = i >= 0 ? cnt_i : 0, nfe = i >= 0 ? nfe_i : 0;
    const real rc = (real)RC_A;
    const size_t ld = S.N;
    real Fo[3] = {0, 0, 0}, ho[3] = {0, 0, 0};     // own-side sums of this lane's pairs
    // the next pair of this lane, loaded one round ahead
    Flat8 fl;
    int pn = 0, rn = 0;                            // its part and the first pair of its round
    fl.set(nfe);
    int off0 = fl.own(slot), off1 = 0;
    int na = -1, nj = 0, nsr = 0;
    d4 np = {0, 0, 0, 0}, ns = {0, 0, 0, 0};
    auto next = [&]() {
        na = -1;
        if (rn >= fl.off[ANG_ATOMS] && pn == 0) {
            pn = 1;
            rn = 0;
            fl.set(cnt - nfe);
            off1 = fl.own(slot);
        }
        if (rn >= fl.off[ANG_ATOMS]) return;       // no round left
        const int p = rn + tid;
        int o;
        const int q = fl.find(p, o), lead = __shfl(nfe, 8 * q);
        if (p < fl.off[ANG_ATOMS]) {
            na = q;
            const size_t x = (size_t)(i0 + na) * MAXA + (p - o) + (pn ? lead : 0);
            nj = S.actA[x];
            nsr = S.actS[x];
            np = S.pos[nj];
            if (FE && pn == 0) ns = S.spin[nj];
        }
    };
    next();
    if (i >= 0) {
        real *Q = sQ + slot * QSTRIDE;   // QA[n][m], then QS[n][m] on spin carriers
        const real *Fp = W.Fp + (size_t)i * DP;
        const int l3[3] = {l_of_lm(lane) - 1, l_of_lm(8 + lane) - 1, l_of_lm(16 + lane) - 1};
#pragma unroll
        for (int k = 0; k < QL; k++) {
            const int x = 8 * k + lane, nl = 4 * (k / 3) + l3[k % 3];
            if (FE) {
                const real fa = Fp[D_A + nl], fs = Fp[D_SA + nl];
                Q[x] = real(2) * fa * av[k] + fs * bv[k];
                Q[NA * NLM + x] = fs * av[k];
            } else {
                Q[x] = real(2) * Fp[D_A + nl] * av[k];
            }
        }
        as.put(lane, sAt + slot * AT_W);
    }
    __syncthreads();
    // rounds of 64 pairs of the eight atoms, spin-carrying neighbours first
#pragma unroll 1
    while (rn < fl.off[ANG_ATOMS]) {
        const int part = pn, r0 = rn, T = fl.off[ANG_ATOMS];
        const int a = na, j = nj, sr = nsr;
        const d4 pj = np, vj = ns;
        rn += 64;
        next();
        const int tau = (fe ? 0 : 2) + part;
        const real *cA = C + P_CA + tau * NA * NB, *cS = C + P_CSA + tau * NA * NB;
        const bool spins = FE && part == 0;
        real G0 = 0, G1 = 0, G2 = 0, hs = 0, sj[3] = {0, 0, 0};
        if (a >= 0) {
            const double *at = sAt + a * AT_W;
            real d[3];
            const real r2 = geom_lds(at, pj, d);
            real r, ir;
            r_and_inv(r2, r, ir);
            const real rh[3] = {d[0] * ir, d[1] * ir, d[2] * ir};
            real f[NB], df[NB];
            radial_basis_d(r, rc, f, df);
            real sig = 0;
            if (spins) {
                sj[0] = (real)vj.x;
                sj[1] = (real)vj.y;
                sj[2] = (real)vj.z;
                sig = (real)at[3] * sj[0] + (real)at[4] * sj[1] + (real)at[5] * sj[2];
            }
            real gA[NA], dgA[NA], gS[NA], dgS[NA];
#pragma unroll
            for (int n = 0; n < NA; n++) {
                gA[n] = dotc(cA + n * NB, f);
                dgA[n] = dotc(cA + n * NB, df);
                gS[n] = spins ? dotc(cS + n * NB, f) : real(0);
                dgS[n] = spins ? dotc(cS + n * NB, df) : real(0);
            }
            real sv = 0, sl = 0, su0 = 0, su1 = 0, su2 = 0;
            // straight-line over the 24 harmonics; the register fence before
            // each one keeps the compiler from evaluating all of them at once
            static_for<NLM>([&](auto M) {
                constexpr int m = decltype(M)::value;
                real Y, gx, gy, gz;
                real hx = rh[0], hy = rh[1], hz = rh[2];
                int qo = a * QSTRIDE;
                asm volatile("" : "+v"(hx), "+v"(hy), "+v"(hz), "+v"(qo), "+v"(sv), "+v"(sl), "+v"(hs), "+v"(su0),
                             "+v"(su1), "+v"(su2));
                const real *Qm = sQ + qo;
                harmonic_one<m>(hx, hy, hz, Y, gx, gy, gz);
                real qa_g = 0, qa_dg = 0, qs_g = 0, qs_dg = 0;
#pragma unroll
                for (int n = 0; n < NA; n++) {
                    const real qa = Qm[n * NLM + m];
                    qa_g += qa * gA[n];
                    qa_dg += qa * dgA[n];
                }
                if (FE && spins) {
#pragma unroll
                    for (int n = 0; n < NA; n++) {
                        const real qs = Qm[NA * NLM + n * NLM + m];
                        qs_g += qs * gS[n];
                        qs_dg += qs * dgS[n];
                    }
                }
                const real U = qa_g + sig * qs_g, V = qa_dg + sig * qs_dg;
                sv += V * Y;
                sl += real(l_of_lm(m)) * U * Y;
                hs += qs_g * Y;
                su0 += U * gx;
                su1 += U * gy;
                su2 += U * gz;
            });
            G0 = sv * rh[0] + (su0 - sl * rh[0]) * ir;
            G1 = sv * rh[1] + (su1 - sl * rh[1]) * ir;
            G2 = sv * rh[2] + (su2 - sl * rh[2]) * ir;
            // the record goes where the partner's gather reads it
            real *rec = W.pbA + ((size_t)(sr >> 8) * ld + j) * 4;
            rec[0] = G0;
            rec[1] = G1;
            rec[2] = G2;
            rec[3] = hs;
        }
        // Own sums: lane l of an atom takes its pairs of rank l modulo 8 (ranks
        // over both parts) from the lanes that formed them, so the order of
        // the sum does not depend on which atoms share the wavefront.
        const int n = part ? cnt - nfe : nfe, mo = part ? off1 : off0;
        const int lo = max(r0 - mo, 0), hi = min(n, min(r0 + 64, T) - mo);   // this round's ranks of the atom
        int r = lo + ((lane - (part ? nfe : 0) - lo) & 7);
        while (__any(r < hi)) {
            const bool ok = r < hi;
            const int src = ok ? mo + r - r0 : tid;
            const real x0 = __shfl(G0, src), x1 = __shfl(G1, src), x2 = __shfl(G2, src);
            if (ok) {
                Fo[0] += x0;
                Fo[1] += x1;
                Fo[2] += x2;
            }
            if (spins) {
                const real y0 = __shfl(hs * sj[0], src), y1 = __shfl(hs * sj[1], src), y2 = __shfl(hs * sj[2], src);
                if (ok) {
                    ho[0] += y0;
                    ho[1] += y1;
                    ho[2] += y2;
                }
            }
            r += 8;
        }
    }
    // own-side sums over the atom's eight lanes (fixed xor tree)
#pragma unroll
    for (int x = 0; x < 3; x++) {
        Fo[x] = lane_sum<8>(Fo[x]);
        ho[x] = lane_sum<8>(ho[x]);
    }
    if (lane == 0 && i >= 0) put_pair(W.ownA, (size_t)i, Fo, ho);
}

template <typename real, bool FE>
__global__ void __launch_bounds__(64) k_bwd_angular(Sys S, const real *__restrict__ C, Work<real> W, int first,
                                                    int last) {
    __shared__ real sQ[ANG_ATOMS * qstride<FE>()];
    __shared__ double sAt[ANG_ATOMS * AT_W];
    bwd_angular<real, FE>(S, C, W, first, last, blockIdx.x, sQ, sAt);
}

// The whole backward pass of a batch with wide replicas: the angular set of
// both species and, of the wide replicas, the radial set and the magnetic pairs,
// which do not depend on each other, in blocks of eight atoms (see k_desc_both):
// nb of them for all atoms; the first na of the grid are the angular set's, those
// before nbA of species 0 (na = nb, nbA = nbFe: everything; na = 0: the radial
// set alone; nbA = 0: species 1 and what follows).
template <typename real, bool MAG>
__global__ void __launch_bounds__(64, 2) k_bwd_both(Sys S, const real *__restrict__ C, Work<real> W, int nbA, int na,
                                                    int nbFe, int nb) {
    __shared__ real sQ[ANG_ATOMS * qstride<MAG>()];
    __shared__ double sAt[ANG_ATOMS * AT_W];
    int b = blockIdx.x;
    if (b < nbA) return bwd_angular<real, MAG>(S, C, W, 0, S.N_fe, b, sQ, sAt);
    if (b < na) return bwd_angular<real, false>(S, C, W, S.N_fe, S.N, b - nbA, sQ, sAt);
    b -= na;
    if (b < nb) return bwd_radial<real, WIDE_LANES, 64>(S, C, W, b, nbFe);
    if constexpr (MAG) bwd_mag<real, WIDE_LANES, 64>(S, W, b - nb);
}

// -------------------------------------------------------------------------
// gather: forces and fields
// -------------------------------------------------------------------------

// Eight lanes per atom over its in-cutoff pairs, rank modulo 8, then a fixed
// xor tree: the partner records sit in the atom's own slots.
template <typename real>
__global__ void __launch_bounds__(256) k_gather(Sys S, Work<real> W) {
    const int lane = threadIdx.x & 7;
    const int k0 = blockIdx.x * 32 + (threadIdx.x >> 3);
    const int k = live(S, k0 < S.N ? k0 : -1);   // a paused replica keeps its last forces and fields
    if (k < 0) return;
    const size_t ld = S.N;
    const bool fe = S.mag && k < S.N_fe;   // spin carrier
    const int na = S.cntA[k], nfe = fe ? S.cntFeA[k] : 0;
    real F[3] = {0, 0, 0}, h[3] = {0, 0, 0};
    for (int s = lane; s < na; s += 8) {
        const real *p = W.pbA + ((size_t)(S.actS[(size_t)k * MAXA + s] & 0xff) * ld + k) * 4;
        F[0] -= p[0];
        F[1] -= p[1];
        F[2] -= p[2];
        if (s < nfe) {
            real sj[3];
            load_spin(S.spin, S.actA[(size_t)k * MAXA + s], sj);
            h[0] += p[3] * sj[0];
            h[1] += p[3] * sj[1];
            h[2] += p[3] * sj[2];
        }
    }
#pragma unroll
    for (int x = 0; x < 3; x++) {
        F[x] = lane_sum<8>(F[x]);
        h[x] = lane_sum<8>(h[x]);
    }
    if (lane >= 3) return;   // lanes 0-2 finish one component each
    real Fx = lane == 0 ? F[0] : lane == 1 ? F[1] : F[2], hx = lane == 0 ? h[0] : lane == 1 ? h[1] : h[2];
    const real *aR = W.ownR + (size_t)k * 6, *aA = W.ownA + (size_t)k * 6;
    Fx += aR[lane] + aA[lane];
    hx += aR[3 + lane] + aA[3 + lane];
    if (fe) {
        const real *aM = W.ownM + (size_t)k * 6;
        Fx += aM[lane];
        hx += aM[3 + lane];
    }
    (&S.force[k].x)[lane] = (double)Fx;
    double H = 0;
    if (fe) {
        const RepDev &R = S.rep[S.rid[k]];
        H = -(double)hx + R.mu_s * MUB * (R.B0[lane] + (R.B1[lane] - R.B0[lane]) * ramp_frac(R));
    }
    (&S.field[k].x)[lane] = H;
}

// -------------------------------------------------------------------------
// spin couplings of the frozen-Fp magnetic energy
//   E_lin = sum_i sum_j [a_ij s_i.s_j + d_ij rhat_ij.(s_i x s_j) + b_ij (s_i.rhat)(s_j.rhat)]
//           + sum_i s_i^T A_i s_i + o_i |s_i|^2  (+ Zeeman)
// -------------------------------------------------------------------------

// spin-angular part of a_ij: sum_n g^sa_n(r_ij) sum_lm Fp^sa_nl A_nlm Y_lm(rhat_ij);
// a lane per pair of the wavefront's eight spins, P = Fp^sa A in LDS. Two rounds
// of pairs per wavefront: its time is that of the prologue's loads, issued
// together (2,097,152 atoms, FP64: 1.02 -> 0.66 ms; 262,144: 146 -> 90 us).
constexpr int PSTRIDE = NA * NLM + 1;

template <typename real>
__global__ void __launch_bounds__(64) k_assemble_angular(Sys S, const real *__restrict__ C, Work<real> W) {
    __shared__ real sP[ANG_ATOMS * PSTRIDE];
    __shared__ double sAt[ANG_ATOMS * AT_W];
    const int tid = threadIdx.x, lane = tid & 7, slot = tid >> 3;
    const int i0 = blockIdx.x * ANG_ATOMS;
    const int ii = min(i0 + slot, S.N_fe - 1);
    const int nfe_i = S.cntFeA[ii];     // the prologue's loads together, as in the backward pass
    AtomStage as;
    as.load(S, S.spin, ii, lane);
    constexpr int QL = NA * NLM / 8;
    real av[QL];
    {
        const real *ab = W.AB + (size_t)ii * NA * NAB + lane;
#pragma unroll
        for (int k = 0; k < QL; k++) av[k] = ab[k / 3 * NAB + 8 * (k % 3)];
    }
    const int i = i0 + slot < S.N_fe && as.active ? ii : -1;
    const int nfe = i >= 0 ? nfe_i : 0;
    const real *cS = C + P_CSA;   // tau = (Fe, Fe)
    const real rc = (real)RC_A;
    const size_t lf = S.N_fe;
    Flat8 fl;
    fl.set(nfe);
    // this lane's next pair, loaded one round ahead
    int na = -1, ns = 0;
    d4 np = {0, 0, 0, 0};
    auto next = [&](int p) {
        na = -1;
        if (p < fl.off[ANG_ATOMS]) {
            int o;
            na = fl.find(p, o);
            const size_t x = (size_t)(i0 + na) * MAXA + (p - o);
            ns = S.actS[x] & 0xff;
            np = S.pos[S.actA[x]];
        }
    };
    next(tid);
    if (i >= 0) {
        real *P = sP + slot * PSTRIDE;
        const real *Fp = W.Fp + (size_t)i * DP + D_SA;
        const int l3[3] = {l_of_lm(lane) - 1, l_of_lm(8 + lane) - 1, l_of_lm(16 + lane) - 1};
#pragma unroll
        for (int k = 0; k < QL; k++) P[8 * k + lane] = Fp[4 * (k / 3) + l3[k % 3]] * av[k];
        as.put(lane, sAt + slot * AT_W);
    }
    __syncthreads();
#pragma unroll 1
    for (int r0 = 0; r0 < fl.off[ANG_ATOMS]; r0 += 64) {
        const int at = na, s = ns;
        const d4 pj = np;
        next(r0 + 64 + tid);
        if (at < 0) continue;
        real d[3];
        const real r2 = geom_lds(sAt + at * AT_W, pj, d);
        real r, ir;
        r_and_inv(r2, r, ir);
        real f[NB];
        radial_basis(r, rc, f);
        real gS[NA];
#pragma unroll
        for (int n = 0; n < NA; n++) gS[n] = dotc(cS + n * NB, f);
        real a = 0;
        real Y[NLM];
        harmonics(d[0] * ir, d[1] * ir, d[2] * ir, Y);
        const real *P = sP + at * PSTRIDE;
#pragma unroll
        for (int m = 0; m < NLM; m++) {
            real w = 0;
#pragma unroll
            for (int n = 0; n < NA; n++) w += P[n * NLM + m] * gS[n];
            a += w * Y[m];
        }
        // angular slots of spin carriers lead, so s < MAXFE, but for a row that
        // overflowed in this step, which is void only at its end
        if (s < MAXFE) W.csa[(size_t)s * lf + i0 + at] = a;
    }
}

// Couplings of the spin-carrying pairs inside rc_R, J_ij = a_ij + a_ji,
// D_ij = d_ij + d_ji, K_ij = b_ij + b_ji: the radial-set parts are sums over
// the basis with the summed contracted coefficients of both spins, the
// spin-angular parts (inside rc_A) the two atoms' records. Stored with rhat_ij
// by in-cutoff rank, so the sweep's split of a spin's couplings over lanes
// depends on the positions alone and not on which farther atoms the Verlet list
// happens to hold. The same pass sums the single-ion tensor
// A_i = sum_j g^si(r_ij) rhat rhat^T over all neighbours.
template <typename real, int L>
__global__ void __launch_bounds__(256) k_assemble_pairs(Sys S, const real *__restrict__ C, Work<real> W) {
    const int l = threadIdx.x % L;
    const int i0 = blockIdx.x * (256 / L) + threadIdx.x / L;
    const int i = live_lanes<L>(S, i0 < S.N_fe ? i0 : -1);
    if (i < 0) return;
    const Img R = img_of(S.rep[S.rid[i]]);
    const d4 pi = S.pos[i];
    const real rc = (real)RC_R, near2 = (real)((RC_A + 0.01) * (RC_A + 0.01));
    const int cnt = S.cntR[i], nfe_all = S.cntFeR[i], nfe = min(nfe_all, MAXFE);
    const size_t ld = S.N, lf = S.N_fe;
    const int *row = S.actR + i;
    const int p = S.colpos[i];
    const real *Fp = W.Fp + (size_t)i * DP;
    real Ci[MCOEF];
    {
        const real *m = W.mcoef + (size_t)i * MCOEF;
#pragma unroll
        for (int k = 0; k < MCOEF; k++) Ci[k] = m[k];
    }
    real Axx = 0, Ayy = 0, Azz = 0, Axy = 0, Axz = 0, Ayz = 0;
    {
        real CS[NB];
        contract((C + P_CSI), Fp + D_SI, NR, CS);
        // neighbour index two slots ahead, its position one slot ahead
        int j1 = l < nfe ? row[(size_t)l * ld] : 0;
        int j2 = l + L < nfe ? row[(size_t)(l + L) * ld] : j1;
        d4 p1 = S.pos[j1];
        for (int s = l; s < nfe; s += L) {
            const int j = j1;
            const d4 pj = p1;
            j1 = j2;
            p1 = S.pos[j1];
            if (s + 2 * L < nfe) j2 = row[(size_t)(s + 2 * L) * ld];
            real d[3];
            const real r2 = geom_p(R, pi, pj, d);
            real r, ir;
            r_and_inv(r2, r, ir);
            const real rh[3] = {d[0] * ir, d[1] * ir, d[2] * ir};
            real f[NB];
            radial_basis(r, rc, f);
            const real *mj = W.mcoef + (size_t)j * MCOEF;
            real J = 0, D = 0, K = 0;
#pragma unroll
            for (int k = 0; k < NB; k++) {
                J += (Ci[k] + mj[k]) * f[k];
                D += (Ci[NB + k] + mj[NB + k]) * f[k];
                K += (Ci[2 * NB + k] + mj[2 * NB + k]) * f[k];
            }
            // whether a pair is inside rc_A was decided once, for its list entry;
            // the distance only saves the farther ones the look
            if (r2 < near2) {
                const int a = S.xS[(size_t)s * lf + i];
                if (a != NO_RECORD) J += W.csa[(size_t)(a & 0xff) * lf + i] + W.csa[(size_t)(a >> 8) * lf + j];
            }
            const real g = dotk(CS, f);
            Axx += g * rh[0] * rh[0];
            Ayy += g * rh[1] * rh[1];
            Azz += g * rh[2] * rh[2];
            Axy += g * rh[0] * rh[1];
            Axz += g * rh[0] * rh[2];
            Ayz += g * rh[1] * rh[2];
            real *c = W.cpl + ((size_t)s * lf + p) * 6;
            c[0] = J;
            c[1] = D;
            c[2] = K;
            c[3] = rh[0];
            c[4] = rh[1];
            c[5] = rh[2];
            W.cpl_j[(size_t)s * lf + p] = j;
        }
    }
    {
        real CS[NB];
        contract((C + P_CSI) + 1 * NR * NB, Fp + D_SI, NR, CS);
        const int b = nfe_all + l;
        int j1 = b < cnt ? row[(size_t)b * ld] : 0;
        int j2 = b + L < cnt ? row[(size_t)(b + L) * ld] : j1;
        d4 p1 = S.pos[j1];
        for (int s = b; s < cnt; s += L) {
            const d4 pj = p1;
            j1 = j2;
            p1 = S.pos[j1];
            if (s + 2 * L < cnt) j2 = row[(size_t)(s + 2 * L) * ld];
            real d[3];
            const real r2 = geom_p(R, pi, pj, d);
            real r, ir;
            r_and_inv(r2, r, ir);
            const real rh[3] = {d[0] * ir, d[1] * ir, d[2] * ir};
            real f[NB];
            radial_basis(r, rc, f);
            const real g = dotk(CS, f);
            Axx += g * rh[0] * rh[0];
            Ayy += g * rh[1] * rh[1];
            Azz += g * rh[2] * rh[2];
            Axy += g * rh[0] * rh[1];
            Axz += g * rh[0] * rh[2];
            Ayz += g * rh[1] * rh[2];
        }
    }
    Axx = lane_sum<L>(Axx);
    Ayy = lane_sum<L>(Ayy);
    Azz = lane_sum<L>(Azz);
    Axy = lane_sum<L>(Axy);
    Axz = lane_sum<L>(Axz);
    Ayz = lane_sum<L>(Ayz);
    if (l) return;
    real *o = W.selfc + (size_t)p * 8;
    o[0] = Axx;
    o[1] = Ayy;
    o[2] = Azz;
    o[3] = Axy;
    o[4] = Axz;
    o[5] = Ayz;
    o[6] = Fp[D_OS];
    o[7] = 0;
    W.cpl_n[p] = nfe;
}

inline int nblk(int n, int b) { return (n + b - 1) / b; }

}  // namespace

#define NEP_SPLIT(per)                                  \
    const int ge = S.N - S.N_fe;                        \
    const int nb_fe = nblk(S.N_fe, per), nb_ge = nblk(ge, per);

template <typename real>
void launch_active(const Sys &S, int mode, hipStream_t st) {
    const int n = mode == PASS_FULL ? S.N : S.N_fe;
    if (n) hipLaunchKernelGGL(k_active<real>, dim3(nblk(n, 32)), dim3(256), 0, st, S, n);
}

// The launches that wide replicas share: everything at once, or where their
// groups are timed (S.apart) each group's own blocks. The kernel is the same, and
// so are the bits.
template <typename real>
void bwd_both(const Sys &S, const ModelDev<real> &M, const Work<real> &W, int blocks, int nbA, int na, int nb_fe, int nb,
              hipStream_t st) {
    if (!blocks) return;
    const dim3 g(blocks), t(8 * ANG_ATOMS);
    if (S.mag) hipLaunchKernelGGL((k_bwd_both<real, true>), g, t, 0, st, S, M.cR, W, nbA, na, nb_fe, nb);
    else hipLaunchKernelGGL((k_bwd_both<real, false>), g, t, 0, st, S, M.cR, W, nbA, na, nb_fe, nb);
}

// spin-step passes (PASS_SPIN, PASS_SPIN_REUSE) cover the spin carriers only:
// the frozen-Fp magnetic energy has no term on atoms without a spin
template <typename real>
void launch_desc_radial(const Sys &S, const ModelDev<real> &M, const Work<real> &W, const d4 *spin, int mode,
                        hipStream_t st) {
    if (S.N == 0) return;
    if (S.narrow) {
        NEP_SPLIT(256)
        const int nb = mode == PASS_FULL ? nb_fe + nb_ge : nb_fe;
        if (nb) hipLaunchKernelGGL(k_desc_radial<real>, dim3(nb), dim3(256), 0, st, S, M.cR, W, spin, nb_fe);
    }
    if (S.wide && S.apart) {
        NEP_SPLIT(ANG_ATOMS)
        const int nb = mode == PASS_FULL ? nb_fe + nb_ge : nb_fe;
        if (nb)
            hipLaunchKernelGGL(k_desc_both<real>, dim3(nb), dim3(8 * ANG_ATOMS), 0, st, S, M.cR, W, spin, nb_fe, 0, mode);
    }
}

template <typename real>
void launch_desc_angular(const Sys &S, const ModelDev<real> &M, const Work<real> &W, const d4 *spin, int mode,
                         hipStream_t st) {
    if (S.N == 0) return;
    NEP_SPLIT(ANG_ATOMS)
    const int nb = mode == PASS_FULL ? nb_fe + nb_ge : nb_fe;
    if (!nb) return;
    if (S.wide)
        hipLaunchKernelGGL(k_desc_both<real>, dim3(S.apart ? nb : 2 * nb), dim3(8 * ANG_ATOMS), 0, st, S, M.cR, W, spin,
                           nb_fe, nb, mode);
    else
        hipLaunchKernelGGL(k_desc_angular<real>, dim3(nb), dim3(8 * ANG_ATOMS), 0, st, S, M.cR, W, spin, nb_fe, mode);
}

template <typename real>
void launch_mlp(const Sys &S, const ModelDev<real> &M, const Work<real> &W, int mode, hipStream_t st) {
    if (S.N == 0) return;
    const int t_fe = nblk(S.N_fe, 16), tiles = mode == PASS_FULL ? t_fe + nblk(S.N - S.N_fe, 16) : t_fe;
    if (!tiles) return;
    if (tiles <= MLP_SPLIT_TILES) {
        const int nb_fe = t_fe;
        const dim3 g(tiles), b(256);
        if (!S.mag) hipLaunchKernelGGL((k_mlp<real, DS_PAD, false, true>), g, b, 0, st, S, M, W, nb_fe);
        else if (mode == PASS_FULL) hipLaunchKernelGGL((k_mlp<real, DP, false, true>), g, b, 0, st, S, M, W, nb_fe);
        else hipLaunchKernelGGL((k_mlp<real, DP, true, true>), g, b, 0, st, S, M, W, nb_fe);
        return;
    }
    NEP_SPLIT(MLP_ATOMS)
    const int nb = mode == PASS_FULL ? nb_fe + nb_ge : nb_fe;
    const dim3 g(nb), b(64 * MLP_WAVES);
    if (!S.mag) hipLaunchKernelGGL((k_mlp<real, DS_PAD, false, false>), g, b, 0, st, S, M, W, nb_fe);
    else if (mode == PASS_FULL) hipLaunchKernelGGL((k_mlp<real, DP, false, false>), g, b, 0, st, S, M, W, nb_fe);
    else hipLaunchKernelGGL((k_mlp<real, DP, true, false>), g, b, 0, st, S, M, W, nb_fe);
}

template <typename real>
void launch_bwd_radial(const Sys &S, const ModelDev<real> &M, const Work<real> &W, hipStream_t st) {
    if (S.N == 0) return;
    if (S.narrow) {
        NEP_SPLIT(256)
        hipLaunchKernelGGL(k_bwd_radial<real>, dim3(nb_fe + nb_ge), dim3(256), 0, st, S, M.cR, W, nb_fe);
        if (nb_fe && S.mag) hipLaunchKernelGGL(k_bwd_mag<real>, dim3(nb_fe), dim3(256), 0, st, S, W);
    }
    if (S.wide && S.apart) {
        NEP_SPLIT(ANG_ATOMS)
        const int nb = nb_fe + nb_ge;
        bwd_both(S, M, W, nb + (S.mag ? nb_fe : 0), 0, 0, nb_fe, nb, st);
    }
}

template <typename real>
void launch_bwd_angular(const Sys &S, const ModelDev<real> &M, const Work<real> &W, int species, hipStream_t st) {
    if (S.N == 0) return;
    NEP_SPLIT(ANG_ATOMS)
    if (S.wide) {
        const int nb = nb_fe + nb_ge;
        if (S.apart && species) bwd_both(S, M, W, nb_ge, 0, nb_ge, nb_fe, nb, st);
        else if (S.apart) bwd_both(S, M, W, nb_fe, nb_fe, nb_fe, nb_fe, nb, st);
        else if (!species) bwd_both(S, M, W, 2 * nb + (S.mag ? nb_fe : 0), nb_fe, nb, nb_fe, nb, st);
        return;
    }
    if (species == 0 && nb_fe) {
        if (S.mag)
            hipLaunchKernelGGL((k_bwd_angular<real, true>), dim3(nb_fe), dim3(8 * ANG_ATOMS), 0, st, S, M.cR, W, 0,
                               S.N_fe);
        else
            hipLaunchKernelGGL((k_bwd_angular<real, false>), dim3(nb_fe), dim3(8 * ANG_ATOMS), 0, st, S, M.cR, W, 0,
                               S.N_fe);
    }
    if (species == 1 && nb_ge)
        hipLaunchKernelGGL((k_bwd_angular<real, false>), dim3(nb_ge), dim3(8 * ANG_ATOMS), 0, st, S, M.cR, W, S.N_fe,
                           S.N);
}

template <typename real>
void launch_gather(const Sys &S, const Work<real> &W, hipStream_t st) {
    if (S.N == 0) return;
    hipLaunchKernelGGL(k_gather<real>, dim3(nblk(S.N, 32)), dim3(256), 0, st, S, W);
}

template <typename real>
void launch_assemble_coef(const Sys &S, const ModelDev<real> &M, const Work<real> &W, hipStream_t st) {
    if (S.N_fe == 0) return;
    hipLaunchKernelGGL(k_assemble_angular<real>, dim3(nblk(S.N_fe, ANG_ATOMS)), dim3(8 * ANG_ATOMS), 0, st, S, M.cR, W);
}

template <typename real>
void launch_assemble_pairs(const Sys &S, const ModelDev<real> &M, const Work<real> &W, hipStream_t st) {
    if (S.N_fe == 0) return;
    if (S.narrow)
        hipLaunchKernelGGL((k_assemble_pairs<real, 1>), dim3(nblk(S.N_fe, 256)), dim3(256), 0, st, S, M.cR, W);
    if (S.wide)
        hipLaunchKernelGGL((k_assemble_pairs<real, WIDE_LANES>), dim3(nblk(S.N_fe, 256 / WIDE_LANES)), dim3(256), 0, st,
                           S, M.cR, W);
}

#define NEP_INST(real)                                                                                           \
    template void launch_active<real>(const Sys &, int, hipStream_t);                                            \
    template void launch_desc_radial<real>(const Sys &, const ModelDev<real> &, const Work<real> &, const d4 *, \
                                           int, hipStream_t);                                                    \
    template void launch_desc_angular<real>(const Sys &, const ModelDev<real> &, const Work<real> &, const d4 *,\
                                            int, hipStream_t);                                                   \
    template void launch_mlp<real>(const Sys &, const ModelDev<real> &, const Work<real> &, int, hipStream_t);   \
    template void launch_bwd_radial<real>(const Sys &, const ModelDev<real> &, const Work<real> &, hipStream_t); \
    template void launch_bwd_angular<real>(const Sys &, const ModelDev<real> &, const Work<real> &, int, hipStream_t);\
    template void launch_gather<real>(const Sys &, const Work<real> &, hipStream_t);                             \
    template void launch_assemble_coef<real>(const Sys &, const ModelDev<real> &, const Work<real> &, hipStream_t);\
    template void launch_assemble_pairs<real>(const Sys &, const ModelDev<real> &, const Work<real> &, hipStream_t);

NEP_INST(double)
NEP_INST(float)

}  // namespace nep
