// The MD chain: Verlet-list particles and colloids over the n_md steps of an
// interval.  Its instances are compiled in rmp_chain_f64.hip and
// rmp_chain_f32.hip, next to the other kernels, so that the library builds in
// parallel.
#pragma once
#include "rmp_stream.h"

namespace rmp {

// ------------------------------------------------------------- MD chain

__device__ __forceinline__ double shfl_d(double v, int src)
{
    const int lo = __shfl(__double2loint(v), src, 64);
    const int hi = __shfl(__double2hiint(v), src, 64);
    return __hiloint2double(hi, lo);
}

// Bond of the colloid of lane t (t < nc), loaded once per interval
struct BondLane {
    int other;                 // lane of the bond partner (t itself if none)
    bool has, ia;              // has a bond; is its first colloid a
    double dd, ima, imb, mu;   // bond length, inverse masses of a and b, sum
};

__device__ __forceinline__ BondLane bond_lane(const ColloidParams* cp, int nc)
{
    const int t = threadIdx.x & 63;
    BondLane L;
    const int k = t < nc ? cp->bond_of[t] : -1;
    L.has = k >= 0;
    const int a = L.has ? cp->bond_a[k] : t, b = L.has ? cp->bond_b[k] : t;
    L.ia = t == a;
    L.other = L.ia ? b : a;
    L.dd = L.has ? cp->bond_d[k] : 0.0;
    L.ima = L.has ? cp->imass[a] : 0.0;
    L.imb = L.has ? cp->imass[b] : 0.0;
    L.mu = L.ima + L.imb;
    return L;
}

// RATTLE position stage for the colloid of lane t (t < nc, all 64 lanes of
// the wave call it).  Both colloids of a bond evaluate the bond's
// correction from the same operands in the bond's (a, b) order, so they
// agree exactly; Xo are the positions before the drift.
__device__ __forceinline__ void rattle_pos_lane(const BondLane& L, double dt, double (&X)[3], double (&V)[3],
                                                const double (&Xo)[3], uint32_t& flags)
{
    double pXo[3], pX[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        pXo[d] = shfl_d(Xo[d], L.other);
        pX[d] = shfl_d(X[d], L.other);
    }
    if (!L.has) return;
    const bool ia = L.ia;
    double r0[3], sv[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        r0[d] = ia ? Xo[d] - pXo[d] : pXo[d] - Xo[d];
        sv[d] = ia ? X[d] - pX[d] : pX[d] - X[d];
    }
    const double mu = L.mu;
    const double r0r0 = dot3(r0[0], r0[1], r0[2], r0[0], r0[1], r0[2]);
    const double sr0 = dot3(sv[0], sv[1], sv[2], r0[0], r0[1], r0[2]);
    const double ss = dot3(sv[0], sv[1], sv[2], sv[0], sv[1], sv[2]);
    const double A = (mu * mu) * r0r0;
    const double Bh = mu * sr0;
    const double C = ss - (L.dd * L.dd);
    double disc = (Bh * Bh) - (A * C);
    if (disc < 0.0) {
        flags |= RMP_FLAG_RATTLE;
        disc = 0.0;
    }
    const double gq = C / (Bh + sqrt(disc));
    if (ia) {
        const double ga = gq * L.ima;
        const double gad = ga / dt;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            X[d] = X[d] - (ga * r0[d]);
            V[d] = V[d] - (gad * r0[d]);
        }
    } else {
        const double gb = gq * L.imb;
        const double gbd = gb / dt;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            X[d] = X[d] + (gb * r0[d]);
            V[d] = V[d] + (gbd * r0[d]);
        }
    }
}

// Iterative RATTLE (Andersen 1983) for bond networks, by the 64 lanes of
// wave 0 on the colloid state staged in LDS.  Position stage: sweeps over
// the bonds in order; a bond whose squared length s.s misses d^2 by more than
// 2 tol d^2 is corrected along its direction before the drift, r0: both
// colloids move by g r0 / m, g = (d^2 - s.s) / (2 mu s.r0), mu = 1/m_a +
// 1/m_b, and their velocities by the same displacement over dt; until a
// sweep changes nothing, at most rattle_maxit sweeps (else the RATTLE flag).
// A sweep runs layer by layer, a layer being consecutive bonds with no
// colloid in common, one lane per bond: the corrections within a layer
// commute exactly, so the result is that of the bonds one after another.
//
// A layer's lane reads both ends of its bond, their velocities and the
// bond's constants (LDS tables filled once per interval and per stage) in
// one round trip, and writes the results back together; the ends of the
// next layer's bonds are read a layer ahead.
template <class Ctx>
__device__ __forceinline__ uint32_t rattle_pos_iter(Ctx& S, const ColloidParams* cp, double dt)
{
    const int lane = threadIdx.x & 63;
    const int nl = cp->n_layers, nbond = cp->nbonds;
    for (int q = lane; q < nbond; q += 64) {
        const int a = S.sBa[q], b = S.sBb[q];
        for (int d = 0; d < 3; ++d) S.sBr[q][d] = S.sXoc[a][d] - S.sXoc[b][d];
    }
    wave_sync();
    bool moved = true;
    for (int sweep = 0; sweep < cp->rattle_maxit && moved; ++sweep) {
        bool m = false;
        int s0 = S.sLay[0], s1 = nl > 0 ? S.sLay[1] : s0;
        int a = 0, b = 0;
        if (s0 + lane < s1) {
            a = S.sBa[s0 + lane];
            b = S.sBb[s0 + lane];
        }
        for (int L = 0; L < nl; ++L) {
            const int q = s0 + lane;
            const bool act = q < s1;
            // both ends read at once (a != b) with the bond's constants,
            // written back at once
            double xa[3], xb[3], va[3], vb[3], r0[3];
            double dd2 = 0.0, thr = 0.0, mu2 = 0.0, ima = 0.0, imb = 0.0;
            if (act) {
                for (int d = 0; d < 3; ++d) {
                    xa[d] = S.sXc[a][d];
                    xb[d] = S.sXc[b][d];
                    r0[d] = S.sBr[q][d];
                }
                dd2 = S.sBd2[q];
                thr = S.sBthr[q];
                mu2 = S.sBmu2[q];
                ima = S.sBia[q];
                imb = S.sBib[q];
                for (int d = 0; d < 3; ++d) {
                    va[d] = S.sVc[a][d];
                    vb[d] = S.sVc[b][d];
                }
            }
            // ends of the next layer's bonds (unused past its end)
            const int s2 = S.sLay[min(L + 2, nl)];
            const int qn = s1 + lane;
            int na = 0, nb = 0;
            if (qn < nbond) {
                na = S.sBa[qn];
                nb = S.sBb[qn];
            }
            if (act) {
                double sv[3];
                for (int d = 0; d < 3; ++d) sv[d] = xa[d] - xb[d];
                const double ss = dot3(sv[0], sv[1], sv[2], sv[0], sv[1], sv[2]);
                const double diff = dd2 - ss;
                if (fabs(diff) > thr) {
                    const double sr0 = dot3(sv[0], sv[1], sv[2], r0[0], r0[1], r0[2]);
                    const double g = diff / (mu2 * sr0);
                    const double ga = g * ima, gb = g * imb;
                    for (int d = 0; d < 3; ++d) {
                        S.sXc[a][d] = xa[d] + (ga * r0[d]);
                        S.sXc[b][d] = xb[d] - (gb * r0[d]);
                    }
                    const double gad = ga / dt, gbd = gb / dt;
                    for (int d = 0; d < 3; ++d) {
                        S.sVc[a][d] = va[d] + (gad * r0[d]);
                        S.sVc[b][d] = vb[d] - (gbd * r0[d]);
                    }
                    m = true;
                }
            }
            wave_sync();
            s0 = s1;
            s1 = s2;
            a = na;
            b = nb;
        }
        moved = __ballot(m) != 0ull;
    }
    return moved ? RMP_FLAG_RATTLE : 0u;
}

// Iterative RATTLE, velocity stage: sweeps removing the relative velocity
// along each bond, k = (r.v) / (mu d^2), while |r.v| exceeds tol d^2 / dt
// (layer by layer, as above; the bond vectors r are fixed for the stage).
template <class Ctx>
__device__ __forceinline__ uint32_t rattle_vel_iter(Ctx& S, const ColloidParams* cp, double dt)
{
    (void)dt;
    const int lane = threadIdx.x & 63;
    const int nl = cp->n_layers, nbond = cp->nbonds;
    for (int q = lane; q < nbond; q += 64) {
        const int a = S.sBa[q], b = S.sBb[q];
        for (int d = 0; d < 3; ++d) S.sBr[q][d] = S.sXc[a][d] - S.sXc[b][d];
    }
    wave_sync();
    bool moved = true;
    for (int sweep = 0; sweep < cp->rattle_maxit && moved; ++sweep) {
        bool m = false;
        int s0 = S.sLay[0], s1 = nl > 0 ? S.sLay[1] : s0;
        int a = 0, b = 0;
        if (s0 + lane < s1) {
            a = S.sBa[s0 + lane];
            b = S.sBb[s0 + lane];
        }
        for (int L = 0; L < nl; ++L) {
            const int q = s0 + lane;
            const bool act = q < s1;
            double va[3], vb[3], r[3];
            double thv = 0.0, mud = 0.0, ima = 0.0, imb = 0.0;
            if (act) {
                for (int d = 0; d < 3; ++d) {
                    va[d] = S.sVc[a][d];
                    vb[d] = S.sVc[b][d];
                    r[d] = S.sBr[q][d];
                }
                thv = S.sBthv[q];
                mud = S.sBmud[q];
                ima = S.sBia[q];
                imb = S.sBib[q];
            }
            const int s2 = S.sLay[min(L + 2, nl)];
            const int qn = s1 + lane;
            int na = 0, nb = 0;
            if (qn < nbond) {
                na = S.sBa[qn];
                nb = S.sBb[qn];
            }
            if (act) {
                double vr[3];
                for (int d = 0; d < 3; ++d) vr[d] = va[d] - vb[d];
                const double rv = dot3(r[0], r[1], r[2], vr[0], vr[1], vr[2]);
                if (fabs(rv) > thv) {
                    const double k = rv / mud;
                    const double ka = k * ima, kb = k * imb;
                    for (int d = 0; d < 3; ++d) {
                        S.sVc[a][d] = va[d] - (ka * r[d]);
                        S.sVc[b][d] = vb[d] + (kb * r[d]);
                    }
                    m = true;
                }
            }
            wave_sync();
            s0 = s1;
            s1 = s2;
            a = na;
            b = nb;
        }
        moved = __ballot(m) != 0ull;
    }
    return moved ? RMP_FLAG_RATTLE : 0u;
}

// RATTLE velocity stage for the colloid of lane t (same conventions)
__device__ __forceinline__ void rattle_vel_lane(const BondLane& L, const double (&X)[3], double (&V)[3])
{
    double pX[3], pV[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        pX[d] = shfl_d(X[d], L.other);
        pV[d] = shfl_d(V[d], L.other);
    }
    if (!L.has) return;
    const bool ia = L.ia;
    double r[3], vr[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        r[d] = ia ? X[d] - pX[d] : pX[d] - X[d];
        vr[d] = ia ? V[d] - pV[d] : pV[d] - V[d];
    }
    const double rr = dot3(r[0], r[1], r[2], r[0], r[1], r[2]);
    const double vrr = dot3(vr[0], vr[1], vr[2], r[0], r[1], r[2]);
    const double kk = vrr / (L.mu * rr);
    if (ia) {
        const double ka = kk * L.ima;
#pragma unroll
        for (int d = 0; d < 3; ++d) V[d] = V[d] - (ka * r[d]);
    } else {
        const double kb = kk * L.imb;
#pragma unroll
        for (int d = 0; d < 3; ++d) V[d] = V[d] + (kb * r[d]);
    }
}

// Bound by the latency of its dependent steps: 32^3 with one dimer, 34
// workgroups, 4.6 us per MD step, of which the colloid update takes 1.0, the
// forces with the workgroup's tree 1.3 and the exchange 2.0 (5.2 before the
// trees gave each lane one value and the image of a colloid near the box
// needed no division).
//
// Chain workgroup g of a replica holds Verlet-list positions
// [g*B, (g+1)*B), B = NT*K (NT = 256 or 512 threads), K consecutive
// positions per thread, in registers for the whole interval.
// Descriptor fields used in every MD step, copied to scalar registers once:
// read through the descriptor they are fetched again after each fence of
// the exchange.
struct ChainConst {
    double Lv[3], hv[3];       // box lengths and half lengths
    uint64_t* partv;           // exchange buffers, two of stridev words
    int64_t stridev;           // G * ROWW + BCW
    int Gv;                    // workgroups of the replica's exchange buffers
    double catv;
    uint64_t seedv;
    uint64_t budgetv;          // longest wait for the other workgroups (ticks)
    __device__ double L(int d) const { return Lv[d]; }
    __device__ double h(int d) const { return hv[d]; }
    __device__ gptr<uint64_t> part() const { return (gptr<uint64_t>)partv; }
    __device__ int G() const { return Gv; }
    __device__ int64_t stride() const { return stridev; }
    __device__ double cat_prob() const { return catv; }
    __device__ uint64_t seed() const { return seedv; }
    __device__ uint64_t budget() const { return budgetv; }
};

__device__ __forceinline__ ChainConst chain_const(const RepDesc& D, uint64_t budget)
{
    ChainConst c;
    for (int d = 0; d < 3; ++d) {
        c.Lv[d] = uniform_d(D.Ld[d]);
        c.hv[d] = uniform_d(D.halfL[d]);
    }
    c.partv = reinterpret_cast<uint64_t*>(uniform_u64((uint64_t)(uintptr_t)D.partials));
    c.Gv = __builtin_amdgcn_readfirstlane(D.G);
    c.stridev = (int64_t)c.Gv * ROWW + BCW;
    c.catv = uniform_d(D.cat_prob);
    c.seedv = uniform_u64(D.seed);
    c.budgetv = uniform_u64(budget);
    return c;
}

// NB: bond capacity of the iterative-RATTLE tables (1 in the variants
// unrolled for one or two colloids, which never run it).
template <int NT, int NB>
struct ChainCtx {
    // periodic images of the colloid positions, the buffer step & 1 for MD step
    // `step` (0 at the start): wave 0 sets those of the next step while the
    // other waves still read this step's
    double sXw[2][MAXC][3];
    // colloid constants read in every MD step, staged once per interval
    double cRc2[MAXC], cSig2[MAXC], cEpsA[MAXC], cEpsB[MAXC], cSigma[MAXC];
    double cCull2[MAXC];       // (cut-off + reach margin)^2 of the interval's cull
    int32_t cCat[MAXC], cType[MAXC], cBody[MAXC];
    double cEcc[2][2];
    double sRed[NT / 64][NVAL_MAX];
    double sNode[NVAL_MAX];
    uint32_t sWhit[NT / 64];   // colloids that some entry of the wave is within cut-off of
    // master of the multi-workgroup exchange: the colloids each row listed
    // at the last look, a chunk of XV values by row and value, and the
    // trees' partial sums of each wave (the variants for one or two colloids
    // have at most 7 values)
    static constexpr int XV = NB > 1 ? XTAB_V : 8;
    uint32_t sE[MAX_CHAIN_G];
    double sTab[XTAB_R][XV];
    double sPart[NT / 64][XV];
    uint32_t sPairMask[MAXC];  // colloid c: bit a set when the pair (c, a) interacts
    uint32_t sFull;            // a colloid left its interval-start reach margin: no cull
    // colloid-colloid pairs (a < b) of the current positions: force on the
    // lower colloid and potential, and whether the pair interacts
    static constexpr int NPAIR = NB > 1 ? MAXC * (MAXC - 1) / 2 : 1;
    double sPairF[NPAIR][4];
    uint8_t sPairOn[NPAIR];
    double sU;
    uint32_t sflags;
    // colloid state and bonds staged for the iterative RATTLE (bond networks)
    static constexpr int NCI = NB > 1 ? MAXC : 1;
    double sXc[NCI][3], sVc[NCI][3], sXoc[NCI][3];
    int32_t sBa[NB], sBb[NB], sLay[NB + 1];
    // per bond, for the interval: d^2, the two thresholds, the two mass
    // factors and the inverse masses of its ends; for the stage under way:
    // the bond vector that the stage holds fixed
    double sBd2[NB], sBthr[NB], sBthv[NB];
    double sBmu2[NB], sBmud[NB], sBia[NB], sBib[NB];
    double sBr[NB][3];
};

// species_dU for an A -> B flip inside the MD chain, with the colloid
// constants from LDS (same arithmetic); mask: the colloids that the wave's
// entries can be within cut-off of, so that the others add nothing
template <class Ctx>
__device__ __forceinline__ double species_dU_lds(const Ctx& S, const double (*Xw)[3], const ChainConst& cc, uint32_t mask,
                                                 double x0, double x1, double x2)
{
    double du = 0.0;
    for (; mask; mask &= mask - 1u) {
        const int c = __ffs(mask) - 1;
        double dx = min_image(x0 - Xw[c][0], cc.L(0), cc.h(0));
        double dy = min_image(x1 - Xw[c][1], cc.L(1), cc.h(1));
        double dz = min_image(x2 - Xw[c][2], cc.L(2), cc.h(2));
        double r2 = dot3(dx, dy, dz, dx, dy, dz);
        if (r2 < S.cRc2[c]) {
            double cf, p0, p1;
            wca(r2, S.cSig2[c], S.cEpsA[c], cf, p0);
            wca(r2, S.cSig2[c], S.cEpsB[c], cf, p1);
            du += p1 - p0;
        }
    }
    return du;
}

// WCA force of colloid b on colloid a (a < b, sigma_ab = sigma_a + sigma_b,
// epsilon by the pair's types) and its potential, for the current colloid
// images; `on` is 0 when the two are of one rigid body or beyond the cut-off
// (then the values are not used)
template <class Ctx>
__device__ __forceinline__ void pair_force(const Ctx& S, const double (*Xw)[3], const ChainConst& cc, const ColloidParams* cp, int a,
                                           int b, double (&out)[4], uint8_t& on)
{
    on = 0;
    out[0] = 0.0; out[1] = 0.0; out[2] = 0.0; out[3] = 0.0;
    if (S.cBody[a] == S.cBody[b]) return;
    const double dx = min_image(Xw[a][0] - Xw[b][0], cc.L(0), cc.h(0));
    const double dy = min_image(Xw[a][1] - Xw[b][1], cc.L(1), cc.h(1));
    const double dz = min_image(Xw[a][2] - Xw[b][2], cc.L(2), cc.h(2));
    const double r2 = dot3(dx, dy, dz, dx, dy, dz);
    const double sab = S.cSigma[a] + S.cSigma[b];
    const double rc = 0x1.1f59ac3c7d6c0p+0 * sab;
    if (r2 < rc * rc) {
        double coef, pot;
        wca(r2, sab * sab, S.cEcc[S.cType[a]][S.cType[b]], coef, pot);
        out[0] = coef * dx; out[1] = coef * dy; out[2] = coef * dz; out[3] = pot;
        on = 1;
    }
}

// First half of a force evaluation: forces on this workgroup's list
// entries from all colloids, and the per-colloid force sums and the
// potential reduced over this workgroup's list positions with the fixed
// binary tree (within a thread over K, over the lanes of a wave, over the
// waves).  With several workgroups the node values are then published for
// the others (chain_collect completes the tree over workgroups).
template <class T, int K, int NT, int NB>
__device__ __forceinline__ void chain_compute(ChainCtx<NT, NB>& S, const double (*Xw)[3], const ChainConst& cc, const ColloidParams* cp,
                              int nc, const bool* valid, const T (*x)[3], const T (*x0)[3], const uint8_t* st,
                              double (*f)[3], bool* inside, int g, int Gact, bool solo,
                              uint32_t& wmask, double me2, uint32_t& nbar, uint32_t epoch0)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    double u[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        f[j][0] = 0.0; f[j][1] = 0.0; f[j][2] = 0.0;
        u[j] = 0.0;
        inside[j] = false;
    }
    // Colloids within reach of this wave: wmask, set at the start of the
    // interval from the box of the wave's entries (reach_box).  It holds
    // while every entry stays within the margin me of its position at the
    // start and every colloid within half the skin of its own; once either
    // fails the wave tests every colloid for the rest of the interval.  A
    // colloid out of reach contributes exactly zero to every entry of the
    // wave, so its distances are not computed.
    const uint32_t all_mask = nc >= 32 ? 0xffffffffu : ((1u << nc) - 1u);
    if (wmask != all_mask) {
        bool moved = false;
#pragma unroll
        for (int j = 0; j < K; ++j)
            if (valid[j]) {
                const double dx = min_image((double)x[j][0] - (double)x0[j][0], cc.L(0), cc.h(0));
                const double dy = min_image((double)x[j][1] - (double)x0[j][1], cc.L(1), cc.h(1));
                const double dz = min_image((double)x[j][2] - (double)x0[j][2], cc.L(2), cc.h(2));
                moved = moved || !(dot3(dx, dy, dz, dx, dy, dz) < me2);
            }
        if (__ballot(moved) != 0 || S.sFull != 0) wmask = all_mask;
    }
    const uint32_t reach_mask = wmask;
    uint32_t whit = 0;           // colloids some entry of the wave is within cut-off of
    // colloids two at a time: forces and the reduction over the K entries
    // of each thread, then the wave trees of the six components (and, after
    // the last pair, of the potential) side by side
    constexpr int CB = 2;
    bool hit_any = false;        // some entry of this wave hit some colloid so far
    // pairs with a colloid in reach (bit 2 p: pair p); the others' values are
    // zero (128^3 with 8 dimers: walking all 16 colloids in every wave, with the
    // positions awaited behind their flag, 805 us a launch alone, now 633)
    uint32_t pairs = nc > 2 ? (reach_mask | (reach_mask >> 1)) & 0x55555555u : (nc > 0 ? 1u : 0u);
    if (nc > 2)
        for (int k = lane; k < 3 * nc + 1; k += 64) S.sRed[wave][k] = 0.0;
    while (pairs) {
        const int c0 = __ffs(pairs) - 1;
        pairs &= pairs - 1u;
        double tv[8];
        bool hit_chunk = false;  // ... one of this pair of colloids
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int c = c0 + cb;
            tv[3 * cb + 0] = 0.0; tv[3 * cb + 1] = 0.0; tv[3 * cb + 2] = 0.0;
            if (c >= nc || !((reach_mask >> c) & 1u)) continue;
            const double Xc0 = Xw[c][0], Xc1 = Xw[c][1], Xc2 = Xw[c][2];
            const double rc2 = S.cRc2[c], sig2 = S.cSig2[c];
            const double eA = S.cEpsA[c], eB = S.cEpsB[c];
            const bool cat = S.cCat[c] != 0;
            double gx[K], gy[K], gz[K];
            bool any = false;
            // distances for the K entries, then the WCA terms only if some
            // lane of the wave is inside this colloid's cut-off (wave-uniform
            // test); within it the K entries are evaluated branch-free with
            // selects, the untaken case at the cut-off radius (discarded)
            double dxs[K], dys[K], dzs[K], r2s[K];
            bool hit[K];
#pragma unroll
            for (int j = 0; j < K; ++j) {
                dxs[j] = min_image((double)x[j][0] - Xc0, cc.L(0), cc.h(0));
                dys[j] = min_image((double)x[j][1] - Xc1, cc.L(1), cc.h(1));
                dzs[j] = min_image((double)x[j][2] - Xc2, cc.L(2), cc.h(2));
                r2s[j] = dot3(dxs[j], dys[j], dzs[j], dxs[j], dys[j], dzs[j]);
                hit[j] = valid[j] && (r2s[j] < rc2);
                any = any || hit[j];
                gx[j] = 0.0; gy[j] = 0.0; gz[j] = 0.0;
            }
            if (__ballot(any) != 0) {
                hit_chunk = true;
                whit |= 1u << c;
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    double coef, pot;
                    wca(hit[j] ? r2s[j] : rc2, sig2, (st[j] & 1) ? eB : eA, coef, pot);
                    const double ax = coef * dxs[j], ay = coef * dys[j], az = coef * dzs[j];
                    gx[j] = hit[j] ? ax : 0.0;
                    gy[j] = hit[j] ? ay : 0.0;
                    gz[j] = hit[j] ? az : 0.0;
                    f[j][0] = hit[j] ? f[j][0] + ax : f[j][0];
                    f[j][1] = hit[j] ? f[j][1] + ay : f[j][1];
                    f[j][2] = hit[j] ? f[j][2] + az : f[j][2];
                    u[j] = hit[j] ? u[j] + pot : u[j];
                    inside[j] = inside[j] || (hit[j] && cat);
                }
            }
            // the three components over this thread's K list positions
#pragma unroll
            for (int s2 = 1; s2 < K; s2 <<= 1)
#pragma unroll
                for (int j = 0; j + s2 < K; j += 2 * s2) {
                    gx[j] = gx[j] + gx[j + s2];
                    gy[j] = gy[j] + gy[j + s2];
                    gz[j] = gz[j] + gz[j + s2];
                }
            tv[3 * cb + 0] = gx[0]; tv[3 * cb + 1] = gy[0]; tv[3 * cb + 2] = gz[0];
        }
        const bool last = pairs == 0u;
        tv[3 * CB] = tv[7] = 0.0;
        if (last) {
            double a[K];
#pragma unroll
            for (int j = 0; j < K; ++j) a[j] = u[j];
#pragma unroll
            for (int s2 = 1; s2 < K; s2 <<= 1)
#pragma unroll
                for (int j = 0; j + s2 < K; j += 2 * s2) a[j] = a[j] + a[j + s2];
            tv[3 * CB] = a[0];
        }
        hit_any = hit_any || hit_chunk;
        // no entry of the wave inside either colloid's cut-off (and, for the
        // potential, inside any): every value is +0.0, and so is its tree
        // (lane k: component k of the pair, lane 6 the potential)
        double sum = 0.0;
        if (hit_chunk || (last && hit_any)) sum = wave_tree_spread<8>(tv);
        const int o = lane == 3 * CB ? 3 * nc : 3 * c0 + lane;
        if (lane < 3 * CB ? o < 3 * nc : (lane == 3 * CB && last)) S.sRed[wave][o] = sum;
    }
    if (nc == 0) {
        // no colloid: the potential of the list is zero (tree of zeros)
        if (lane == 0) S.sRed[wave][0] = 0.0;
    }
    if (lane == 0) S.sWhit[wave] = whit;
    __syncthreads();
    const int nv = 3 * nc + 1;
    constexpr int NW = NT / 64;
    if (t < nv) {
        double a[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) a[k] = S.sRed[k][t];
#pragma unroll
        for (int s = 1; s < NW; s <<= 1)
#pragma unroll
            for (int k = 0; k + s < NW; k += 2 * s) a[k] = a[k] + a[k + s];
        S.sNode[t] = a[0];
    }
    if (Gact > 1) {
        // Publish this workgroup's node values, each double as two 64-bit
        // words (low and high half, each with the barrier's epoch in its low
        // 32 bits), so that a reader accepts a word only when its epoch
        // matches and needs no separate flag or fence.  Epochs are unique per
        // barrier of the replica; the two buffers alternate between barriers.
        // Solo form: value v in planes 2v and 2v + 1, column g (every value).
        // Otherwise the packed row g of the master exchange (exchange_master).
        nbar++;
        const uint32_t epoch = epoch0 + nbar;
        const int64_t Gs = cc.G();
        const gptr<uint64_t> P = cc.part() + (int64_t)(nbar & 1) * cc.stride();
        uint32_t m = 0;
        if (t < nv || t == 0)
#pragma unroll
            for (int w2 = 0; w2 < NW; ++w2) m |= S.sWhit[w2];
        if (t < nv) {
            const double val = S.sNode[t];
            const uint64_t lo = ((uint64_t)(uint32_t)__double2loint(val) << 32) | epoch;
            const uint64_t hi = ((uint64_t)(uint32_t)__double2hiint(val) << 32) | epoch;
            int64_t o = -1;
            if (solo) {
                o = (int64_t)(2 * t) * Gs + g;          // planes 2t, 2t + 1 (all values)
            } else if (t == 3 * nc) {
                o = (int64_t)g * ROWW + 2;               // potential: slot 1
            } else if ((m >> (t / 3)) & 1u) {
                const int c = t / 3;
                o = (int64_t)g * ROWW + 2 * (2 + 3 * __popc(m & ((1u << c) - 1u)) + (t - 3 * c));
            }
            if (o >= 0) {
                __hip_atomic_store(&P[o], lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&P[solo ? o + Gs : o + 1], hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (t == 0 && !solo)
            __hip_atomic_store(&P[(int64_t)g * ROWW], ((uint64_t)m << 32) | epoch, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Colloids within reach of this wave for an interval: the bounding box of
// the wave's entries at its start (minimum-image offsets from its first
// entry, which is valid whenever any is) against each colloid's sphere of
// the cut-off plus the reach margin (me plus half the skin, cCull2), one lane
// per colloid.  Systems of one or two colloids test them all.
template <class T, int K, int NT, int NB>
__device__ __forceinline__ uint32_t reach_box(const ChainCtx<NT, NB>& S, const double (*Xw)[3], const ChainConst& cc, int nc,
                                              const bool* valid, const T (*x)[3])
{
    const int lane = threadIdx.x & 63;
    uint32_t mask = nc >= 32 ? 0xffffffffu : ((1u << nc) - 1u);
    if (nc <= 2) return mask;
    double ref[3], lo[3], hi[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        ref[d] = __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint((double)x[0][d])),
                                  __builtin_amdgcn_readfirstlane(__double2loint((double)x[0][d])));
        lo[d] = 1e300; hi[d] = -1e300;
#pragma unroll
        for (int j = 0; j < K; ++j)
            if (valid[j]) {
                const double o = min_image((double)x[j][d] - ref[d], cc.L(d), cc.h(d));
                lo[d] = o < lo[d] ? o : lo[d];
                hi[d] = o > hi[d] ? o : hi[d];
            }
        wave_min_max(lo[d], hi[d]);
    }
    bool near = true;
    if (lane < nc) {
        double r2 = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if (!(hi[d] - lo[d] < cc.h(d))) continue;          // wide (or no entry): no bound
            const double oc = min_image(Xw[lane][d] - ref[d], cc.L(d), cc.h(d));
            double dd = 1e300;
#pragma unroll
            for (int img = -1; img <= 1; ++img) {
                const double ci = oc + (double)img * cc.L(d);
                double e = lo[d] - ci > ci - hi[d] ? lo[d] - ci : ci - hi[d];
                e = e > 0.0 ? e : 0.0;
                dd = e < dd ? e : dd;
            }
            r2 += dd * dd;
        }
        // margin far above the rounding of the entries' own r^2
        near = r2 <= S.cCull2[lane] * (1.0 + 1e-9) + 1e-9;
    }
    return mask & (uint32_t)__ballot(near);
}

// Exchange through a master workgroup (workgroup 0), used when the solo
// form does not apply.  Every workgroup publishes a packed row: the header
// (the mask of the colloids some entry of the workgroup was within cut-off
// of, and the barrier's epoch), the potential, then the three components
// of each listed colloid in ascending order, each double as two 64-bit
// words tagged with the epoch.  The node value of an unlisted colloid is
// exactly +0.0 (a tree of zeros), so it is not sent.  The master reads the
// rows in slots of two words (slot 0 the header, 1 the potential, 2 + 3j + d
// component d of the j-th listed colloid), a fixed group of NT / XTAB_R
// threads per row, expecting the colloids each row listed at the last look
// (sE); a round is repeated until every header is current and lists what
// was expected and every slot read is current.  The values go into a table
// by row and value; each value is then summed over the rows in the balanced
// binary tree (the wave w of NW takes a block of rows, the blocks pairwise),
// an entry the final round did not list counting as +0.0.  The master alone
// then updates the colloids and broadcasts their positions (broadcast_images
// / await_images).
constexpr int XSLOTS = 4;      // slots per thread and batch of the master's reads

__device__ __forceinline__ int nth_bit(uint32_t m, int j)
{
    for (int i = 0; i < j; ++i) m &= m - 1u;
    return __ffs(m) - 1;
}

// Balanced binary tree over N (a power of two) values get(0..N-1), formed
// in one pass as a binary counter: the partial sum of each complete block of
// 2^k values is kept until its sibling block is complete.
template <int N, class F>
__device__ __forceinline__ double tree_sum(F get)
{
    constexpr int LG = N <= 1 ? 0 : N <= 2 ? 1 : N <= 4 ? 2 : N <= 8 ? 3 : N <= 16 ? 4 : N <= 32 ? 5 : N <= 64 ? 6 : 7;
    static_assert((1 << LG) == N, "a power of two up to 128");
    double st[LG + 1];
#pragma unroll
    for (int r = 0; r < N; ++r) {
        double c = get(r);
        int lvl = 0;
#pragma unroll
        for (int b = 1; b < N; b <<= 1) {
            if (!(r & b)) break;
            c = st[lvl] + c;
            ++lvl;
        }
        st[lvl] = c;
    }
    return st[LG];
}

template <int NT, int NB>
__device__ __forceinline__ void exchange_master(ChainCtx<NT, NB>& S, const ChainConst& cc, int nc, int Gact,
                                                uint32_t nbar, uint32_t epoch0)
{
    constexpr int NW = NT / 64;
    constexpr int TPR = NT / XTAB_R;          // threads per row
    constexpr int RB = XTAB_R / NW;           // rows per wave in the trees
    constexpr int XV = ChainCtx<NT, NB>::XV;  // values per table chunk
    static_assert(TPR >= 1 && (64 % TPR) == 0 && RB >= 1, "row groups within a wave");
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const uint32_t epoch = epoch0 + nbar;
    const gptr<const uint64_t> P = cc.part() + (int64_t)(nbar & 1) * cc.stride();
    const int nv = 3 * nc + 1;
    const uint64_t t_start = wall_clock64();
    const int rt = t / TPR, sub = t - rt * TPR;   // this thread's row of the chunk, place in its group
    // passes over chunks of XV values and of XTAB_R rows of the table
    for (int v0 = 0; v0 < nv; v0 += XV)
        for (int r0 = 0; r0 < Gact; r0 += XTAB_R) {
            const int nr = Gact - r0 < XTAB_R ? Gact - r0 : XTAB_R;
            const bool rv = rt < nr;
            const gptr<const uint64_t> row = P + (int64_t)(r0 + (rv ? rt : 0)) * ROWW;
            int nap = 0;
            while (true) {
                __asm__ __volatile__("" ::: "memory");
                const uint32_t e = rv ? S.sE[r0 + rt] : 0u;
                const int ns = rv ? 2 + 3 * __popc(e) : 0;       // slots of the row
                int ok = 1;
                uint32_t mnew = e;
                for (int s0 = sub; s0 < ns; s0 += XSLOTS * TPR) {
                    uint64_t wl[XSLOTS], wh[XSLOTS];
#pragma unroll
                    for (int k = 0; k < XSLOTS; ++k) {
                        const int sl = s0 + k * TPR;
                        wl[k] = wh[k] = 0ull;
                        if (sl < ns) {
                            // slot 0: the header word; slot s > 0: words 2s, 2s + 1
                            wl[k] = __hip_atomic_load(&row[sl == 0 ? 0 : 2 * sl], __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
                            if (sl > 0)
                                wh[k] = __hip_atomic_load(&row[2 * sl + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < XSLOTS; ++k) {
                        const int sl = s0 + k * TPR;
                        if (sl >= ns) continue;
                        if (sl == 0) {
                            const bool cur = (uint32_t)wl[k] == epoch;
                            const uint32_t m = (uint32_t)(wl[k] >> 32);
                            ok &= (cur && m == e) ? 1 : 0;
                            if (cur) mnew = m;
                            continue;
                        }
                        ok &= ((uint32_t)wl[k] == epoch && (uint32_t)wh[k] == epoch) ? 1 : 0;
                        // value index of the slot
                        int v = 3 * nc;
                        if (sl >= 2) {
                            const int j = (sl - 2) / 3, d = (sl - 2) - 3 * j;
                            v = 3 * nth_bit(e, j) + d;
                        }
                        if (v >= v0 && v < v0 + XV)
                            S.sTab[rt][v - v0] = __hiloint2double((int)(wh[k] >> 32), (int)(wl[k] >> 32));
                    }
                }
                // the row's header thread: look for the listed colloids next
                // round (the row's threads share a wave, so every one of them
                // read e above)
                if (rv && sub == 0 && mnew != e) S.sE[r0 + rt] = mnew;
                if (__syncthreads_and(ok)) break;
                // the time budget, decided for the workgroup by thread 0; once
                // given up (RMP_FLAG_BARRIER) later barriers do not wait
                if (t == 0 && !(S.sflags & RMP_FLAG_BARRIER) && wall_clock64() - t_start > cc.budget())
                    atomicOr(&S.sflags, RMP_FLAG_BARRIER);
                __syncthreads();
                if (S.sflags & RMP_FLAG_BARRIER) break;
                if (++nap > 16) __builtin_amdgcn_s_sleep(2);
            }
            // trees: lane l the value v0 + l; wave w the rows [w RB, (w + 1) RB)
            // of the chunk, then wave 0 the NW blocks pairwise.  An entry of a
            // row past Gact, or of a colloid the row did not list, is +0.0.
            const int nvc = nv - v0 < XV ? nv - v0 : XV;
            if (lane < nvc) {
                const int v = v0 + lane;
                const bool isU = v == 3 * nc;
                const int c = v / 3;
                const int rb = wave * RB;
                const double part = tree_sum<RB>([&](int q) {
                    const int r = rb + q;
                    const bool listed = r < nr && (isU || ((S.sE[r0 + r] >> c) & 1u) != 0u);
                    return listed ? S.sTab[r][lane] : 0.0;
                });
                S.sPart[wave][lane] = part;
            }
            __syncthreads();
            if (wave == 0 && lane < nvc) {
                const double tot = tree_sum<NW>([&](int w) { return S.sPart[w][lane]; });
                S.sNode[v0 + lane] = r0 == 0 ? tot : S.sNode[v0 + lane] + tot;
            }
            // the next chunk rewrites the table only after every wave has read it
            __syncthreads();
        }
}

// Master: the colloid positions of the coming MD step (their images, as in
// sXw) for the other workgroups, each double as two words tagged with the
// barrier's epoch, then the flag word (sFull << 32 | epoch).  Wave 0.
template <int NT, int NB>
__device__ __forceinline__ void broadcast_images(ChainCtx<NT, NB>& S, const double (*Xw)[3], const ChainConst& cc, int nc, uint32_t nbar,
                                                 uint32_t epoch0)
{
    const int lane = threadIdx.x & 63;
    const uint32_t epoch = epoch0 + nbar;
    const gptr<uint64_t> B = cc.part() + (int64_t)(nbar & 1) * cc.stride() + cc.G() * (int64_t)ROWW;
    for (int k = lane; k < 3 * nc; k += 64) {
        const double val = Xw[k / 3][k % 3];
        const uint64_t lo = ((uint64_t)(uint32_t)__double2loint(val) << 32) | epoch;
        const uint64_t hi = ((uint64_t)(uint32_t)__double2hiint(val) << 32) | epoch;
        __hip_atomic_store(&B[2 * k], lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&B[2 * k + 1], hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0)
        __hip_atomic_store(&B[6 * nc], ((uint64_t)S.sFull << 32) | epoch, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// Other workgroups: wait (bounded) for the master's positions of the coming
// MD step into Xw, and its flag word into sFull.  Wave 0; every lane polls the
// words it needs.
template <int NT, int NB>
__device__ __forceinline__ void await_images(ChainCtx<NT, NB>& S, double (*Xw)[3], const ChainConst& cc, int nc,
                                             uint32_t nbar, uint32_t epoch0)
{
    const int lane = threadIdx.x & 63;
    const uint32_t epoch = epoch0 + nbar;
    const gptr<const uint64_t> B = cc.part() + (int64_t)(nbar & 1) * cc.stride() + cc.G() * (int64_t)ROWW;
    const uint64_t t_start = wall_clock64();
    int nap = 0;
    // value k of the 3 nc: its two words; k = 3 nc: the flag word
    const int nk = 3 * nc + 1;
    while (true) {
        // every round loads anew (no load of the words may be carried over
        // from an earlier round)
        __asm__ __volatile__("" ::: "memory");
        constexpr int KL = (3 * MAXC + 1 + 63) / 64;
        uint64_t lo[KL], hi[KL];
#pragma unroll
        for (int q = 0; q < KL; ++q) {
            const int k = lane + 64 * q;
            lo[q] = hi[q] = epoch;
            if (k < nk) {
                lo[q] = __hip_atomic_load(&B[2 * k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (k < 3 * nc) hi[q] = __hip_atomic_load(&B[2 * k + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        bool good = true;
#pragma unroll
        for (int q = 0; q < KL; ++q) good = good && (uint32_t)lo[q] == epoch && (uint32_t)hi[q] == epoch;
        const bool all = __ballot(!good) == 0;
        const bool late = !all && wall_clock64() - t_start > cc.budget();
        const bool gave_up = (__hip_atomic_load(&S.sflags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) &
                              RMP_FLAG_BARRIER) != 0;
        if (all) {
#pragma unroll
            for (int q = 0; q < KL; ++q) {
                const int k = lane + 64 * q;
                if (k < 3 * nc) Xw[k / 3][k % 3] = __hiloint2double((int)(hi[q] >> 32), (int)(lo[q] >> 32));
                else if (k == 3 * nc && (lo[q] >> 32) != 0) S.sFull = 1u;
            }
            break;
        }
        if (late && lane == 0) atomicOr(&S.sflags, RMP_FLAG_BARRIER);
        if (late || gave_up) break;
        if (++nap > 16) __builtin_amdgcn_s_sleep(2);
    }
}

// Wait (bounded) for the exchange words of values v = v0 + vb*vs (vb < VB,
// v < nv) of workgroups [0, Gact) at this barrier, then reduce each value
// over the workgroups with the fixed tree: lane l holds workgroups
// [l*Q, l*Q+Q) (Q <= QM), summed pairwise, then the wave tree, padded with
// zeros to a power of two.  Lane l returns value v0 + (l % VB) vs.  Only slots
// that exist are loaded (wave-uniform guards): a co-resident workgroup that
// is still computing must not be starved by polling traffic.
template <int VB, int QM, class Ctx>
__device__ __forceinline__ double poll_reduce(Ctx& S, gptr<const uint64_t> part, int64_t Gs, int v0, int vs, int nv,
                                            int Gact, int Q, uint32_t epoch, uint64_t budget)
{
    const int lane = threadIdx.x & 63;
    double b4[VB][QM];
    // once this workgroup has given up on one barrier (RMP_FLAG_BARRIER) it
    // does not wait on later ones, so a kernel whose peers cannot all run
    // ends within about one time budget (wall_clock64 counts at 100 MHz)
    const uint64_t t_start = wall_clock64();
    int nap = 0;
    while (true) {
        // every round loads anew
        __asm__ __volatile__("" ::: "memory");
        uint64_t wl[VB][QM], wh[VB][QM];
#pragma unroll
        for (int vb = 0; vb < VB; ++vb) {
            const int v = v0 + vb * vs;
#pragma unroll
            for (int q = 0; q < QM; ++q) {
                const int gg = lane * Q + q;
                const int gc = gg < Gact ? gg : 0;
                const int64_t o = (int64_t)(2 * v) * Gs + gc;
                if (v < nv && q < Q) {
                    wl[vb][q] = __hip_atomic_load(&part[o], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    wh[vb][q] = __hip_atomic_load(&part[o + Gs], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    wl[vb][q] = 0;
                    wh[vb][q] = 0;
                }
            }
        }
        bool ok = true;
#pragma unroll
        for (int vb = 0; vb < VB; ++vb) {
            const int v = v0 + vb * vs;
#pragma unroll
            for (int q = 0; q < QM; ++q) {
                const int gg = lane * Q + q;
                const bool use = v < nv && q < Q && gg < Gact;
                const bool good = ((uint32_t)wl[vb][q] == epoch) & ((uint32_t)wh[vb][q] == epoch);
                ok = ok & (!use | good);
                b4[vb][q] = use ? __hiloint2double((int)(wh[vb][q] >> 32), (int)(wl[vb][q] >> 32)) : 0.0;
            }
        }
        if (__ballot(!ok) == 0) break;
        if (__hip_atomic_load(&S.sflags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & RMP_FLAG_BARRIER)
            break;
        if (wall_clock64() - t_start > budget) {
            if (lane == 0) atomicOr(&S.sflags, RMP_FLAG_BARRIER);
            break;
        }
        // a long wait backs off (128 clocks a round after the first 16)
        if (++nap > 16) __builtin_amdgcn_s_sleep(2);
    }
    double out[VB];
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) {
        double a2 = b4[vb][0];
        if (QM >= 2 && Q == 2) a2 = b4[vb][0] + b4[vb][QM >= 2 ? 1 : 0];
        if (QM >= 4 && Q == 4)
            a2 = (b4[vb][0] + b4[vb][QM >= 4 ? 1 : 0]) + (b4[vb][QM >= 4 ? 2 : 0] + b4[vb][QM >= 4 ? 3 : 0]);
        out[vb] = a2;
    }
    return wave_tree_spread<VB>(out);
}

// Second half: wait for the other workgroups' node values of this
// evaluation, finish the tree over workgroups, then the colloid forces
// (solvent part, then colloid-colloid pairs in (a<b) order) into cF of
// thread c (c < nc) and, when requested, the potential into sU.  With at
// most 8 values and 64 workgroups (one workgroup per lane) wave 0 does all
// of it alone (the solo form: it reads every value of every row) and the
// other waves go straight on; otherwise the whole workgroup takes part in
// the sparse exchange.
// Constants of the colloid of lane c (c < nc) used by the pair forces,
// loaded once per interval
struct PairLane {
    uint32_t same;             // bit a set: colloid a is in this colloid's rigid body (no force)
    int ctype;
    double sigma;
};

template <class T, int K, int NT, int NB>
__device__ __forceinline__ void chain_collect(ChainCtx<NT, NB>& S, const double (*Xw)[3], const ChainConst& cc, const ColloidParams* cp,
                              int nc, int g, int Gact, int Gpad, uint32_t nbar, uint32_t epoch0,
                              bool want_potential, double (&cF)[3], const PairLane& PL)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int nv = 3 * nc + 1;
    const int Q = Gpad > 64 ? Gpad / 64 : 1;
    const bool solo = Q == 1 && nv <= 8;
    if (solo && wave != 0) return;
    if constexpr (NB > 1) {
        // colloid-colloid pair forces (a < b, enumerated row by row), one
        // thread per pair, and the mask of the interacting pairs of each
        // colloid (cleared with the colloid position update)
        const int np = nc * (nc - 1) / 2;
        const int ps = solo ? 64 : NT;
        for (int p = t; p < np; p += ps) {
            int a = 0, rem = p;
            while (rem >= nc - 1 - a) { rem -= nc - 1 - a; ++a; }
            const int b = a + 1 + rem;
            pair_force(S, Xw, cc, cp, a, b, S.sPairF[p], S.sPairOn[p]);
            if (S.sPairOn[p]) {
                atomicOr(&S.sPairMask[a], 1u << b);
                atomicOr(&S.sPairMask[b], 1u << a);
            }
        }
    }
    if (Gact > 1) {
        if (solo) {
            const uint32_t epoch = epoch0 + nbar;
            const gptr<const uint64_t> part = cc.part() + (int64_t)(nbar & 1) * cc.stride();
            const double out = poll_reduce<8, 1>(S, part, cc.G(), 0, 1, nv, Gact, 1, epoch, cc.budget());
            if (lane < nv) S.sNode[lane] = out;
        } else {
            exchange_master(S, cc, nc, Gact, nbar, epoch0);
        }
    }
    if (solo) wave_sync();
    else __syncthreads();
    // colloid forces: solvent part, then colloid-colloid pairs in (a<b) order
    if constexpr (NB > 1) {
        // pairs from LDS: colloid c adds those that interact in the order of
        // the other colloid, + for the lower index
        if (t < nc) {
            const int c = t;
            double F[3] = {-S.sNode[3 * c + 0], -S.sNode[3 * c + 1], -S.sNode[3 * c + 2]};
            uint32_t m = S.sPairMask[c];
            while (m) {
                const int a = __ffs(m) - 1;
                m &= m - 1u;
                const bool c_lo = c < a;
                const int lo = c_lo ? c : a, hi = c_lo ? a : c;
                const int p = lo * nc - (lo * (lo + 1)) / 2 + (hi - lo - 1);
                for (int d = 0; d < 3; ++d) F[d] = c_lo ? F[d] + S.sPairF[p][d] : F[d] - S.sPairF[p][d];
            }
            for (int d = 0; d < 3; ++d) cF[d] = F[d];
        }
        if (t == 0 && want_potential) {
            double ucc = 0.0;
            const int np = nc * (nc - 1) / 2;
            for (int p = 0; p < np; ++p)
                if (S.sPairOn[p]) ucc = ucc + S.sPairF[p][3];
            S.sU = S.sNode[3 * nc] + ucc;
        }
        return;
    }
    if (t < nc) {
        const int c = t;
        double F[3] = {-S.sNode[3 * c + 0], -S.sNode[3 * c + 1], -S.sNode[3 * c + 2]};
        for (int a = 0; a < nc; ++a) {
            if ((PL.same >> a) & 1u) continue;      // itself or its own rigid body
            // colloid a's constants by its (uniform) index, this lane's from
            // registers; operands in the pair's (lo, hi) order
            const double sig_a = S.cSigma[a];
            const int ct_a = S.cType[a];
            const bool c_lo = c < a;
            const int lo = c_lo ? c : a, hi = c_lo ? a : c;
            double dx = min_image(Xw[lo][0] - Xw[hi][0], cc.L(0), cc.h(0));
            double dy = min_image(Xw[lo][1] - Xw[hi][1], cc.L(1), cc.h(1));
            double dz = min_image(Xw[lo][2] - Xw[hi][2], cc.L(2), cc.h(2));
            double r2 = dot3(dx, dy, dz, dx, dy, dz);
            double sab = c_lo ? PL.sigma + sig_a : sig_a + PL.sigma;
            double rc = 0x1.1f59ac3c7d6c0p+0 * sab;
            if (r2 < rc * rc) {
                const int t_lo = c_lo ? PL.ctype : ct_a, t_hi = c_lo ? ct_a : PL.ctype;
                const double e_lo0 = t_lo == 0 ? cp->eps_cc[0][0] : cp->eps_cc[1][0];
                const double e_lo1 = t_lo == 0 ? cp->eps_cc[0][1] : cp->eps_cc[1][1];
                double coef, pot;
                wca(r2, sab * sab, t_hi == 0 ? e_lo0 : e_lo1, coef, pot);
                double g3[3] = {coef * dx, coef * dy, coef * dz};
                for (int d = 0; d < 3; ++d) F[d] = c_lo ? F[d] + g3[d] : F[d] - g3[d];
            }
        }
        for (int d = 0; d < 3; ++d) cF[d] = F[d];
    }
    if (t == 0 && want_potential) {
        double ucc = 0.0;
        for (int a = 0; a < nc; ++a)
            for (int b = a + 1; b < nc; ++b) {
                if (cp->body[a] == cp->body[b]) continue;
                double dx = min_image(Xw[a][0] - Xw[b][0], cc.L(0), cc.h(0));
                double dy = min_image(Xw[a][1] - Xw[b][1], cc.L(1), cc.h(1));
                double dz = min_image(Xw[a][2] - Xw[b][2], cc.L(2), cc.h(2));
                double r2 = dot3(dx, dy, dz, dx, dy, dz);
                double sab = cp->sigma[a] + cp->sigma[b];
                double rc = 0x1.1f59ac3c7d6c0p+0 * sab;
                if (r2 < rc * rc) {
                    double coef, pot;
                    wca(r2, sab * sab, cp->eps_cc[cp->ctype[a]][cp->ctype[b]], coef, pot);
                    ucc = ucc + pot;
                }
            }
        S.sU = S.sNode[3 * nc] + ucc;
    }
    // no barrier here: the node values and colloid images are next written
    // after the workgroup barrier that follows the colloid position update
}

template <class T, int K, int NC, int NT>
__device__ __forceinline__ void chain_body(Work w, int g, const RepDesc& D, const ChainConst& cc)
{
    if (!D.active) return;
    RepState* rs = D.rs;
    const ColloidParams* cp = D.cp;
    // NC > 0: every system of the launch has NC colloids (loops over the
    // colloids unrolled at compile time); NC == 0: read per system
    const int nc = NC > 0 ? NC : cp->nc;
    constexpr int B = NT * K;
    int64_t ncand = rs->n_cand;
    if (ncand > D.cand_cap) ncand = D.cand_cap;
    int Gact = (int)((ncand + B - 1) / B);
    if (Gact < 1) Gact = 1;
    if (Gact > D.G) Gact = D.G;
    if (g >= Gact) return;
    if (nc == 0 && ncand == 0) {
        // no colloid and an empty list (flows, bare solvent): nothing moves
        // in the chain; close the interval's counters as the full path would
        if (g == 0 && threadIdx.x == 0) {
            D.epart[0] = 0.0;
            D.epart[1] = 0.0;
            rs->U = 0.0;
            rs->md_step = rs->md_step + D.n_md;
            rs->n_cand_used = 0;
        }
        return;
    }
    int Gpad = 1;
    while (Gpad < Gact) Gpad <<= 1;

    __shared__ ChainCtx<NT, NC == 0 ? RMP_MAX_BONDS : 1> S;
    const int t = threadIdx.x;
    if (t == 0) {
        S.sflags = 0;
        S.sFull = 0;
    }
    if (t < MAXC) S.sPairMask[t] = 0u;
    for (int r = t; r < MAX_CHAIN_G; r += NT) S.sE[r] = 0u;
    if (t < 4) S.cEcc[t >> 1][t & 1] = cp->eps_cc[t >> 1][t & 1];
    // colloid c lives in registers of thread c (c < nc, wave 0): position,
    // velocity, force, position at the start of the interval
    double cX[3] = {0.0, 0.0, 0.0}, cV[3] = {0.0, 0.0, 0.0}, cF[3] = {0.0, 0.0, 0.0};
    double cX0[3] = {0.0, 0.0, 0.0};
    const BondLane BL = bond_lane(cp, nc);
    // iterative RATTLE (bond networks, or asked for): generic variant only,
    // the host launches it whenever a system of the launch needs it
    const bool iter = NC == 0 && cp->iterative != 0;
    PairLane PL;
    PL.same = 0u;
    if (t < nc)
        for (int a = 0; a < nc; ++a)
            if (cp->body[a] == cp->body[t]) PL.same |= 1u << a;
    PL.ctype = t < nc ? cp->ctype[t] : 0;
    PL.sigma = t < nc ? cp->sigma[t] : 0.0;
    const double chc = t < nc ? cp->hc[t] : 0.0;
    if (t < nc) {
        for (int d = 0; d < 3; ++d) {
            cX[d] = rs->X[t][d];
            cV[d] = rs->V[t][d];
            cX0[d] = cX[d];
            // (both buffers: a wait that is given up leaves one as it was)
            S.sXw[0][t][d] = S.sXw[1][t][d] = colloid_image(cX[d], cc.L(d));
        }
        S.cRc2[t] = cp->rc2[t];
        {
            const double rr = sqrt(cp->rc2[t]) + D.cull_margin;
            S.cCull2[t] = rr * rr;
        }
        S.cSig2[t] = cp->sig2[t];
        S.cEpsA[t] = cp->epsA[t];
        S.cEpsB[t] = cp->epsB[t];
        S.cSigma[t] = cp->sigma[t];
        S.cCat[t] = cp->catalytic[t];
        S.cType[t] = cp->ctype[t];
        S.cBody[t] = cp->body[t];
    }
    if (iter) {
        // bonds of the iterative RATTLE in LDS for the interval
        const double tol = cp->rattle_tol;
        for (int q = t; q < cp->nbonds; q += NT) {
            const int a = cp->bond_a[q], b = cp->bond_b[q];
            const double dd2 = cp->bond_d[q] * cp->bond_d[q];
            const double ima = cp->imass[a], imb = cp->imass[b];
            const double mu = ima + imb;
            S.sBa[q] = a;
            S.sBb[q] = b;
            S.sBd2[q] = dd2;
            S.sBthr[q] = (2.0 * tol) * dd2;
            S.sBthv[q] = (tol * dd2) / D.dt;
            S.sBmu2[q] = 2.0 * mu;
            S.sBmud[q] = mu * dd2;
            S.sBia[q] = ima;
            S.sBib[q] = imb;
        }
        for (int L = t; L <= cp->n_layers; L += NT) S.sLay[L] = cp->layer_start[L];
    }
    const int64_t coll = rs->coll_step;
    const int cur = (int)(coll & 1);
    const int64_t md0 = rs->md_step;
    const int nmd = D.n_md;
    const gptr<Rec<T>> rb = G(recs<T>(D, cur));
    const gptr<const uint32_t> cand = G(D.cand_idx);

    bool valid[K];
    int64_t idx[K];
    T x[K][3], v[K][3], x0[K][3];
    double f[K][3];
    uint8_t st[K];
    uint32_t pid[K];
    bool inside[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        int64_t pos = (int64_t)g * B + (int64_t)t * K + j;
        valid[j] = pos < ncand;
        idx[j] = valid[j] ? (int64_t)cand[pos] : 0;
        for (int d = 0; d < 3; ++d) {
            x[j][d] = valid[j] ? rb[idx[j]].x[d] : (T)0;
            v[j][d] = valid[j] ? rb[idx[j]].v[d] : (T)0;
        }
        st[j] = valid[j] ? (uint8_t)(rb[idx[j]].st & 3u) : (uint8_t)0;
        pid[j] = valid[j] ? rb[idx[j]].id : 0;
        for (int d = 0; d < 3; ++d) x0[j][d] = x[j][d];
    }
    __syncthreads();
    // this wave's colloids within reach for the interval
    uint32_t wmask = reach_box<T, K>(S, S.sXw[0], cc, nc, valid, x);
    const double me2 = D.cull_me * D.cull_me;
    // Roles: with one workgroup, or in the solo form, every workgroup
    // completes the exchange and updates the colloids itself; otherwise
    // workgroup 0 (the master) does, and the others take the colloid
    // positions of each MD step from its broadcast.
    const int Qx = Gpad > 64 ? Gpad / 64 : 1;
    const bool solo = Qx == 1 && 3 * nc + 1 <= 8;
    const bool worker = Gact > 1 && !solo && g != 0;
    const bool updates = !worker;
    uint32_t nbar = 0;
    // barrier epochs: unique per barrier of the replica between list
    // rebuilds (md_step + coll_step grows by n_md + 1 per interval)
    const uint32_t epoch0 = (uint32_t)(md0 + coll);
    const double dt = D.dt;
    const T dtT = (T)dt, hT = (T)D.h;
    const T Lt[3] = {(T)cc.L(0), (T)cc.L(1), (T)cc.L(2)};
    const bool colloid_wave = t < 64;

    // forces at the start of the interval
    chain_compute<T, K, NT>(S, S.sXw[0], cc, cp, nc, valid, x, x0, st, f, inside, g, Gact, solo, wmask, me2, nbar, epoch0);
    if (updates) chain_collect<T, K, NT>(S, S.sXw[0], cc, cp, nc, g, Gact, Gpad, nbar, epoch0, false, cF, PL);
    // list entries: first half kick and drift of step 0
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            v[j][d] = tfma(hT, (T)f[j][d], v[j][d]);
            x[j][d] = wrap_coord<T>(tfma(dtT, v[j][d], x[j][d]), Lt[d]);
        }

    double eu = 0.0, ef = 0.0;
    // The loop's code starts on a 64-byte line, in the one- and two-colloid
    // variants 16 bytes into it: where its branch targets fall in a line of the
    // instruction fetch changes a step's time by up to 3 % (32^3 with one dimer
    // FP64 289 us an interval, 286 so; iterative RATTLE 6890 and with the 16 bytes
    // 7120), and would otherwise follow from the length of the code before it.
    [[clang::code_align(64)]]
    for (int step = 0; step < nmd; ++step) {
        if constexpr (NC > 0) __asm__ __volatile__(".rept 4\n s_nop 0\n .endr");
        double (*Xw)[3] = S.sXw[(step + 1) & 1];
        const int64_t md = md0 + step;
        // colloids (wave 0, in registers): half kick, drift, RATTLE
        // position stage, periodic images for the force evaluation
        if (worker) {
            if (colloid_wave) await_images(S, Xw, cc, nc, nbar, epoch0);
        } else if (colloid_wave) {
            double cXo[3];
            if (t < nc) {
                for (int d = 0; d < 3; ++d) {
                    cV[d] = fma(chc, cF[d], cV[d]);
                    cXo[d] = cX[d];
                    cX[d] = fma(dt, cV[d], cX[d]);
                }
            } else {
                for (int d = 0; d < 3; ++d) cXo[d] = cX[d];
            }
            uint32_t lflags = 0;
            if (iter) {
                // bond network: wave 0 sweeps over the bonds on the
                // colloid state staged in LDS
                if (t < nc)
                    for (int d = 0; d < 3; ++d) {
                        S.sXc[t][d] = cX[d];
                        S.sVc[t][d] = cV[d];
                        S.sXoc[t][d] = cXo[d];
                    }
                wave_sync();
                {
                    const uint32_t f = rattle_pos_iter(S, cp, dt);   // all lanes of wave 0
                    if (t == 0) lflags |= f;
                }
                wave_sync();
                if (t < nc)
                    for (int d = 0; d < 3; ++d) {
                        cX[d] = S.sXc[t][d];
                        cV[d] = S.sVc[t][d];
                    }
            } else {
                rattle_pos_lane(BL, dt, cX, cV, cXo, lflags);
            }
            if (lflags) atomicOr(&S.sflags, lflags);
            if (t < nc) {
                for (int d = 0; d < 3; ++d) Xw[t][d] = colloid_image(cX[d], cc.L(d));
                // a colloid beyond half the skin from its interval-start
                // position voids the reach masks of the interval
                const double dx = cX[0] - cX0[0], dy = cX[1] - cX0[1], dz = cX[2] - cX0[2];
                if (dot3(dx, dy, dz, dx, dy, dz) >= D.skin_half2) S.sFull = 1u;
                S.sPairMask[t] = 0u;
            }
            if (Gact > 1 && !solo) {
                wave_sync();
                broadcast_images(S, Xw, cc, nc, nbar, epoch0);
            }
        }
        __syncthreads();
        chain_compute<T, K, NT>(S, Xw, cc, cp, nc, valid, x, x0, st, f, inside, g, Gact, solo, wmask, me2, nbar,
                                epoch0);
        // while the other workgroups' sums arrive: the list entries' second
        // half kick, catalysis, and (except after the last step) the next
        // step's first half kick and drift -- each entry's own arithmetic,
        // in the same order as a step-by-step update
#pragma unroll
        for (int j = 0; j < K; ++j)
#pragma unroll
            for (int d = 0; d < 3; ++d) v[j][d] = tfma(hT, (T)f[j][d], v[j][d]);
        // catalysis: A inside a catalytic sphere is flagged; a flagged A
        // outside all of them converts to B with probability cat_prob
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (!valid[j]) continue;
            uint8_t s = st[j];
            if (s & 1) continue;
            if (inside[j]) {
                st[j] = (uint8_t)(s | 2);
            } else if (s & 2) {
                bool flip = true;
                if (cc.cat_prob() < 1.0) {
                    uint64_t wv[4];
                    philox((uint64_t)md, pid[j], 0, cc.seed(), TAG_CAT, wv);
                    flip = u01(wv[0]) < cc.cat_prob();
                }
                if (flip) {
                    st[j] = 1;
                    ef += 1.0;
                    eu += species_dU_lds(S, Xw, cc, wmask, (double)x[j][0], (double)x[j][1], (double)x[j][2]);
                } else {
                    st[j] = 0;
                }
            }
        }
        if (step < nmd - 1) {
#pragma unroll
            for (int j = 0; j < K; ++j)
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    v[j][d] = tfma(hT, (T)f[j][d], v[j][d]);
                    x[j][d] = wrap_coord<T>(tfma(dtT, v[j][d], x[j][d]), Lt[d]);
                }
        }
        // the potential energy is an observable of the last force evaluation
        if (updates)
            chain_collect<T, K, NT>(S, Xw, cc, cp, nc, g, Gact, Gpad, nbar, epoch0, step == nmd - 1, cF, PL);
        // colloids (wave 0, in registers): second half kick, RATTLE
        // velocity stage, Verlet-list soundness check (displacement within
        // the interval)
        if (updates && colloid_wave) {
            if (t < nc)
                for (int d = 0; d < 3; ++d) cV[d] = fma(chc, cF[d], cV[d]);
            if (iter) {
                if (t < nc)
                    for (int d = 0; d < 3; ++d) {
                        S.sXc[t][d] = cX[d];
                        S.sVc[t][d] = cV[d];
                    }
                wave_sync();
                uint32_t vflags = 0;
                vflags = rattle_vel_iter(S, cp, dt);
                if (t != 0) vflags = 0;
                if (vflags) atomicOr(&S.sflags, vflags);
                wave_sync();
                if (t < nc)
                    for (int d = 0; d < 3; ++d) cV[d] = S.sVc[t][d];
            } else {
                rattle_vel_lane(BL, cX, cV);
            }
            if (t < nc) {
                double dx = cX[0] - cX0[0], dy = cX[1] - cX0[1], dz = cX[2] - cX0[2];
                if (dot3(dx, dy, dz, dx, dy, dz) >= D.skin_half2)
                    atomicOr(&S.sflags, RMP_FLAG_DISPLACEMENT);
            }
        }
    }
    __syncthreads();
    // write back list entries and bin them for the coming collision
    const double s3[3] = {rs->shift[0], rs->shift[1], rs->shift[2]};
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (!valid[j]) continue;
        const int64_t i = idx[j];
        for (int d = 0; d < 3; ++d) {
            rb[i].x[d] = x[j][d];
            rb[i].v[d] = v[j][d];
        }
        rb[i].st = (uint32_t)st[j] & 3u;
        uint32_t key = cell_key(D, (double)x[j][0], (double)x[j][1], (double)x[j][2], s3);
        const uint32_t rank = __hip_atomic_fetch_add(G(D.count) + key, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        G(D.keyrank)[i] = ((uint64_t)key << 32) | rank;
    }
    // reaction bookkeeping of this workgroup (combined after the collision)
    __shared__ double sred[NT / 64 + 1];
    eu = block_sum<NT>(eu, sred);
    ef = block_sum<NT>(ef, sred);
    if (t == 0) {
        G(D.epart)[(int64_t)g * 2 + 0] = eu;
        G(D.epart)[(int64_t)g * 2 + 1] = ef;
        if (S.sflags) atomicOr(&rs->flags, S.sflags);
    }
    if (g == 0) {
        if (t < nc) {
            bool fin = true;
            for (int d = 0; d < 3; ++d) {
                rs->X[t][d] = cX[d];
                rs->V[t][d] = cV[d];
                rs->F[t][d] = cF[d];
                fin = fin && isfinite(cF[d]);
            }
            if (!fin) atomicOr(&rs->flags, RMP_FLAG_NONFINITE);
        }
        if (t == 0) {
            rs->U = S.sU;
            rs->md_step = md0 + nmd;
            rs->n_cand_used = ncand;
        }
    }
}

// Work-list position of a chain workgroup.  When every workgroup of the
// launch fits on the device at once it is blockIdx.  Otherwise (TICKET)
// workgroups take their positions in the order they start running, from a
// device counter: the workgroups of one system hold consecutive positions,
// so every system whose positions have all been taken is entirely resident
// and its exchange waits end, even though the launch runs in waves.  The
// last workgroup to finish puts the counters back to zero for the next
// launch.  (The ticket is a separate instantiation because an atomic at
// kernel entry keeps the descriptor loads of the whole kernel off the
// scalar unit.)
template <class T, int K, int NC, int NT>
__device__ __forceinline__ void chain_run(Work w, int item)
{
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int g = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    chain_body<T, K, NC, NT>(w, g, D, chain_const(D, w.budget));
}

// Waves per SIMD that the chain's registers leave room for: two (one with four
// entries per thread).  Launches in waves of one- and two-colloid systems take
// three, so that more systems run at once (64 dimer systems, one interval:
// FP64 1989 -> 1921 us, FP32 1752 -> 1619; four spill: 2090).
constexpr int chain_waves(int k, bool ticket, int nc) { return k == 4 ? 1 : ticket && nc > 0 ? 3 : 2; }

template <class T, int K, bool TICKET, int NC, int NT>
__global__ __launch_bounds__(NT, chain_waves(K, TICKET, NC)) void k_chain(Work w)
{
    // only in the one- and two-colloid variants: with the priority code in
    // the generic variant its 128^3 launches ran 10 % slower even with the
    // flag off
    if constexpr (!TICKET && NC > 0) {
        // the workgroups past the chain's stream, where the streaming shares
        // the launch (they start after the chain's and wait for nothing)
        const int sb = (int)blockIdx.x - w.n_chain;
        if (sb >= 0) {
            stream_body<T, 1, false, NT>(w.desc, w.chunks, w.nrep, xcd_range(sb, (int)gridDim.x - w.n_chain),
                                         CHUNK / NT);
            return;
        }
    }
    if constexpr (NC > 0)
        if (w.flags & WORK_CHAIN_PRIO) __builtin_amdgcn_s_setprio(3);
    if (!TICKET) {
        chain_run<T, K, NC, NT>(w, (int)blockIdx.x);
        return;
    }
    __shared__ int s_item;
    if (threadIdx.x == 0)
        s_item = (int)__hip_atomic_fetch_add(&w.tick[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    chain_run<T, K, NC, NT>(w, s_item);
    if (threadIdx.x == 0) {
        const uint32_t fin = __hip_atomic_fetch_add(&w.tick[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (fin == gridDim.x - 1) {
            __hip_atomic_store(&w.tick[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&w.tick[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// explicit instances: X(T, K, TICKET, NC, NT) for every shape of type T
#define RMP_CHAIN_SHAPE(X, T, K, NT)                                             \
    X(T, K, false, 0, NT) X(T, K, false, 1, NT) X(T, K, false, 2, NT)            \
    X(T, K, true, 0, NT) X(T, K, true, 1, NT) X(T, K, true, 2, NT)
#define RMP_CHAIN_SHAPES(X, T)                                                   \
    RMP_CHAIN_SHAPE(X, T, 1, 256) RMP_CHAIN_SHAPE(X, T, 2, 256)                  \
    RMP_CHAIN_SHAPE(X, T, 4, 256) RMP_CHAIN_SHAPE(X, T, 1, 512)                  \
    RMP_CHAIN_SHAPE(X, T, 2, 512)
#define RMP_CHAIN_DECL(T, K, TICKET, NC, NT)                                     \
    extern template __global__ void k_chain<T, K, TICKET, NC, NT>(Work);
#define RMP_CHAIN_DEF(T, K, TICKET, NC, NT)                                      \
    template __global__ void k_chain<T, K, TICKET, NC, NT>(Work);

}  // namespace rmp
