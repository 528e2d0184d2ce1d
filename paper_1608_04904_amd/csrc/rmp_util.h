// Device helpers shared by the kernels: wave and block reductions, scans,
// the cell key, the Verlet-list test, streaming and in-cell ranks.
#pragma once
#include "rmp_device.h"

namespace rmp {

// ------------------------------------------------------------------ utils

// Pairwise binary tree over the 64 lanes of a wave with DPP moves:
// xor 1 and xor 2 (quad permutes), 4-blocks (half-row mirror), 8-blocks (row
// mirror), 16-blocks (row broadcast of lane 15 into rows 1 and 3), and the
// two 32-blocks combined from lanes 31 and 63.  Each level adds the value of
// the adjacent block of the same size, so the result is the tree
// node(l, j) = node(l-1, 2j) + node(l-1, 2j+1) over lanes; it is returned in
// every lane.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_d(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double wave_tree_sum(double v)
{
    v = v + dpp_d<0xB1, 0xF>(v);     // quad_perm [1,0,3,2]
    v = v + dpp_d<0x4E, 0xF>(v);     // quad_perm [2,3,0,1]
    v = v + dpp_d<0x141, 0xF>(v);    // row_half_mirror
    v = v + dpp_d<0x140, 0xF>(v);    // row_mirror
    v = v + dpp_d<0x142, 0xA>(v);    // row_bcast15 into rows 1 and 3
    const double a = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 31),
                                      __builtin_amdgcn_readlane(__double2loint(v), 31));
    const double b = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                                      __builtin_amdgcn_readlane(__double2loint(v), 63));
    return a + b;
}

// wave_tree_sum of N = 4 or 8 values, lane l returning that of value l % N: at
// each of the first levels a lane keeps one of two values and gives the other
// to its partner, so that a level handles half the values of the one before
// (8 values: 64 instructions, one after the other 160).  The same two operands
// are added at every level as above.
__device__ __forceinline__ double sel_d(bool c, double a, double b)
{
    return __hiloint2double(c ? __double2hiint(a) : __double2hiint(b), c ? __double2loint(a) : __double2loint(b));
}

// the value of lane l ^ 4
__device__ __forceinline__ int dpp_xor4(int v)
{
    const int up = __builtin_amdgcn_update_dpp(0, v, 0x104, 0xF, 0x5, false);    // row_shl:4 into banks 0, 2
    return __builtin_amdgcn_update_dpp(up, v, 0x114, 0xF, 0xA, false);           // row_shr:4 into banks 1, 3
}

// x of the lanes' 16- or 32-lane block and of the adjacent one, added
template <int B>
__device__ __forceinline__ double add_block(double v)
{
    const uint32_t lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
    if constexpr (B == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
    } else {
        const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
    }
}

template <int N>
__device__ __forceinline__ double wave_tree_spread(const double (&v)[N])
{
    static_assert(N == 4 || N == 8, "values");
    const int lane = threadIdx.x & 63;
    const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0, b2 = (lane & 4) != 0;
    double w[N / 2], u[N / 4];
#pragma unroll
    for (int i = 0; i < N / 2; ++i)
        w[i] = sel_d(b0, v[2 * i + 1], v[2 * i]) + dpp_d<0xB1, 0xF>(sel_d(b0, v[2 * i], v[2 * i + 1]));
#pragma unroll
    for (int i = 0; i < N / 4; ++i)
        u[i] = sel_d(b1, w[2 * i + 1], w[2 * i]) + dpp_d<0x4E, 0xF>(sel_d(b1, w[2 * i], w[2 * i + 1]));
    double q = u[0], p = u[0];
    if constexpr (N == 8) {
        q = sel_d(b2, u[1], u[0]);
        p = sel_d(b2, u[0], u[1]);
    }
    q = q + __hiloint2double(dpp_xor4(__double2hiint(p)), dpp_xor4(__double2loint(p)));
    q = q + dpp_d<0x128, 0xF>(q);                                                // row_ror:8
    return add_block<32>(add_block<16>(q));
}

// minimum of lo and maximum of hi over the 64 lanes (DPP within rows of 16,
// then the four rows' results read from lanes 15, 31, 47, 63); exact, in
// every lane
__device__ __forceinline__ void wave_min_max(double& lo, double& hi)
{
#define RMP_MM_STEP(CTRL)                                                       \
    {                                                                           \
        const double ol = dpp_d<CTRL, 0xF>(lo), oh = dpp_d<CTRL, 0xF>(hi);      \
        lo = ol < lo ? ol : lo;                                                 \
        hi = oh > hi ? oh : hi;                                                 \
    }
    RMP_MM_STEP(0xB1)       // quad_perm [1,0,3,2]
    RMP_MM_STEP(0x4E)       // quad_perm [2,3,0,1]
    RMP_MM_STEP(0x141)      // row_half_mirror
    RMP_MM_STEP(0x140)      // row_mirror
#undef RMP_MM_STEP
    double l = lo, h = hi;
#pragma unroll
    for (int r = 15; r < 64; r += 16) {
        const double rl = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(lo), r),
                                           __builtin_amdgcn_readlane(__double2loint(lo), r));
        const double rh = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(hi), r),
                                           __builtin_amdgcn_readlane(__double2loint(hi), r));
        l = rl < l ? rl : l;
        h = rh > h ? rh : h;
    }
    lo = l;
    hi = h;
}

// minimum of lo and maximum of hi over the 64 lanes, for integers (same
// pattern as wave_min_max)
__device__ __forceinline__ void wave_min_max_i(int& lo, int& hi)
{
#define RMP_MMI_STEP(CTRL)                                                      \
    {                                                                           \
        const int ol = __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xF, 0xF, false);  \
        const int oh = __builtin_amdgcn_update_dpp(0, hi, CTRL, 0xF, 0xF, false);  \
        lo = ol < lo ? ol : lo;                                                 \
        hi = oh > hi ? oh : hi;                                                 \
    }
    RMP_MMI_STEP(0xB1)
    RMP_MMI_STEP(0x4E)
    RMP_MMI_STEP(0x141)
    RMP_MMI_STEP(0x140)
#undef RMP_MMI_STEP
    int l = lo, h = hi;
#pragma unroll
    for (int r = 15; r < 64; r += 16) {
        const int rl = __builtin_amdgcn_readlane(lo, r), rh = __builtin_amdgcn_readlane(hi, r);
        l = rl < l ? rl : l;
        h = rh > h ? rh : h;
    }
    lo = l;
    hi = h;
}

// maximum of v over the 64 lanes (exact), in every lane
__device__ __forceinline__ double wave_max_d(double v)
{
#define RMP_MX_STEP(CTRL)                                                       \
    {                                                                           \
        const double o = dpp_d<CTRL, 0xF>(v);                                   \
        v = o > v ? o : v;                                                      \
    }
    RMP_MX_STEP(0xB1)
    RMP_MX_STEP(0x4E)
    RMP_MX_STEP(0x141)
    RMP_MX_STEP(0x140)
#undef RMP_MX_STEP
    double m = v;
#pragma unroll
    for (int r = 15; r < 64; r += 16) {
        const double o = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), r),
                                          __builtin_amdgcn_readlane(__double2loint(v), r));
        m = o > m ? o : m;
    }
    return m;
}

// deterministic block sum: wave butterfly, then a pairwise tree over the
// wave sums (xor butterfly over the first NT/64 lanes of wave 0)
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* sbuf)
{
    v = wave_tree_sum(v);
    constexpr int NW = NT / 64;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) sbuf[wave] = v;
    __syncthreads();
    if (NW > 1) {
        if (wave == 0) {
            double a = lane < NW ? sbuf[lane] : 0.0;
#pragma unroll
            for (int m = 1; m < NW; m <<= 1) a = a + __shfl_xor(a, m, 64);
            if (lane == 0) sbuf[NW] = a;
        }
        __syncthreads();
    }
    double r = sbuf[NW > 1 ? NW : 0];
    __syncthreads();
    return r;
}

// N sums over the workgroup; sbuf holds (NT / 64 + 1) * N doubles.  Every
// thread receives the totals.
template <int NT, int N>
__device__ __forceinline__ void block_sum_n(double (&v)[N], double* sbuf)
{
    constexpr int NW = NT / 64;
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] = wave_tree_sum(v[q]);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0)
#pragma unroll
        for (int q = 0; q < N; ++q) sbuf[wave * N + q] = v[q];
    __syncthreads();
    if (threadIdx.x < N) {
        double a = 0.0;
#pragma unroll 4
        for (int w = 0; w < NW; ++w) a = a + sbuf[w * N + threadIdx.x];
        sbuf[NW * N + threadIdx.x] = a;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] = sbuf[NW * N + q];
    __syncthreads();
}

template <int NT>
__device__ __forceinline__ uint32_t block_sum_u32(uint32_t v, uint32_t* sbuf)
{
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m, 64);
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sbuf[wave] = v;
    __syncthreads();
    uint32_t r = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) r += sbuf[k];
    __syncthreads();
    return r;
}

// ordering of LDS accesses between lanes of one wave (no workgroup barrier)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a value known to be the same in all lanes, in scalar registers
__device__ __forceinline__ uint64_t uniform_u64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ double uniform_d(double v)
{
    return __longlong_as_double((long long)uniform_u64((uint64_t)__double_as_longlong(v)));
}

// exclusive block scan of u32, returns the prefix of this thread; *total set
template <int NT>
__device__ __forceinline__ uint32_t block_exscan_u32(uint32_t v, uint32_t* sbuf, uint32_t* total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        uint32_t o = __shfl_up(inc, m, 64);
        if (lane >= m) inc += o;
    }
    __syncthreads();
    if (lane == 63) sbuf[wave] = inc;
    __syncthreads();
    uint32_t wpre = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) {
        if (k < wave) wpre += sbuf[k];
        tot += sbuf[k];
    }
    __syncthreads();
    *total = tot;
    return wpre + inc - v;
}

__device__ __forceinline__ void shift_of(uint64_t seed, int64_t coll, double s[3])
{
    uint64_t w[4];
    philox((uint64_t)coll, 0, 0, seed, TAG_SHIFT, w);
    s[0] = u01(w[0]);
    s[1] = u01(w[1]);
    s[2] = u01(w[2]);
}

// Sort key of the shifted cell holding (x0, x1, x2): its linear index
// x + Lx (y + Ly z) in the row-major order; in the compact-Hilbert order its
// rank along the curve, computed for a cubic power-of-two box and otherwise
// looked up by the linear index.
// FLOW false: known not to be a flow (no plates).
template <bool FLOW = true>
__device__ __forceinline__ uint32_t cell_key(const RepDesc& D, double x0, double x1, double x2,
                                             const double s[3])
{
    int c[3];
    const double xs[3] = {x0, x1, x2};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double fq = floor(xs[d] - s[d]);
        const bool in = fq >= -1.0 && fq < D.Ld[d];        // NaN-safe
        const int q = in ? (int)fq : (FLOW && d == 2 && D.walls ? -1 : 0);
        // plates: layers floor(z - s) + 1 in [0, L_z], not periodic
        c[d] = FLOW && d == 2 && D.walls ? q + 1 : (q < 0 ? q + D.L[d] : q);
    }
    const uint32_t lin = (uint32_t)c[0] + (uint32_t)D.L[0] * ((uint32_t)c[1] + (uint32_t)D.L[1] * (uint32_t)c[2]);
    if (D.hbits == KEY_ROW) return lin;
    if (D.hbits >= 0) return hilbert_index((uint32_t)c[0], (uint32_t)c[1], (uint32_t)c[2], D.hbits);
    return D.rank_of[lin];
}

// Verlet-list membership for the coming interval of length tau: flagged
// particles, or r_ic^2 < (r_cut,c + skin + |v| tau)^2 for some colloid c.
__device__ __forceinline__ bool is_candidate(const RepDesc& D, const ColloidParams* cp, int nc,
                                             const double (*Xw)[3], uint8_t st,
                                             double x0, double x1, double x2,
                                             double v0, double v1, double v2)
{
    if (D.flow) return false;     // flows: no colloids, every particle streams
    if (st & 2) return true;
    if (nc == 0) return false;
    double vv = dot3(v0, v1, v2, v0, v1, v2);
    double reach = sqrt(vv) * D.tau;
    for (int c = 0; c < nc; ++c) {
        double dx = min_image(x0 - Xw[c][0], D.Ld[0], D.halfL[0]);
        double dy = min_image(x1 - Xw[c][1], D.Ld[1], D.halfL[1]);
        double dz = min_image(x2 - Xw[c][2], D.Ld[2], D.halfL[2]);
        double r2 = dot3(dx, dy, dz, dx, dy, dz);
        double tt = cp->reachR[c] + reach;
        if (r2 < tt * tt) return true;
    }
    return false;
}

// potential change of a solvent particle whose species changes (bookkeeping)
__device__ __forceinline__ double species_dU(const RepDesc& D, const ColloidParams* cp, int nc,
                                             const double (*Xw)[3], double x0, double x1,
                                             double x2, int from, int to)
{
    double du = 0.0;
    for (int c = 0; c < nc; ++c) {
        double dx = min_image(x0 - Xw[c][0], D.Ld[0], D.halfL[0]);
        double dy = min_image(x1 - Xw[c][1], D.Ld[1], D.halfL[1]);
        double dz = min_image(x2 - Xw[c][2], D.Ld[2], D.halfL[2]);
        double r2 = dot3(dx, dy, dz, dx, dy, dz);
        if (r2 < cp->rc2[c]) {
            double cf, p0, p1;
            wca(r2, cp->sig2[c], from ? cp->epsB[c] : cp->epsA[c], cf, p0);
            wca(r2, cp->sig2[c], to ? cp->epsB[c] : cp->epsA[c], cf, p1);
            du += p1 - p0;
        }
    }
    return du;
}

// list bits of the interval that ends in collision `coll`
__device__ __forceinline__ uint64_t* list_bits(const RepDesc& D, int64_t coll)
{
    return D.lbits + (coll & 1) * (int64_t)(CHUNK / 64) * D.n_chunks;
}

// the records of buffer b
template <class T>
__device__ __forceinline__ Rec<T>* recs(const RepDesc& D, int b)
{
    return reinterpret_cast<Rec<T>*>(D.rec[b]);
}

// ------------------------------------------------------- free streaming

// One streaming step under the constant acceleration g, with the plates at
// z = 0 and z = L_z when present: half kick, drift, half kick; a drift that
// crosses a plate is cut at the crossing time, the velocity reversed
// (bounce-back) and the rest of the step travelled back.
template <class T>
__device__ __forceinline__ T below(T L);
template <>
__device__ __forceinline__ double below<double>(double L) { return nextafter(L, 0.0); }
template <>
__device__ __forceinline__ float below<float>(float L) { return nextafterf(L, 0.0f); }

template <class T>
__device__ __forceinline__ void flow_step(T (&x)[3], T (&v)[3], const T (&g)[3], T dt, T hdt,
                                          const T (&L)[3], bool walls)
{
    T y[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        v[d] = tfma(hdt, g[d], v[d]);
        y[d] = tfma(dt, v[d], x[d]);
    }
    if (walls) {
        if (y[2] < (T)0 || y[2] >= L[2]) {
            const T wz = y[2] < (T)0 ? (T)0 : L[2];
            const T ts = (wz - x[2]) / v[2];
            const T rem = dt - ts;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const T xc = tfma(ts, v[d], x[d]);
                v[d] = -v[d];
                y[d] = tfma(rem, v[d], xc);
            }
            if (y[2] >= L[2]) y[2] = below<T>(L[2]);
            if (y[2] < (T)0) y[2] = (T)0;
        }
        x[0] = wrap_coord<T>(y[0], L[0]);
        x[1] = wrap_coord<T>(y[1], L[1]);
        x[2] = y[2];
    } else {
#pragma unroll
        for (int d = 0; d < 3; ++d) x[d] = wrap_coord<T>(y[d], L[d]);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) v[d] = tfma(hdt, g[d], v[d]);
}

// Streaming of P particles over an interval in registers (those with go[u];
// all lanes of a wave call it).  Flows (constant acceleration, plates) take
// n_md flow_steps.  Otherwise a particle outside the Verlet list feels no
// force: n_md drifts x <- fma(dt, v, x) with a periodic wrap after each.
//
// A coordinate moving down is negated (rounding is symmetric), so every
// coordinate m grows by |v| dt per step and leaves the box at one upper bound:
// moving up at m >= L, moving down at -m < 0, that is m >= the smallest
// positive number; either way the wrap is then m - L (and -L, where y + L
// rounded to L and the wrap subtracts L again, becomes zero).  If no lane's m
// is outside after all n_md drifts, none wrapped (a coordinate moving down that
// ends exactly on zero counts as outside there, since -m would be -0); otherwise
// the drifts are done again in runs of DRIFT_RUN, and a run in which a
// coordinate of some lane left the box once more for that coordinate with the
// wrap after each drift, without branches.  (Doing all n_md drifts again with
// branches, one coordinate after the other, held up whole collision tiles behind
// one wave.)  A coordinate that starts outside the box, or a step longer than it,
// takes the drifts as they are defined (drift_wrapped).
constexpr int DRIFT_RUN = 10;

template <class T> __device__ __forceinline__ T tiny();
template <> __device__ __forceinline__ double tiny<double>() { return 4.9406564584124654e-324; }
template <> __device__ __forceinline__ float tiny<float>() { return 1.401298464e-45f; }

// the drifts as they are defined, for a coordinate outside the box or a step
// beyond its edge (both leave it outside)
template <class T, int P>
__device__ __forceinline__ void drift_wrapped(int nmd, T dt, const T (&Lt)[3], T (&x)[P][3], const T (&v)[P][3],
                                              const bool (&go)[P])
{
    for (int k = 0; k < nmd; ++k)
#pragma unroll
        for (int u = 0; u < P; ++u)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const T y = wrap_coord<T>(tfma(dt, v[u][d], x[u][d]), Lt[d]);
                x[u][d] = go[u] ? y : x[u][d];
            }
}

template <class T, int P, bool FLOW = true>
__device__ __forceinline__ void advance(const RepDesc& D, T (&x)[P][3], T (&v)[P][3], const bool (&go)[P])
{
    const int nmd = D.n_md;
    const T dt = (T)D.dt;
    const T Lt[3] = {(T)D.Ld[0], (T)D.Ld[1], (T)D.Ld[2]};
    if (FLOW && D.flow) {
        const T g[3] = {(T)D.g[0], (T)D.g[1], (T)D.g[2]};
        const T hdt = (T)(0.5 * D.dt);
#pragma unroll
        for (int u = 0; u < P; ++u)
            if (go[u])
                for (int k = 0; k < nmd; ++k) flow_step<T>(x[u], v[u], g, dt, hdt, Lt, D.walls != 0);
        return;
    }
    T m[P][3];
#pragma unroll
    for (int u = 0; u < P; ++u)
#pragma unroll
        for (int d = 0; d < 3; ++d) m[u][d] = v[u][d] < (T)0 ? -x[u][d] : x[u][d];
    {
        T z[P][3];
#pragma unroll
        for (int u = 0; u < P; ++u)
#pragma unroll
            for (int d = 0; d < 3; ++d) z[u][d] = m[u][d];
#pragma unroll 5
        for (int k = 0; k < nmd; ++k)
#pragma unroll
            for (int u = 0; u < P; ++u)
#pragma unroll
                for (int d = 0; d < 3; ++d) z[u][d] = tfma(dt, tabs(v[u][d]), z[u][d]);
        bool out = false, odd = false;
#pragma unroll
        for (int u = 0; u < P; ++u)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                out = out || (go[u] && z[u][d] >= (v[u][d] < (T)0 ? (T)0 : Lt[d]));
                odd = odd || (go[u] && !(m[u][d] > (v[u][d] < (T)0 ? -Lt[d] : -tiny<T>())));
            }
        if (__ballot(out || odd) == 0ull) {
#pragma unroll
            for (int u = 0; u < P; ++u)
#pragma unroll
                for (int d = 0; d < 3; ++d) x[u][d] = go[u] ? (v[u][d] < (T)0 ? -z[u][d] : z[u][d]) : x[u][d];
            return;
        }
    }
    {
        bool odd = false;
#pragma unroll
        for (int u = 0; u < P; ++u)
#pragma unroll
            for (int d = 0; d < 3; ++d)
                odd = odd || (go[u] && (!(m[u][d] > (v[u][d] < (T)0 ? -Lt[d] : -tiny<T>())) ||
                                        !(dt * tabs(v[u][d]) < Lt[d])));
        if (__ballot(odd) != 0ull) {
            drift_wrapped<T, P>(nmd, dt, Lt, x, v, go);
            return;
        }
    }
    for (int k0 = 0; k0 < nmd; k0 += DRIFT_RUN) {
        const int nk = nmd - k0 < DRIFT_RUN ? nmd - k0 : DRIFT_RUN;
        T z[P][3];
#pragma unroll
        for (int u = 0; u < P; ++u)
#pragma unroll
            for (int d = 0; d < 3; ++d) z[u][d] = m[u][d];
#pragma unroll 2
        for (int k = 0; k < nk; ++k)
#pragma unroll
            for (int u = 0; u < P; ++u)
#pragma unroll
                for (int d = 0; d < 3; ++d) z[u][d] = tfma(dt, tabs(v[u][d]), z[u][d]);
#pragma unroll
        for (int u = 0; u < P; ++u)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const T top = v[u][d] < (T)0 ? tiny<T>() : Lt[d];
                if (__ballot(go[u] && z[u][d] >= top) != 0ull) {
                    T y = m[u][d];
                    for (int k = 0; k < nk; ++k) {
                        y = tfma(dt, tabs(v[u][d]), y);
                        T w = y - Lt[d];
                        w = w <= -Lt[d] ? (T)0 : w;
                        y = y >= top ? w : y;
                    }
                    z[u][d] = y;
                }
                m[u][d] = z[u][d];
            }
    }
#pragma unroll
    for (int u = 0; u < P; ++u)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const T y = v[u][d] < (T)0 ? (T)0 - m[u][d] : m[u][d];
            x[u][d] = go[u] ? y : x[u][d];
        }
}

// Workgroups are dealt to the eight XCDs in turn: work item of workgroup b of
// a launch of g such that each XCD takes a contiguous range of items, so that
// neighbouring items, which touch the same lines, share an L2.
__device__ __forceinline__ int xcd_range(unsigned b, unsigned g)
{
    const unsigned x = b & 7u, per = g >> 3, rem = g & 7u;
    return (int)(x * per + (x < rem ? x : rem) + (b >> 3));
}

}  // namespace rmp
