// Device helpers shared by the kernels: wave and block reductions, scans,
// the cell key, the Verlet-list test.
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

// wave_tree_sum of N independent values, level by level so that the N
// dependent chains overlap (each value's additions are the same as above)
template <int N>
__device__ __forceinline__ void wave_tree_sum_n(double (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = v[i] + dpp_d<0xB1, 0xF>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = v[i] + dpp_d<0x4E, 0xF>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = v[i] + dpp_d<0x141, 0xF>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = v[i] + dpp_d<0x140, 0xF>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = v[i] + dpp_d<0x142, 0xA>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const double a = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v[i]), 31),
                                          __builtin_amdgcn_readlane(__double2loint(v[i]), 31));
        const double b = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v[i]), 63),
                                          __builtin_amdgcn_readlane(__double2loint(v[i]), 63));
        v[i] = a + b;
    }
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
__device__ __forceinline__ uint32_t cell_key(const RepDesc& D, double x0, double x1, double x2,
                                             const double s[3])
{
    int64_t c[3];
    const double xs[3] = {x0, x1, x2};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double fq = floor(xs[d] - s[d]);
        if (d == 2 && D.walls) {
            // plates: layers floor(z - s) + 1 in [0, L_z], not periodic
            c[d] = (fq >= -1.0 && fq < (double)(D.L[d] - 1)) ? (int64_t)fq + 1 : 0;
            continue;
        }
        int64_t q = (fq >= -1.0 && fq < (double)D.L[d]) ? (int64_t)fq : 0;   // NaN-safe
        if (q < 0) q += D.L[d];
        c[d] = q;
    }
    const uint32_t lin = (uint32_t)(c[0] + (int64_t)D.L[0] * (c[1] + (int64_t)D.L[1] * c[2]));
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

template <class T>
__device__ __forceinline__ T* comp(void* base, int64_t n, int d)
{
    return reinterpret_cast<T*>(base) + (int64_t)d * n;
}

}  // namespace rmp
