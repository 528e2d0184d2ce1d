// gfx950 kernels of the MPCD+MD solvent path.
//
// One interval (paper, "Algorithms"): n_md velocity-Verlet steps with WCA
// colloid-solvent forces over a Verlet list built from the cell sort, exact
// RATTLE for dimers and catalytic conversion, then one MPCD collision on a
// randomly shifted grid with the RMPCD bulk reaction.  Kernels of one
// interval, in stream order:
//
//   k_stream_bin   particles outside the Verlet list: n_md drifts held in
//                  registers, then the cell key of the next collision and an
//                  atomic rank (HBM-bound, one pass over x, v)
//   k_chain        Verlet-list particles and colloids: n_md MD steps in
//                  persistent workgroups; colloid forces reduced with a fixed
//                  binary tree over list positions; inter-workgroup barrier
//                  per step when the list spans several workgroups
//   k_scan_*       exclusive scan of the cell counts -> cell_start
//   k_scatter      each particle's record (x, v, id, old index, state) to
//                  slot cell_start[key] + rank of the staging array
//   k_collide      per tile of cells: read the tile's records (contiguous),
//                  restore the stable (old-index) order inside each cell,
//                  FP64 centre-of-mass sums,
//                  rotation about a random axis (or Anderson thermostat),
//                  bulk B->A reaction, Verlet-list flags for the next
//                  interval, coalesced write of the cell-ordered arrays
//   k_chunk_scan   list compaction offsets, per-interval bookkeeping
//   k_cand_write   compacted Verlet list
//
// Data layout in HBM: structure-of-arrays, x[3][N] and v[3][N] in the
// storage precision (double or float), double-buffered across collisions.
#include "rmp_chain.h"

namespace rmp {

RMP_CHAIN_SHAPES(RMP_CHAIN_DECL, double)
RMP_CHAIN_SHAPES(RMP_CHAIN_DECL, float)

// ------------------------------------------------------------------- init

// Solvent initial state: uniform positions rejected inside colloid cores,
// Maxwellian velocities; per-chunk velocity sums for the mean removal.
template <class T>
__global__ __launch_bounds__(256) void k_init(const RepDesc* Dp)
{
    const RepDesc& D = *Dp;
    const ColloidParams* cp = D.cp;
    RepState* rs = D.rs;
    __shared__ double sXw[MAXC][3];
    __shared__ double sred[8];
    const int nc = cp->nc;
    const int t = threadIdx.x;
    if (t < nc)
        for (int d = 0; d < 3; ++d) sXw[t][d] = colloid_image(rs->X[t][d], D.Ld[d]);
    __syncthreads();
    const int64_t n = D.n;
    const int64_t base = (int64_t)blockIdx.x * CHUNK;
    double sum[3] = {0.0, 0.0, 0.0};
    bool bad = false;
    for (int j = t; j < CHUNK; j += 256) {
        int64_t i = base + j;
        if (i >= n) break;
        double xi[3] = {0.0, 0.0, 0.0};
        bool ok = false;
        for (uint64_t att = 0; att < 4096 && !ok; ++att) {
            uint64_t w[4];
            philox(att, (uint64_t)i, 0, D.seed, TAG_INIT_POS, w);
            for (int d = 0; d < 3; ++d) xi[d] = u01(w[d]) * D.Ld[d];
            ok = true;
            for (int c = 0; c < nc && ok; ++c) {
                double dx = min_image(xi[0] - sXw[c][0], D.Ld[0], D.halfL[0]);
                double dy = min_image(xi[1] - sXw[c][1], D.Ld[1], D.halfL[1]);
                double dz = min_image(xi[2] - sXw[c][2], D.Ld[2], D.halfL[2]);
                if (dot3(dx, dy, dz, dx, dy, dz) < cp->sig2[c]) ok = false;
            }
        }
        bad |= !ok;
        uint64_t w[4];
        double z[3];
        philox(0, (uint64_t)i, 0, D.seed, TAG_INIT_VEL, w);
        normals3(w, z);
        for (int d = 0; d < 3; ++d) {
            T xv = (T)xi[d];
            if (xv >= (T)D.Ld[d]) xv = (T)0;    // FP32 rounding up to L
            comp<T>(D.x[0], n, d)[i] = xv;
            T vv = (T)(D.vscale * z[d]);
            comp<T>(D.v[0], n, d)[i] = vv;
            sum[d] += (double)vv;
        }
        D.id[0][i] = (uint32_t)i;
        D.st[0][i] = 0;
    }
    if (bad) atomicOr(&rs->flags, RMP_FLAG_INIT);
    for (int d = 0; d < 3; ++d) {
        double s = block_sum<256>(sum[d], sred);
        if (t == 0) D.obs_part[(int64_t)blockIdx.x * 8 + d] = s;
    }
}

// mean velocity from the chunk sums (one workgroup)
__global__ __launch_bounds__(256) void k_init_mean(const RepDesc* Dp, double* mean_out)
{
    const RepDesc& D = *Dp;
    __shared__ double sred[8];
    for (int d = 0; d < 3; ++d) {
        double s = 0.0;
        for (int k = threadIdx.x; k < D.n_chunks; k += 256) s += D.obs_part[(int64_t)k * 8 + d];
        s = block_sum<256>(s, sred);
        if (threadIdx.x == 0) mean_out[d] = D.n > 0 ? s / (double)D.n : 0.0;
    }
}

template <class T>
__global__ __launch_bounds__(256) void k_init_sub(const RepDesc* Dp, const double* mean)
{
    const RepDesc& D = *Dp;
    const int64_t n = D.n;
    const int64_t base = (int64_t)blockIdx.x * CHUNK;
    for (int j = threadIdx.x; j < CHUNK; j += 256) {
        int64_t i = base + j;
        if (i >= n) break;
        for (int d = 0; d < 3; ++d) {
            T* v = comp<T>(D.v[0], n, d);
            v[i] = (T)((double)v[i] - mean[d]);
        }
    }
}

// ------------------------------------------------------- Verlet list build

// Stand-alone list flags (first interval, or a change of n_md).
template <class T>
__global__ __launch_bounds__(256) void k_list(Work w)
{
    const int item = blockIdx.x;
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int chunk = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active) return;
    const ColloidParams* cp = D.cp;
    RepState* rs = D.rs;
    __shared__ double sXw[MAXC][3];
    __shared__ uint32_t sred[4];
    const int nc = cp->nc;
    const int t = threadIdx.x;
    if (t < nc)
        for (int d = 0; d < 3; ++d) sXw[t][d] = colloid_image(rs->X[t][d], D.Ld[d]);
    __syncthreads();
    const int cur = (int)(rs->coll_step & 1);
    const int64_t n = D.n;
    const int64_t base = (int64_t)chunk * CHUNK;
    uint32_t cnt = 0;
    for (int j = t; j < CHUNK; j += 256) {
        int64_t i = base + j;
        if (i >= n) break;
        double x0 = comp<T>(D.x[cur], n, 0)[i], x1 = comp<T>(D.x[cur], n, 1)[i],
               x2 = comp<T>(D.x[cur], n, 2)[i];
        double v0 = comp<T>(D.v[cur], n, 0)[i], v1 = comp<T>(D.v[cur], n, 1)[i],
               v2 = comp<T>(D.v[cur], n, 2)[i];
        bool c = is_candidate(D, cp, nc, sXw, D.st[cur][i], x0, x1, x2, v0, v1, v2);
        D.cflag[i] = c ? 1 : 0;
        cnt += c ? 1u : 0u;
    }
    uint32_t tot = block_sum_u32<256>(cnt, sred);
    if (t == 0) D.chunk_cnt[chunk] = tot;
}

// Per replica (one workgroup each): exclusive scan of the chunk counts of
// Verlet-list members, list length and capacity check, barrier reset.  When
// `after_collision` is set it also closes the interval: collision-step
// counter, temperature of the collision, reaction bookkeeping.
__global__ __launch_bounds__(1024) void k_chunk_scan(Work w, int after_collision)
{
    const int rep = blockIdx.x;
    const RepDesc& D = w.desc[rep];
    if (!D.active) return;
    RepState* rs = D.rs;
    __shared__ uint32_t sbuf[16];
    __shared__ double dbuf[17 * 6];
    const int t = threadIdx.x;
    const int nch = D.n_chunks;
    const int per = (nch + 1023) / 1024;
    const gptr<const uint32_t> cnt = G(D.chunk_cnt);
    const gptr<uint32_t> off = G(D.chunk_off);
    // a single workgroup walks all chunks: latency, not bandwidth, bounds
    // this, so each thread's counts (up to CS_REG of them) are loaded at
    // once and kept for the second pass; more are read in batches, twice
    constexpr int CS_REG = 32, UB = 4;
    const int q0 = t * per;
    uint32_t c[CS_REG];
    uint32_t local = 0;
    if (per <= CS_REG) {
#pragma unroll
        for (int u = 0; u < CS_REG; ++u) c[u] = (u < per && q0 + u < nch) ? cnt[q0 + u] : 0u;
#pragma unroll
        for (int u = 0; u < CS_REG; ++u) local += c[u];
    } else {
        int kk = 0;
        for (; kk + UB <= per; kk += UB) {
            uint32_t b[UB];
#pragma unroll
            for (int u = 0; u < UB; ++u) b[u] = q0 + kk + u < nch ? cnt[q0 + kk + u] : 0u;
#pragma unroll
            for (int u = 0; u < UB; ++u) local += b[u];
        }
        for (; kk < per; ++kk)
            if (q0 + kk < nch) local += cnt[q0 + kk];
    }
    uint32_t total;
    uint32_t pre = block_exscan_u32<1024>(local, sbuf, &total);
    if (per <= CS_REG) {
#pragma unroll
        for (int u = 0; u < CS_REG; ++u) {
            if (u < per && q0 + u < nch) off[q0 + u] = pre;
            pre += c[u];
        }
    } else {
        int kk = 0;
        for (; kk + UB <= per; kk += UB) {
            uint32_t b[UB];
#pragma unroll
            for (int u = 0; u < UB; ++u) b[u] = q0 + kk + u < nch ? cnt[q0 + kk + u] : 0u;
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                if (q0 + kk + u < nch) off[q0 + kk + u] = pre;
                pre += b[u];
            }
        }
        for (; kk < per; ++kk) {
            const int q = q0 + kk;
            if (q < nch) {
                off[q] = pre;
                pre += cnt[q];
            }
        }
    }
    if (after_collision) {
        // tile partials (temperature sum and cells, reaction energy, bulk
        // flips): eight 32-byte loads in flight per round into two
        // accumulators; the order is fixed for a given tile count
        double a[2][4] = {};
        const gptr<const double> tp = G(D.tpart);
        constexpr int TL = 8;
        int k = t;
        for (; k + (TL - 1) * 1024 < D.n_tiles; k += TL * 1024) {
            double q[TL][4];
#pragma unroll
            for (int j = 0; j < TL; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) q[j][e] = tp[(int64_t)(k + j * 1024) * 4 + e];
#pragma unroll
            for (int j = 0; j < TL; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) a[j & 1][e] += q[j][e];
        }
        for (; k < D.n_tiles; k += 1024)
#pragma unroll
            for (int e = 0; e < 4; ++e) a[0][e] += tp[(int64_t)k * 4 + e];
        double v[6];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = a[0][j] + a[1][j];
        v[4] = 0.0;
        v[5] = 0.0;
        for (int g = t; g < D.G; g += 1024) {
            v[4] += D.epart[(int64_t)g * 2 + 0];
            v[5] += D.epart[(int64_t)g * 2 + 1];
            D.epart[(int64_t)g * 2 + 0] = 0.0;
            D.epart[(int64_t)g * 2 + 1] = 0.0;
        }
        block_sum_n<1024, 6>(v, dbuf);
        if (t == 0) {
            rs->T_sum = v[0];
            rs->T_cells = v[1];
            rs->e_rxn += v[2] + v[4];
            rs->n_bulk += (int64_t)v[3];
            rs->n_cat += (int64_t)v[5];
            rs->coll_step += 1;
        }
    }
    if (!after_collision) {
        // a stand-alone list build follows init or set_state, where the step
        // counters may have moved backwards: clear the exchange words so no
        // stale epoch can match
        uint64_t* part = reinterpret_cast<uint64_t*>(D.partials);
        for (int64_t k = t; k < 2 * ((int64_t)D.G * ROWW + BCW); k += 1024) part[k] = 0ull;
    }
    if (t == 0) {
        rs->n_cand = total;
        if ((int64_t)total > (int64_t)D.cand_cap) rs->flags |= RMP_FLAG_LIST_OVERFLOW;
        rs->bar = 0;
        rs->list_nmd = D.n_md;
    }
}

// Compacted Verlet list in array order.
__global__ __launch_bounds__(256) void k_cand_write(Work w)
{
    const int item = blockIdx.x;
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int chunk = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active) return;
    // most chunks hold no list member (the list gathers around the
    // colloids): their flags are not read at all, and their count is zero
    // already
    if (D.chunk_cnt[chunk] == 0u) return;
    __shared__ uint32_t sbuf[4];
    const int64_t n = D.n;
    const int64_t base = (int64_t)chunk * CHUNK;
    constexpr int PER = CHUNK / 256;
    const int t = threadIdx.x;
    uint32_t f[PER];
    uint32_t cnt = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        int64_t i = base + (int64_t)t * PER + k;
        f[k] = (i < n) ? (uint32_t)D.cflag[i] : 0u;
        cnt += f[k];
    }
    uint32_t total;
    uint32_t pre = block_exscan_u32<256>(cnt, sbuf, &total) + D.chunk_off[chunk];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (f[k]) {
            const int64_t i = base + (int64_t)t * PER + k;
            if ((int64_t)pre < (int64_t)D.cand_cap) {
                D.cand_idx[pre] = (uint32_t)i;
            } else {
                // beyond the list capacity (RMP_FLAG_LIST_OVERFLOW is set):
                // the particle is streamed freely so that every particle is
                // still binned exactly once
                D.cflag[i] = 0;
            }
            pre++;
        }
    }
    if (t == 0) D.chunk_cnt[chunk] = 0;
}

// ------------------------------------------------- free streaming + binning

// Rank of this lane's particle within its cell, with one atomic per run of
// equal keys in consecutive lanes (particles arrive sorted by the previous
// collision's cells, so runs are common).  All 64 lanes must call it.
struct RankIssue {
    uint32_t base;             // the run head's atomic result (head lanes only)
    int h;                     // lane of this lane's run head
};

__device__ __forceinline__ RankIssue wave_rank_issue(gptr<uint32_t> count, uint32_t key, bool valid)
{
    const int lane = threadIdx.x & 63;
    const uint32_t k = valid ? key : 0xffffffffu;
    const uint32_t prev = __shfl_up(k, 1, 64);
    const bool head = (lane == 0) || (k != prev);
    const uint64_t H = __ballot(head);
    const uint64_t upto = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
    const int h = 63 - __clzll(H & upto);
    const uint64_t above = (h == 63) ? 0ull : (H & (~0ull << (h + 1)));
    const int nexth = above ? (__ffsll((long long)above) - 1) : 64;
    RankIssue r;
    r.base = 0;
    r.h = h;
    if (head && valid)
        r.base = __hip_atomic_fetch_add(count + key, (uint32_t)(nexth - h), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return r;
}

__device__ __forceinline__ uint32_t wave_rank_finish(const RankIssue& r)
{
    const int lane = threadIdx.x & 63;
    return __shfl(r.base, r.h, 64) + (uint32_t)(lane - r.h);
}

__device__ __forceinline__ uint32_t wave_rank(gptr<uint32_t> count, uint32_t key, bool valid)
{
    return wave_rank_finish(wave_rank_issue(count, key, valid));
}

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

// Flows (constant acceleration, plates) stream every particle with flow_step
// and write back positions and velocities.  Otherwise:
// particles outside the Verlet list feel no force during the interval: n_md
// drifts x <- fma(dt, v, x) with a periodic wrap after each.  The drift of a
// coordinate is monotone, so if its final value is still inside the box no
// wrap occurred and the per-step wrap can be skipped; otherwise the drifts
// are replayed with the wrap.  Then the key of the shifted cell of the coming
// collision and a rank within the cell.  Workgroup `sub` of a chunk covers
// particles [sub*span, (sub+1)*span) of it, span = blockDim.x * PPT; thread t
// holds particles t, t + blockDim.x, ... of its span: every load is issued
// before the drifts, every rank atomic before the first of them is waited
// for.
template <class T, int PPT>
__global__ __launch_bounds__(256) void k_stream_bin(Work w, int wg_per_chunk)
{
    const int item = blockIdx.x / wg_per_chunk;
    const int sub = blockIdx.x - item * wg_per_chunk;
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int chunk = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active) return;
    RepState* rs = D.rs;
    __shared__ double sshift[3];
    const int64_t coll = rs->coll_step;
    if (threadIdx.x == 0) shift_of(D.seed, coll, sshift);
    __syncthreads();
    const double s[3] = {sshift[0], sshift[1], sshift[2]};
    const int cur = (int)(coll & 1);
    const int64_t n = D.n;
    const int nmd = D.n_md;
    const T dt = (T)D.dt;
    const T Lt[3] = {(T)D.Ld[0], (T)D.Ld[1], (T)D.Ld[2]};
    const gptr<T> xs[3] = {G(comp<T>(D.x[cur], n, 0)), G(comp<T>(D.x[cur], n, 1)), G(comp<T>(D.x[cur], n, 2))};
    const gptr<T> vs[3] = {G(comp<T>(D.v[cur], n, 0)), G(comp<T>(D.v[cur], n, 1)), G(comp<T>(D.v[cur], n, 2))};
    const gptr<const uint8_t> cflag = G(D.cflag);
    const gptr<uint64_t> keyrank = G(D.keyrank);
    const gptr<uint32_t> count = G(D.count);
    const int span = CHUNK / wg_per_chunk;
    const int64_t base = (int64_t)chunk * CHUNK + (int64_t)sub * span;
    if (D.flow) {
        const T g[3] = {(T)D.g[0], (T)D.g[1], (T)D.g[2]};
        const T hdt = (T)(0.5 * D.dt);
        for (int j0 = 0; j0 < span; j0 += blockDim.x) {
            const int64_t i = base + j0 + threadIdx.x;
            bool valid = (j0 + (int)threadIdx.x < span) && (i < n);
            if (valid) valid = cflag[i] == 0;
            uint32_t key = 0;
            if (valid) {
                T x[3], v[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) { x[d] = xs[d][i]; v[d] = vs[d][i]; }
                for (int k = 0; k < nmd; ++k) flow_step<T>(x, v, g, dt, hdt, Lt, D.walls != 0);
#pragma unroll
                for (int d = 0; d < 3; ++d) { xs[d][i] = x[d]; vs[d][i] = v[d]; }
                key = cell_key(D, (double)x[0], (double)x[1], (double)x[2], s);
            }
            const uint32_t rank = wave_rank(count, key, valid);
            if (valid) keyrank[i] = ((uint64_t)key << 32) | rank;
        }
        return;
    }
    bool valid[PPT];
    int64_t ii[PPT];
    T x[PPT][3], v[PPT][3];
    const int bs = (int)blockDim.x;
    // the flag and the state are loaded side by side, so one memory latency
    // precedes the drifts (a list entry's state, which the MD chain on the
    // side stream may be writing meanwhile, is loaded and never used)
    uint8_t fl[PPT];
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        ii[u] = base + u * bs + threadIdx.x;
        valid[u] = (u * bs + (int)threadIdx.x < span) && (ii[u] < n);
        fl[u] = valid[u] ? cflag[ii[u]] : (uint8_t)1;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            x[u][d] = valid[u] ? xs[d][ii[u]] : (T)0;
            v[u][d] = valid[u] ? vs[d][ii[u]] : (T)0;
        }
    }
#pragma unroll
    for (int u = 0; u < PPT; ++u) valid[u] = valid[u] && fl[u] == 0;
    uint32_t key[PPT];
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            T y = x[u][d];
            for (int k = 0; k < nmd; ++k) y = tfma(dt, v[u][d], y);
            const bool inside = (v[u][d] >= (T)0) ? (y < Lt[d]) : (y >= (T)0);
            if (!inside) {
                y = x[u][d];
                for (int k = 0; k < nmd; ++k) y = wrap_coord<T>(tfma(dt, v[u][d], y), Lt[d]);
            }
            x[u][d] = y;
        }
        key[u] = valid[u] ? cell_key(D, (double)x[u][0], (double)x[u][1], (double)x[u][2], s) : 0u;
    }
    RankIssue ri[PPT];
#pragma unroll
    for (int u = 0; u < PPT; ++u) ri[u] = wave_rank_issue(count, key[u], valid[u]);
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const uint32_t rank = wave_rank_finish(ri[u]);
        if (valid[u]) {
#pragma unroll
            for (int d = 0; d < 3; ++d) xs[d][ii[u]] = x[u][d];
            keyrank[ii[u]] = ((uint64_t)key[u] << 32) | rank;
        }
    }
}

// ------------------------------------------------------------- cell scan

__global__ __launch_bounds__(1024) void k_scan_blocks(Work w)
{
    const int item = blockIdx.x;
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int blk = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active) return;
    __shared__ uint32_t sbuf[16];
    const int64_t c0 = (int64_t)blk * SCAN_BLK;
    uint32_t s = 0;
    for (int k = 0; k < SCAN_BLK / 1024; ++k) {
        int64_t c = c0 + (int64_t)threadIdx.x * (SCAN_BLK / 1024) + k;
        if (c < D.ncell) s += D.count[c];
    }
    uint32_t tot = block_sum_u32<1024>(s, sbuf);
    if (threadIdx.x == 0) D.scanblk[blk] = tot;
}

// `direct`: the launch's grids are small (at most SCAN_DIRECT_BLOCKS blocks
// each), so a block sums the counts of the blocks before it itself and no
// k_scan_blocks pass is launched.
__global__ __launch_bounds__(1024) void k_scan_final(Work w, int direct)
{
    const int item = blockIdx.x;
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int blk = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active) return;
    __shared__ uint32_t sbuf[16];
    uint32_t pre = 0;
    if (direct) {
        // counts of cells [0, blk * SCAN_BLK): 4 loads in flight per thread
        const int64_t m = (int64_t)blk * SCAN_BLK;
        for (int64_t c = threadIdx.x; c < m; c += 4 * 1024) {
            uint32_t q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = c + u * 1024 < m ? D.count[c + u * 1024] : 0u;
            pre += (q[0] + q[1]) + (q[2] + q[3]);
        }
    } else {
        for (int k = threadIdx.x; k < blk; k += 1024) pre += D.scanblk[k];
    }
    pre = block_sum_u32<1024>(pre, sbuf);
    constexpr int PER = SCAN_BLK / 1024;
    const int64_t c0 = (int64_t)blk * SCAN_BLK + (int64_t)threadIdx.x * PER;
    uint32_t cnt[PER];
    uint32_t loc = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        int64_t c = c0 + k;
        cnt[k] = c < D.ncell ? D.count[c] : 0u;
        loc += cnt[k];
    }
    uint32_t total;
    uint32_t p = block_exscan_u32<1024>(loc, sbuf, &total) + pre;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        int64_t c = c0 + k;
        if (c < D.ncell) {
            D.start[c] = p;
            p += cnt[k];
        }
    }
    if (blk == D.n_scanblk - 1 && threadIdx.x == 0) D.start[D.ncell] = pre + total;
}

// Particle records of the staging array (Rec<T>): packed and unpacked with
// the state byte split into the spare top bits of id and index in FP32.
__device__ __forceinline__ void rec_put(Rec<double>* r, const double (&x)[3], const double (&v)[3],
                                        uint32_t id, uint32_t idx, uint8_t st)
{
    Rec<double> q;
    q.x[0] = x[0]; q.x[1] = x[1]; q.x[2] = x[2];
    q.v[0] = v[0]; q.v[1] = v[1]; q.v[2] = v[2];
    q.id = id; q.idx = idx; q.st = st; q.pad = 0u;
    *r = q;
}
__device__ __forceinline__ void rec_put(Rec<float>* r, const float (&x)[3], const float (&v)[3],
                                        uint32_t id, uint32_t idx, uint8_t st)
{
    Rec<float> q;
    q.x[0] = x[0]; q.x[1] = x[1]; q.x[2] = x[2];
    q.v[0] = v[0]; q.v[1] = v[1]; q.v[2] = v[2];
    q.id_f = id | ((uint32_t)((st >> 1) & 1u) << 31);
    q.idx_s = idx | ((uint32_t)(st & 1u) << 31);
    *r = q;
}
template <class RP>
__device__ __forceinline__ void rec_get(RP r, double (&x)[3], double (&v)[3], uint32_t& id, uint32_t& idx,
                                        uint8_t& st)
{
    x[0] = r->x[0]; x[1] = r->x[1]; x[2] = r->x[2];
    v[0] = r->v[0]; v[1] = r->v[1]; v[2] = r->v[2];
    id = r->id; idx = r->idx; st = (uint8_t)r->st;
}
template <class RP>
__device__ __forceinline__ void rec_get(RP r, float (&x)[3], float (&v)[3], uint32_t& id, uint32_t& idx,
                                        uint8_t& st)
{
    x[0] = r->x[0]; x[1] = r->x[1]; x[2] = r->x[2];
    v[0] = r->v[0]; v[1] = r->v[1]; v[2] = r->v[2];
    const uint32_t id_f = r->id_f, idx_s = r->idx_s;
    id = id_f & 0x7fffffffu;
    idx = idx_s & 0x7fffffffu;
    st = (uint8_t)(((idx_s >> 31) & 1u) | (((id_f >> 31) & 1u) << 1));
}

// single fields of a record (the oversized-cell path reads them one by one)
__device__ __forceinline__ uint32_t rec_idx(const Rec<double>* r) { return r->idx; }
__device__ __forceinline__ uint32_t rec_idx(const Rec<float>* r) { return r->idx_s & 0x7fffffffu; }
__device__ __forceinline__ uint8_t rec_st(const Rec<double>* r) { return (uint8_t)r->st; }
__device__ __forceinline__ uint8_t rec_st(const Rec<float>* r)
{
    return (uint8_t)(((r->idx_s >> 31) & 1u) | (((r->id_f >> 31) & 1u) << 1));
}
__device__ __forceinline__ uint32_t rec_id(const Rec<double>* r) { return r->id; }
__device__ __forceinline__ uint32_t rec_id(const Rec<float>* r) { return r->id_f & 0x7fffffffu; }
template <class T>
__device__ __forceinline__ double rec_v(const Rec<T>* r, int d) { return (double)r->v[d]; }

// Counting-sort scatter: particle i (read in array order, coalesced) goes to
// slot start[key] + rank of the staging array as one whole record, so the
// collision reads each tile of cells as one contiguous run.
template <class T>
__global__ __launch_bounds__(256) void k_scatter(Work w)
{
    const int item = blockIdx.x;
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int chunk = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active) return;
    const int64_t n = D.n;
    const int cur = (int)(D.rs->coll_step & 1);
    const gptr<const T> xs[3] = {G(comp<T>(D.x[cur], n, 0)), G(comp<T>(D.x[cur], n, 1)),
                                 G(comp<T>(D.x[cur], n, 2))};
    const gptr<const T> vs[3] = {G(comp<T>(D.v[cur], n, 0)), G(comp<T>(D.v[cur], n, 1)),
                                 G(comp<T>(D.v[cur], n, 2))};
    const gptr<const uint32_t> ids = G(D.id[cur]);
    const gptr<const uint8_t> sts = G(D.st[cur]);
    const gptr<const uint64_t> keyrank = G(D.keyrank);
    const gptr<const uint32_t> start = G(D.start);
    const int64_t base = (int64_t)chunk * CHUNK;
    // the chunk's four particles per thread: every load before the stores
    constexpr int P = CHUNK / 256;
    constexpr int RW = (int)(sizeof(Rec<T>) / 16);
    int64_t ii[P];
    uint32_t key[P], rank[P];
#pragma unroll
    for (int u = 0; u < P; ++u) {
        ii[u] = base + u * 256 + threadIdx.x;
        const uint64_t kr = ii[u] < n ? keyrank[ii[u]] : 0ull;
        key[u] = (uint32_t)(kr >> 32);
        rank[u] = (uint32_t)kr;
    }
    int64_t slot[P];
#pragma unroll
    for (int u = 0; u < P; ++u) slot[u] = ii[u] < n ? (int64_t)start[key[u]] + rank[u] : n;
    T x[P][3], v[P][3];
    uint32_t idv[P];
    uint8_t stv[P];
#pragma unroll
    for (int u = 0; u < P; ++u) {
        const int64_t i = ii[u] < n ? ii[u] : 0;
#pragma unroll
        for (int d = 0; d < 3; ++d) { x[u][d] = xs[d][i]; v[u][d] = vs[d][i]; }
        idv[u] = ids[i];
        stv[u] = sts[i];
    }
    // each record through LDS, then written by RW consecutive lanes (one
    // 16-byte word each), so a record leaves as one contiguous request
    __shared__ Rec<T> s_out[256];
    __shared__ int64_t s_slot[256];
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4* s_out4 = reinterpret_cast<const u32x4*>(s_out);
    const gptr<u32x4> stage4 = G(reinterpret_cast<u32x4*>(D.stage));
#pragma unroll
    for (int u = 0; u < P; ++u) {
        if (u) __syncthreads();
        rec_put(&s_out[threadIdx.x], x[u], v[u], idv[u], (uint32_t)ii[u], stv[u]);
        s_slot[threadIdx.x] = (ii[u] < n && slot[u] < n) ? slot[u] : -1;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < RW; ++q) {
            const int k4 = q * 256 + (int)threadIdx.x;
            const int r = k4 / RW, part = k4 - r * RW;
            const int64_t sl = s_slot[r];
            if (sl >= 0) stage4[sl * RW + part] = s_out4[k4];
        }
    }
}

// ------------------------------------------------------------- collision

// Add the Verlet-list flags of the wave's particles to their chunks' counts.
// The particles of one collision group occupy slots [q0, q0 + ns) with
// ns <= CHUNK, so they span the chunks c_lo = q0 / CHUNK and c_lo + 1 at
// most: one atomic per chunk and wave.  All 64 lanes must call it.
__device__ __forceinline__ void count_flag(gptr<uint32_t> chunk_cnt, int64_t o, bool f, int64_t c_lo)
{
    const int64_t ch = o / CHUNK;
    const uint32_t n_lo = (uint32_t)__popcll(__ballot(f && ch == c_lo));
    const uint32_t n_hi = (uint32_t)__popcll(__ballot(f && ch != c_lo));
    if ((threadIdx.x & 63) == 0) {
        if (n_lo) g_add(chunk_cnt + c_lo, n_lo);
        if (n_hi) g_add(chunk_cnt + c_lo + 1, n_hi);
    }
}

// Verlet-list membership (as is_candidate) tested only against the colloids
// of `mask`: the others were found out of reach of every particle of the
// tile, so they cannot change the outcome.
__device__ __forceinline__ bool is_candidate_masked(const RepDesc& D, const ColloidParams* cp, uint32_t mask,
                                                    const double (*Xw)[3], uint8_t st,
                                                    double x0, double x1, double x2,
                                                    double v0, double v1, double v2)
{
    if (D.flow) return false;
    if (st & 2) return true;
    if (mask == 0) return false;
    const double vv = dot3(v0, v1, v2, v0, v1, v2);
    const double reach = sqrt(vv) * D.tau;
    for (uint32_t m = mask; m; m &= m - 1) {
        const int c = __ffs(m) - 1;
        double dx = min_image(x0 - Xw[c][0], D.Ld[0], D.halfL[0]);
        double dy = min_image(x1 - Xw[c][1], D.Ld[1], D.halfL[1]);
        double dz = min_image(x2 - Xw[c][2], D.Ld[2], D.halfL[2]);
        double r2 = dot3(dx, dy, dz, dx, dy, dz);
        double tt = cp->reachR[c] + reach;
        if (r2 < tt * tt) return true;
    }
    return false;
}

constexpr int COLL_TCMAX = 64;       // cells per tile at most

// One cell of the tile holding more particles than a collision group (rare:
// hundreds of particles in one cell).  Its records are contiguous in the
// staging array; the stable order is found by counting ranks of the old
// indices into scratch (the key/rank array is dead after the scatter), then
// the per-cell quantities by one thread in that order, then every particle.
template <class T, int RULE, int NT>
__device__ void collide_big_cell(const RepDesc& D, const ColloidParams* cp, int nc, const double (*s_Xw)[3],
                                 int64_t coll, int64_t cell, uint32_t q0, int nn,
                                 double* s_u, double* s_n, int32_t* s_flip,
                                 double& t_sum, double& t_cells, double& du_sum, double& n_flip)
{
    RepState* rs = D.rs;
    const int t = threadIdx.x;
    const int64_t n = D.n;
    const int cur = (int)(coll & 1), nxt = cur ^ 1;
    T* xn[3] = {comp<T>(D.x[nxt], n, 0), comp<T>(D.x[nxt], n, 1), comp<T>(D.x[nxt], n, 2)};
    T* vn[3] = {comp<T>(D.v[nxt], n, 0), comp<T>(D.v[nxt], n, 1), comp<T>(D.v[nxt], n, 2)};
    uint32_t* idn = D.id[nxt];
    uint8_t* stn = D.st[nxt];
    const Rec<T>* rec = reinterpret_cast<const Rec<T>*>(D.stage) + q0;
    const double ca = D.ca, sa = D.sa, oma = 1.0 - D.ca;
    uint32_t* srt = reinterpret_cast<uint32_t*>(D.keyrank) + q0;   // stable rank -> record
    for (int j = t; j < nn; j += NT) {
        const uint32_t pj = rec_idx(&rec[j]);
        int r = 0;
        for (int q = 0; q < nn; ++q) r += rec_idx(&rec[q]) < pj ? 1 : 0;
        srt[r] = (uint32_t)j;
    }
    __syncthreads();
    if (t == 0) {
        double S0 = 0.0, S1 = 0.0, S2 = 0.0;
        for (int k = 0; k < nn; ++k) {
            const Rec<T>* q = &rec[srt[k] < (uint32_t)nn ? srt[k] : 0u];
            S0 = S0 + rec_v(q, 0);
            S1 = S1 + rec_v(q, 1);
            S2 = S2 + rec_v(q, 2);
        }
        const double u0 = S0 / (double)nn, u1 = S1 / (double)nn, u2 = S2 / (double)nn;
        double tsum = 0.0, G0 = 0.0, G1 = 0.0, G2 = 0.0;
        int nB = 0;
        for (int k = 0; k < nn; ++k) {
            const Rec<T>* q = &rec[srt[k] < (uint32_t)nn ? srt[k] : 0u];
            double w0 = rec_v(q, 0) - u0, w1 = rec_v(q, 1) - u1, w2 = rec_v(q, 2) - u2;
            tsum = tsum + dot3(w0, w1, w2, w0, w1, w2);
            nB += rec_st(q) & 1;
            if constexpr (RULE == 1) {
                uint64_t wv[4]; double z[3];
                philox<true>((uint64_t)coll, rec_id(q), 0, D.seed, TAG_THERMO, wv);
                normals3(wv, z);
                G0 = G0 + (D.vscale * z[0]);
                G1 = G1 + (D.vscale * z[1]);
                G2 = G2 + (D.vscale * z[2]);
            }
        }
        t_sum += (D.mass * tsum) / (double)(nn - 1);
        t_cells += 1.0;
        if (!(isfinite(u0) && isfinite(u1) && isfinite(u2))) atomicOr(&rs->flags, RMP_FLAG_NONFINITE);
        s_u[0] = u0; s_u[1] = u1; s_u[2] = u2;
        if constexpr (RULE == 1) {
            s_n[0] = G0 / (double)nn; s_n[1] = G1 / (double)nn; s_n[2] = G2 / (double)nn;
        }
        int flipk = -1;
        if (D.bulk_on && nB > 0) {
            uint64_t wv[4];
            philox<true>((uint64_t)coll, (uint64_t)cell, 0, D.seed, TAG_BULK, wv);
            double P = D.ptable[nB < RMP_PTABLE ? nB : RMP_PTABLE - 1];
            if (u01(wv[0]) < P) {
                int jb = (int)(u01(wv[1]) * (double)nB);
                if (jb >= nB) jb = nB - 1;
                for (int k = 0; k < nn; ++k)
                    if (rec_st(&rec[srt[k] < (uint32_t)nn ? srt[k] : 0u]) & 1) {
                        if (jb == 0) { flipk = k; break; }
                        jb--;
                    }
            }
        }
        *s_flip = flipk;
    }
    __syncthreads();
    const double u0 = s_u[0], u1 = s_u[1], u2 = s_u[2];
    const int flipk = *s_flip;
    for (int k0 = 0; k0 < nn; k0 += NT) {
        const int k = k0 + t;
        bool cnd = false;
        const int64_t o = (int64_t)q0 + k;
        if (k < nn) {
            T xt[3], vq[3]; uint32_t idq, pq; uint8_t s;
            rec_get(&rec[srt[k] < (uint32_t)nn ? srt[k] : 0u], xt, vq, idq, pq, s);
            const double vv0 = (double)vq[0], vv1 = (double)vq[1], vv2 = (double)vq[2];
            double v3[3];
            if constexpr (RULE == 0) {
                const double nax[3] = {s_n[0], s_n[1], s_n[2]};
                double rw[3];
                rotate(nax, ca, sa, oma, vv0 - u0, vv1 - u1, vv2 - u2, rw);
                v3[0] = u0 + rw[0]; v3[1] = u1 + rw[1]; v3[2] = u2 + rw[2];
            } else {
                uint64_t wv[4]; double z[3];
                philox<true>((uint64_t)coll, idq, 0, D.seed, TAG_THERMO, wv);
                normals3(wv, z);
                v3[0] = u0 + ((D.vscale * z[0]) - s_n[0]);
                v3[1] = u1 + ((D.vscale * z[1]) - s_n[1]);
                v3[2] = u2 + ((D.vscale * z[2]) - s_n[2]);
            }
            if (k == flipk) {
                du_sum += species_dU(D, cp, nc, s_Xw, (double)xt[0], (double)xt[1], (double)xt[2], 1, 0);
                n_flip += 1.0;
                s = 0;
            }
            const T vt[3] = {(T)v3[0], (T)v3[1], (T)v3[2]};
            for (int d = 0; d < 3; ++d) { xn[d][o] = xt[d]; vn[d][o] = vt[d]; }
            idn[o] = idq;
            stn[o] = s;
            cnd = is_candidate(D, cp, nc, s_Xw, s, (double)xt[0], (double)xt[1], (double)xt[2],
                               (double)vt[0], (double)vt[1], (double)vt[2]);
            D.cflag[o] = cnd ? 1 : 0;
        }
        // the wave's slots lie in [q0 + k0, q0 + k0 + NT): at most two chunks
        count_flag(G(D.chunk_cnt), o, cnd, ((int64_t)q0 + k0) / CHUNK);
    }
    __syncthreads();
}

// MPCD collision on one tile of cells of the shifted grid (sort ranks
// [c0, c0 + TC)).  The scatter has put the tile's particles in the
// contiguous slots [start[c0], start[c0 + TC)) of the staging array, cell
// by cell (in scatter order within a cell).  The tile's cells are taken in
// groups whose particles fit the workgroup (NT threads holding PPT particles
// each); usually the whole tile is one group.  Per group:
//   B  each thread reads whole records of the group's slots (coalesced) and
//      looks up each slot's cell (a slot-to-cell map of the tile built at
//      tile start; binary search over the cell starts past its end);
//   C  it ranks its particle by old index among its cell's records (the
//      stable order), writes position and id to the output slot of that
//      rank, velocity and species to LDS at that slot for the per-cell sums;
//   D  one thread per cell: sequential FP64 sums in the stable order,
//      centre-of-mass velocity, temperature term, bulk reaction decision;
//      one lane per colloid: is the colloid within reach of any particle of
//      the tile (the box of the tile's cells, the particles' largest speed)?
//   E  each thread rotates its particles about their cell's axis, applies
//      the reaction, and writes velocity, species and Verlet-list flag.
// The random axes and bulk-reaction uniforms of all cells of the tile, the
// slot-to-cell map and the tile's box are made at tile start (they depend on
// nothing loaded), next to the loads.
// The register file is held to 96 VGPRs (five waves per SIMD) with one
// particle per thread, or two in FP32, and to 128 (four waves) with two in
// FP64; a few bytes of values spill.
template <class T, int RULE, int NT, int PPT>
__global__ __launch_bounds__(NT, (PPT == 1 || sizeof(T) == 4) ? 5 : 4) void k_collide(Work w, int xcd_map)
{
    constexpr int CAP = NT * PPT;
    constexpr int FILLCAP = 2 * CAP;    // leading slots of the tile with their cell in s_cellof
    static_assert(CAP <= CHUNK, "a collision group spans at most two chunks");
    static_assert(NT >= 256, "the tile-start draws use the last two waves");
    int item = blockIdx.x;
    if (xcd_map && (gridDim.x & 7) == 0) {
        // workgroups are dealt to the eight XCDs in turn: give each XCD a
        // contiguous range of tiles so that neighbouring tiles, which gather
        // from the same source lines, share an L2
        const int per = (int)(gridDim.x >> 3);
        item = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    }
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int tile = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active || D.rule != RULE) return;
    RepState* rs = D.rs;
    const ColloidParams* cp = D.cp;
    const int nc = cp->nc;
    const int t = threadIdx.x;
    const int lane = t & 63;

    __shared__ uint32_t s_start[COLL_TCMAX + 1];
    __shared__ uint8_t s_cellof[FILLCAP];
    __shared__ uint32_t s_perm[CAP];
    __shared__ T s_v[3][CAP];
    __shared__ double s_g[3][RULE ? CAP : 1];
    __shared__ uint8_t s_st[CAP];
    __shared__ double s_u[COLL_TCMAX][3], s_n[COLL_TCMAX][3];
    __shared__ double s_b[COLL_TCMAX][2];       // bulk-reaction uniforms
    __shared__ double s_z[COLL_TCMAX][3];       // virtual-momentum normal of a plate-layer cell
    __shared__ int32_t s_flip[COLL_TCMAX];
    __shared__ uint8_t s_go[COLL_TCMAX];
    __shared__ double s_Xw[MAXC][3];
    __shared__ double s_box[6];        // the tile's box: lower, upper offsets from s_ref
    __shared__ double s_ref[3];        // lower corner of the tile's first cell (unshifted)
    __shared__ uint64_t s_vmax2;       // max |v|^2 (bit patterns order like the values)
    __shared__ uint32_t s_cmask;
    __shared__ double sred[(NT / 64 + 1) * 4];

    const int64_t coll = rs->coll_step;
    const int nxt = (int)(coll & 1) ^ 1;
    const int64_t n = D.n;
    const int TC = D.tile_cells;
    const int64_t c0 = (int64_t)tile * TC;
    const int64_t c1 = (c0 + TC < D.ncell) ? c0 + TC : D.ncell;
    const int ncl = (int)(c1 - c0);
    // the colloid cull needs a bound on the speed after the collision:
    // the rotation gives one (below), the thermostat's fresh draws do not
    const bool cull = RULE == 0 && nc > 0 && !D.flow;

    // ---- A: cell starts (and the counters zeroed for the next binning);
    //         per-cell random draws; colloid images
    for (int k = t; k <= ncl; k += NT) {
        s_start[k] = G(D.start)[c0 + k];
        if (k < ncl) G(D.count)[c0 + k] = 0;
    }
    if (t >= NT - 128 && t < NT - 64) {
        if constexpr (RULE == 0) {
            for (int lc = t - (NT - 128); lc < ncl; lc += 64) {
                const int64_t cell = D.hbits == KEY_ROW ? c0 + lc : G(D.cell_of)[c0 + lc];
                double nax[3];
                marsaglia_axis<true>(D.seed, (uint64_t)coll, (uint64_t)cell, nax);
                s_n[lc][0] = nax[0]; s_n[lc][1] = nax[1]; s_n[lc][2] = nax[2];
            }
        }
    } else if (t >= NT - 64) {
        if (D.bulk_on)
            for (int lc = t - (NT - 64); lc < ncl; lc += 64) {
                const int64_t cell = D.hbits == KEY_ROW ? c0 + lc : G(D.cell_of)[c0 + lc];
                uint64_t wv[4];
                philox<true>((uint64_t)coll, (uint64_t)cell, 0, D.seed, TAG_BULK, wv);
                s_b[lc][0] = u01(wv[0]);
                s_b[lc][1] = u01(wv[1]);
            }
    } else if (t >= 64 && t < 128) {
        if (D.walls) {
            // plates (flows have no colloids): the virtual-momentum normal of
            // every cell of the first and last layer, used if the cell turns
            // out to be cut and under-filled
            for (int lc = t - 64; lc < ncl; lc += 64) {
                const int64_t cell = D.hbits == KEY_ROW ? c0 + lc : G(D.cell_of)[c0 + lc];
                const int64_t cz = cell / ((int64_t)D.L[0] * D.L[1]);
                if (cz == 0 || cz == D.L[2] - 1) {
                    uint64_t wv[4]; double z[3];
                    philox<true>((uint64_t)coll, (uint64_t)cell, 0, D.seed, TAG_VIRT, wv);
                    normals3(wv, z);
                    s_z[lc][0] = z[0]; s_z[lc][1] = z[1]; s_z[lc][2] = z[2];
                }
            }
        } else if (t < 64 + nc) {
            for (int d = 0; d < 3; ++d) s_Xw[t - 64][d] = colloid_image(G(rs)->X[t - 64][d], D.Ld[d]);
        }
    }
    if (cull && t < 64) {
        // the tile's box for the colloid cull, from its cells: a cell
        // (c0, c1, c2) of the grid shifted by s in [0, 1)^3 holds the points
        // with c + s <= x < c + 1 + s, inside [c, c + 2) whatever the shift;
        // cell offsets from the first cell by minimum image, so a tile
        // across the periodic boundary stays compact
        const uint32_t L0 = (uint32_t)D.L[0], L1 = (uint32_t)D.L[1];
        int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
        int ref[3];
        {
            const uint32_t lin = (uint32_t)(D.hbits == KEY_ROW ? c0 : G(D.cell_of)[c0]);
            ref[0] = (int)(lin % L0);
            ref[1] = (int)((lin / L0) % L1);
            ref[2] = (int)(lin / (L0 * L1));
        }
        if (lane < ncl) {
            const uint32_t lin = (uint32_t)(D.hbits == KEY_ROW ? c0 + lane : G(D.cell_of)[c0 + lane]);
            const int cc[3] = {(int)(lin % L0), (int)((lin / L0) % L1), (int)(lin / (L0 * L1))};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                int o = cc[d] - ref[d];
                if (2 * o >= D.L[d]) o -= D.L[d];
                else if (2 * o < -D.L[d]) o += D.L[d];
                lo[d] = hi[d] = o;
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) wave_min_max_i(lo[d], hi[d]);
        if (lane == 0) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                s_ref[d] = (double)ref[d];
                s_box[d] = (double)lo[d];
                s_box[3 + d] = (double)hi[d] + 2.0;
            }
        }
    }
    if (t < 64 && lane < ncl) {
        // tile-local cell of each of the tile's first FILLCAP slots (the
        // cells' slot ranges are contiguous and in order)
        const uint32_t base = G(D.start)[c0], a = G(D.start)[c0 + lane], b = G(D.start)[c0 + lane + 1];
        const uint32_t e = b - base < (uint32_t)FILLCAP ? b - base : (uint32_t)FILLCAP;
        for (uint32_t r = a - base; r < e; ++r) s_cellof[r] = (uint8_t)lane;
    }
    if (t == 64) { s_vmax2 = 0ull; s_cmask = 0u; }
    __syncthreads();

    const gptr<const Rec<T>> stage = G(reinterpret_cast<const Rec<T>*>(D.stage));
    const gptr<T> xn[3] = {G(comp<T>(D.x[nxt], n, 0)), G(comp<T>(D.x[nxt], n, 1)), G(comp<T>(D.x[nxt], n, 2))};
    const gptr<T> vn[3] = {G(comp<T>(D.v[nxt], n, 0)), G(comp<T>(D.v[nxt], n, 1)), G(comp<T>(D.v[nxt], n, 2))};
    const gptr<uint32_t> idn = G(D.id[nxt]);
    const gptr<uint8_t> stn = G(D.st[nxt]);
    const gptr<uint8_t> cflag = G(D.cflag);
    const double ca = D.ca, sa = D.sa, oma = 1.0 - D.ca;

    double t_sum = 0.0, t_cells = 0.0, du_sum = 0.0, n_flip = 0.0;
    uint64_t big = 0;          // tile-local cells left to k_collide_big (uniform)
    int ga = 0;
    while (ga < ncl) {
        int gb;
        if (s_start[ncl] - s_start[ga] <= (uint32_t)CAP) {
            gb = ncl;
        } else {
            // the longest run of cells from ga whose particles fit (at least one cell)
            const int k = ga + 1 + t;
            const bool ok = k <= ncl && s_start[k] - s_start[ga] <= (uint32_t)CAP;
            const int cnt = __syncthreads_count(ok);
            gb = ga + (cnt > 0 ? cnt : 1);
        }
        const uint32_t q0 = s_start[ga], q1 = s_start[gb];
        const int ns = (int)(q1 - q0);
        if (ns > CAP) {
            // one cell beyond a group's capacity: left to k_collide_big
            big |= 1ull << ga;
            ga = gb;
            continue;
        }
        // ---- B: records of the group's slots, cell of each slot
        T xr[PPT][3], vq[PPT][3];
        uint32_t idq[PPT], pj[PPT];
        uint8_t sr[PPT];
        int lcj[PPT];
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int j = t + u * NT;
            lcj[u] = ga;
            pj[u] = 0u;
            sr[u] = 0;
            if (j < ns) {
                rec_get(&stage[q0 + j], xr[u], vq[u], idq[u], pj[u], sr[u]);
                s_perm[j] = pj[u];
                const uint32_t q = q0 + (uint32_t)j;
                if (q - s_start[0] < (uint32_t)FILLCAP) {
                    lcj[u] = s_cellof[q - s_start[0]];
                } else {
                    int lo = ga, hi = gb - 1;
                    while (lo < hi) {
                        const int mid = (lo + hi + 1) >> 1;
                        if (s_start[mid] <= q) lo = mid; else hi = mid - 1;
                    }
                    lcj[u] = lo;
                }
            }
        }
        __syncthreads();
        // ---- C: stable rank; position and id written at the rank's slot
        int slot[PPT];
        double gv2 = 0.0;
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int j = t + u * NT;
            slot[u] = -1;
            if (j < ns) {
                const int cb = (int)(s_start[lcj[u]] - q0), ce = (int)(s_start[lcj[u] + 1] - q0);
                const uint32_t p = pj[u];
                int r = 0, q = cb;
                for (; q + 4 <= ce; q += 4)
                    r += (s_perm[q] < p ? 1 : 0) + (s_perm[q + 1] < p ? 1 : 0) + (s_perm[q + 2] < p ? 1 : 0) +
                         (s_perm[q + 3] < p ? 1 : 0);
                for (; q < ce; ++q) r += s_perm[q] < p ? 1 : 0;
                const int sl = cb + r;
                slot[u] = sl;
                const int64_t o = (int64_t)q0 + sl;
                const T (&xr_)[3] = xr[u];
                const T (&vq_)[3] = vq[u];
#pragma unroll
                for (int d = 0; d < 3; ++d) { xn[d][o] = xr_[d]; s_v[d][sl] = vq_[d]; }
                idn[o] = idq[u];
                s_st[sl] = sr[u];
                if constexpr (RULE == 1) {
                    uint64_t wv[4]; double z[3];
                    philox<true>((uint64_t)coll, idq[u], 0, D.seed, TAG_THERMO, wv);
                    normals3(wv, z);
                    s_g[0][sl] = D.vscale * z[0];
                    s_g[1][sl] = D.vscale * z[1];
                    s_g[2][sl] = D.vscale * z[2];
                }
                if (cull) {
                    // the largest speed vmax of the tile's particles, for the
                    // colloid cull: after the rotation a speed is at most
                    // |u| + |v - u| <= 3 vmax
                    const double vv = dot3((double)vq_[0], (double)vq_[1], (double)vq_[2],
                                           (double)vq_[0], (double)vq_[1], (double)vq_[2]);
                    gv2 = vv > gv2 ? vv : gv2;
                    if (!(vv <= 1e300)) gv2 = 1e300;          // inf or NaN: no cull
                }
            }
        }
        if (cull) {
            // wave maximum by DPP (exact), then one LDS atomic per wave
            // (non-negative doubles order like their bit patterns)
            gv2 = wave_max_d(gv2);
            if (lane == 0) atomicMax((unsigned long long*)&s_vmax2, (unsigned long long)__double_as_longlong(gv2));
        }
        __syncthreads();
        // ---- D: per cell (one thread each); colloid cull (second wave)
        for (int cl = ga + t; cl < gb; cl += NT) {
            const int cb = (int)(s_start[cl] - q0), ce = (int)(s_start[cl + 1] - q0);
            const int nn = ce - cb;
            s_flip[cl] = -1;
            // Lamura et al. (2001): a cell of the first or last layer (cut by
            // a plate) with fewer than n0 particles holds n0 - n virtual ones
            // at rest on average; only their summed momentum enters, a normal
            // vector of variance (n0 - n) kT / m per component
            bool virt = false;
            if (D.walls && nn >= 1 && nn < D.wall_n0) {
                const int64_t cell = D.hbits == KEY_ROW ? c0 + cl : G(D.cell_of)[c0 + cl];
                const int64_t cz = cell / ((int64_t)D.L[0] * D.L[1]);
                virt = cz == 0 || cz == D.L[2] - 1;
            }
            const bool go = nn >= 2 || virt;
            s_go[cl] = go ? 1 : 0;
            int nB = 0;
            if (go) {
                double S0 = 0.0, S1 = 0.0, S2 = 0.0;
                for (int q = cb; q < ce; ++q) {
                    S0 = S0 + (double)s_v[0][q];
                    S1 = S1 + (double)s_v[1][q];
                    S2 = S2 + (double)s_v[2][q];
                    nB += s_st[q] & 1;
                }
                double u0, u1, u2;
                if (virt) {
                    const double sd = sqrt((double)(D.wall_n0 - nn)) * D.vscale;
                    const double n0 = (double)D.wall_n0;
                    u0 = (S0 + (sd * s_z[cl][0])) / n0;
                    u1 = (S1 + (sd * s_z[cl][1])) / n0;
                    u2 = (S2 + (sd * s_z[cl][2])) / n0;
                } else {
                    u0 = S0 / (double)nn; u1 = S1 / (double)nn; u2 = S2 / (double)nn;
                    double tsum = 0.0;
                    for (int q = cb; q < ce; ++q) {
                        const double w0 = (double)s_v[0][q] - u0, w1 = (double)s_v[1][q] - u1,
                                     w2 = (double)s_v[2][q] - u2;
                        tsum = tsum + dot3(w0, w1, w2, w0, w1, w2);
                    }
                    t_sum += (D.mass * tsum) / (double)(nn - 1);
                    t_cells += 1.0;
                }
                // a non-finite centre-of-mass velocity would spread through
                // its cell: latched for the caller
                if (!(isfinite(u0) && isfinite(u1) && isfinite(u2))) atomicOr(&rs->flags, RMP_FLAG_NONFINITE);
                s_u[cl][0] = u0; s_u[cl][1] = u1; s_u[cl][2] = u2;
                if constexpr (RULE == 1) {
                    double G0 = 0.0, G1 = 0.0, G2 = 0.0;
                    for (int q = cb; q < ce; ++q) {
                        G0 = G0 + s_g[0][q];
                        G1 = G1 + s_g[1][q];
                        G2 = G2 + s_g[2][q];
                    }
                    s_n[cl][0] = G0 / (double)nn; s_n[cl][1] = G1 / (double)nn; s_n[cl][2] = G2 / (double)nn;
                }
            } else if (nn == 1) {
                nB = s_st[cb] & 1;
            }
            if (D.bulk_on && nB > 0) {
                const double P = G(D.ptable)[nB < RMP_PTABLE ? nB : RMP_PTABLE - 1];
                if (s_b[cl][0] < P) {
                    int jb = (int)(s_b[cl][1] * (double)nB);
                    if (jb >= nB) jb = nB - 1;
                    for (int q = cb; q < ce; ++q)
                        if (s_st[q] & 1) {
                            if (jb == 0) { s_flip[cl] = q; break; }
                            jb--;
                        }
                }
            }
        }
        if (cull && t >= 64 && t < 128) {
            // colloid c can reach a particle of the tile only if its reach
            // sphere, widened by the largest speed times tau, meets the
            // tile's box (minimum image per axis, margin far above rounding)
            bool near = false;
            // c is made opaque here so that the per-thread addresses below
            // are formed inside the group loop: hoisted out of it, they were
            // held across the whole tile and spilled to scratch (FP32 form)
            int c = t - 64;
            asm volatile("" : "+v"(c));
            if (c < nc) {
                const double vmax2 = __longlong_as_double((long long)s_vmax2);
                const double reach = ((3.0 * sqrt(vmax2)) * D.tau + cp->reachR[c]) * (1.0 + 1e-6) + 1e-6;
                double r2 = 0.0;
                bool wide = !(reach < 1e200);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    // box [lo, hi] of offsets from s_ref; the colloid's offset
                    // and its periodic images: the nearest one counts
                    const double lo = s_box[d], hi = s_box[3 + d];
                    if (!(hi - lo < 0.5 * D.Ld[d])) { wide = true; continue; }
                    const double oc = min_image(s_Xw[c][d] - s_ref[d], D.Ld[d], D.halfL[d]);
                    double dd = 1e300;
#pragma unroll
                    for (int img = -1; img <= 1; ++img) {
                        const double ci = oc + (double)img * D.Ld[d];
                        double e = lo - ci > ci - hi ? lo - ci : ci - hi;
                        e = e > 0.0 ? e : 0.0;
                        dd = e < dd ? e : dd;
                    }
                    r2 += dd * dd;
                }
                near = wide || r2 < reach * reach;
            }
            const uint64_t m = __ballot(near);
            if (lane == 0) s_cmask = (uint32_t)m;
        }
        __syncthreads();
        // ---- E: rotate (or thermostat), react, write, Verlet-list flag
        // without the cull every colloid is tested
        const uint32_t cmask = cull ? s_cmask : (nc >= 32 ? 0xffffffffu : ((1u << nc) - 1u));
        const int64_t c_lo = (int64_t)q0 / CHUNK;
        bool fl[PPT];
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            bool cnd = false;
            fl[u] = false;
            int64_t o = (int64_t)q0;
            if (slot[u] >= 0) {
                const int cl = lcj[u];
                double v3[3] = {(double)s_v[0][slot[u]], (double)s_v[1][slot[u]], (double)s_v[2][slot[u]]};
                if (s_go[cl]) {
                    const double u0 = s_u[cl][0], u1 = s_u[cl][1], u2 = s_u[cl][2];
                    if constexpr (RULE == 0) {
                        const double nax[3] = {s_n[cl][0], s_n[cl][1], s_n[cl][2]};
                        double rw[3];
                        rotate(nax, ca, sa, oma, v3[0] - u0, v3[1] - u1, v3[2] - u2, rw);
                        v3[0] = u0 + rw[0]; v3[1] = u1 + rw[1]; v3[2] = u2 + rw[2];
                    } else {
                        v3[0] = u0 + (s_g[0][slot[u]] - s_n[cl][0]);
                        v3[1] = u1 + (s_g[1][slot[u]] - s_n[cl][1]);
                        v3[2] = u2 + (s_g[2][slot[u]] - s_n[cl][2]);
                    }
                }
                uint8_t s = sr[u];
                o = (int64_t)q0 + slot[u];
                const bool flip = s_flip[cl] == slot[u];
                // the position (written to the output slot in C by this
                // thread) is read back only for a colloid within reach of
                // the tile
                T xo3[3] = {(T)0, (T)0, (T)0};
                if (cmask != 0u)
#pragma unroll
                    for (int d = 0; d < 3; ++d) xo3[d] = xn[d][o];
                if (flip) {
                    fl[u] = true;
                    n_flip += 1.0;
                    s = 0;
                }
                const T vt[3] = {(T)v3[0], (T)v3[1], (T)v3[2]};
#pragma unroll
                for (int d = 0; d < 3; ++d) vn[d][o] = vt[d];
                stn[o] = s;
                cnd = is_candidate_masked(D, cp, cmask, s_Xw, s, (double)xo3[0], (double)xo3[1],
                                          (double)xo3[2], (double)vt[0], (double)vt[1], (double)vt[2]);
                cflag[o] = cnd ? 1 : 0;
            }
            count_flag(G(D.chunk_cnt), o, cnd, c_lo);
        }
        // the potential change of a flipped particle, in the same order per
        // thread, after the writes: inside their loop its colloid loop
        // raised the register peak beyond the budget (spills to scratch)
#pragma unroll
        for (int u = 0; u < PPT; ++u)
            if (fl[u]) {
                const int64_t o = (int64_t)q0 + slot[u];
                du_sum += species_dU(D, cp, nc, s_Xw, (double)xn[0][o], (double)xn[1][o], (double)xn[2][o], 1, 0);
            }
        ga = gb;
        if (ga < ncl) __syncthreads();   // the next group reuses the LDS
    }
    // the tile's sums: the wave trees, then the waves in order (as
    // block_sum_n).  The temperature terms live in wave 0 alone (one thread
    // per cell, at most 64 cells) and the reaction terms only where a flip
    // happened; a wave holding only +0.0 has the tree +0.0, which is not
    // formed (no sum here is ever -0.0)
    {
        constexpr int NW = NT / 64;
        const int wave = t >> 6;
        double red[4] = {0.0, 0.0, 0.0, 0.0};
        if (wave == 0) {
            red[0] = wave_tree_sum(t_sum);
            red[1] = wave_tree_sum(t_cells);
        }
        if (__ballot(n_flip != 0.0) != 0) {
            red[2] = wave_tree_sum(du_sum);
            red[3] = wave_tree_sum(n_flip);
        }
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < 4; ++q) sred[wave * 4 + q] = red[q];
        __syncthreads();
        if (t < 4) {
            double a = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) a = a + sred[w * 4 + t];
            G(D.tpart)[(int64_t)tile * 4 + t] = a;
        }
        if (t == 0) G(D.bigmask)[tile] = big;
    }
}

// The cells that k_collide found beyond a group's capacity (a bit per
// tile-local cell in bigmask[tile]).  Workgroup w looks at tiles
// [64 w, 64 w + 64) of the launch and collides each such cell with all its
// threads (collide_big_cell); the cell's temperature, reaction energy and
// flips are added to its tile's partials after those of the tile's other
// cells, cell by cell, so the sums stay deterministic.
template <class T, int RULE>
__global__ __launch_bounds__(256) void k_collide_big(Work w, int n_items)
{
    constexpr int NT = 256;
    const int t = threadIdx.x;
    __shared__ uint64_t s_mask[64];
    __shared__ double s_u[3], s_n[3];
    __shared__ int32_t s_flip;
    __shared__ double s_Xw[MAXC][3];
    __shared__ double sred[(NT / 64 + 1) * 4];
    const int item0 = blockIdx.x * 64;
    bool any = false;
    if (t < 64) {
        const int item = item0 + t;
        uint64_t m = 0;
        if (item < n_items) {
            const int rep = find_rep(w.prefix, w.nrep, item);
            const RepDesc& D = w.desc[rep];
            if (D.active && D.rule == RULE) m = D.bigmask[item - w.prefix[rep]];
        }
        s_mask[t] = m;
        any = m != 0;
    }
    if (__syncthreads_or(any) == 0) return;
    for (int q = 0; q < 64; ++q) {
        const uint64_t mask = s_mask[q];
        if (mask == 0) continue;
        const int item = item0 + q;
        const int rep = find_rep(w.prefix, w.nrep, item);
        const int tile = item - w.prefix[rep];
        const RepDesc& D = w.desc[rep];
        RepState* rs = D.rs;
        const ColloidParams* cp = D.cp;
        const int nc = cp->nc;
        const int64_t coll = rs->coll_step;
        if (t < nc)
            for (int d = 0; d < 3; ++d) s_Xw[t][d] = colloid_image(rs->X[t][d], D.Ld[d]);
        const int64_t c0 = (int64_t)tile * D.tile_cells;
        double t_sum = 0.0, t_cells = 0.0, du_sum = 0.0, n_flip = 0.0;
        for (uint64_t m = mask; m; m &= m - 1) {
            const int ga = __ffsll((long long)m) - 1;
            const int64_t cell = D.hbits == KEY_ROW ? c0 + ga : D.cell_of[c0 + ga];
            const uint32_t q0 = D.start[c0 + ga];
            const int nn = (int)(D.start[c0 + ga + 1] - q0);
            if (RULE == 0 && t == 0) marsaglia_axis<true>(D.seed, (uint64_t)coll, (uint64_t)cell, s_n);
            __syncthreads();
            collide_big_cell<T, RULE, NT>(D, cp, nc, s_Xw, coll, cell, q0, nn, s_u, s_n, &s_flip,
                                          t_sum, t_cells, du_sum, n_flip);
        }
        double red[4] = {t_sum, t_cells, du_sum, n_flip};
        block_sum_n<NT, 4>(red, sred);
        if (t == 0)
            for (int j = 0; j < 4; ++j) D.tpart[(int64_t)tile * 4 + j] = D.tpart[(int64_t)tile * 4 + j] + red[j];
        __syncthreads();
    }
}

// ---------------------------------------------------------- observables

// part: where the per-chunk partials go (nullptr: the replica's own
// workspace region)
template <class T>
__global__ __launch_bounds__(256) void k_observe(Work w, double* part)
{
    const int item = blockIdx.x;
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int chunk = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active) return;
    __shared__ double sred[8];
    const int cur = (int)(D.rs->coll_step & 1);
    const int64_t n = D.n;
    const int64_t base = (int64_t)chunk * CHUNK;
    double P0 = 0.0, P1 = 0.0, P2 = 0.0, ke = 0.0, nb = 0.0;
    for (int j = threadIdx.x; j < CHUNK; j += 256) {
        int64_t i = base + j;
        if (i >= n) break;
        double v0 = comp<T>(D.v[cur], n, 0)[i], v1 = comp<T>(D.v[cur], n, 1)[i],
               v2 = comp<T>(D.v[cur], n, 2)[i];
        P0 += v0; P1 += v1; P2 += v2;
        ke += dot3(v0, v1, v2, v0, v1, v2);
        nb += (double)(D.st[cur][i] & 1);
    }
    double r[5] = {P0, P1, P2, ke, nb};
    double* out = part ? part : D.obs_part;
    for (int k = 0; k < 5; ++k) {
        double s = block_sum<256>(r[k], sred);
        if (threadIdx.x == 0) out[(int64_t)chunk * 8 + k] = s;
    }
}

// Totals of the k_observe partials: lane k (< 5) adds quantity k over the
// chunks in chunk order, the order of the host-side sum, so both give the
// same totals bit for bit.
__global__ __launch_bounds__(64) void k_observe_total(const double* part, int cnt, double* tot)
{
    const int k = threadIdx.x;
    if (k >= 5) return;
    double s = 0.0;
    for (int c = 0; c < cnt; ++c) s += part[(int64_t)c * 8 + k];
    tot[k] = s;
}

// ------------------------------------------------------------ dimer analysis
// Quantities of the paper's dimer analysis programs ("Applications of
// RMPCDMD"), sampled on the device after a collision: the dimer record
// (centre of mass, its velocity, unit axis from bond_a to bond_b, directed
// velocity) and integer counts of A and B in cylindrical shells around the
// dimer's axis.  The same operations in the same order as the definitions
// (no contraction), so records and counts are exact, independent of launch
// shape.
__device__ __forceinline__ void dimer_record(const ColloidParams* cp, const RepState* rs, int k,
                                             double rec[RMP_SERIES_FIELDS])
{
    const int a = cp->bond_a[k], b = cp->bond_b[k];
    const double ma = cp->mass[a], mb = cp->mass[b];
    double dX[3];
    for (int d = 0; d < 3; ++d) {
        rec[d] = (ma * rs->X[a][d] + mb * rs->X[b][d]) / (ma + mb);
        rec[3 + d] = (ma * rs->V[a][d] + mb * rs->V[b][d]) / (ma + mb);
        dX[d] = rs->X[b][d] - rs->X[a][d];
    }
    const double len = sqrt(dot3(dX[0], dX[1], dX[2], dX[0], dX[1], dX[2]));
    for (int d = 0; d < 3; ++d) rec[6 + d] = dX[d] / len;
    rec[9] = dot3(rec[3], rec[4], rec[5], rec[6], rec[7], rec[8]);
}

// One workgroup per particle chunk (after the collision): chunk 0 also
// stores the series record.  After a collision the arrays are in cell order,
// so a chunk occupies a small region: its bounding box culls, for the whole
// workgroup, every dimer whose cylinder cannot reach it (the cylinder lies
// within a sphere of radius sqrt(zmax^2 + rmax^2) about the centre of mass;
// the bound carries a relative margin far above the rounding of z and rho,
// so no counted particle is ever culled).  Hits are sparse, so they go
// straight to 64-bit device atomics.
template <class T>
__global__ __launch_bounds__(256) void k_analysis(Work w)
{
    constexpr int PPT = CHUNK / 256;
    const int item = blockIdx.x;
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int chunk = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active || D.an == nullptr) return;
    Analysis* A = D.an;
    const RepState* rs = D.rs;
    if (rs->coll_step % A->every != 0) return;
    __shared__ double sR[MAXC][3], sU[MAXC][3];
    __shared__ double sBox[4][6];
    __shared__ int sLive[MAXC];
    const int nb = A->nb;
    const int t = threadIdx.x;
    const int cur = (int)(rs->coll_step & 1);
    const int64_t n = D.n;
    const int64_t base = (int64_t)chunk * CHUNK;
    // every load of the chunk first
    double px[PPT][3];
    int psp[PPT];
    bool pv[PPT];
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const int64_t i = base + t + 256 * q;
        pv[q] = i < n;
        const int64_t ic = pv[q] ? i : base;
        px[q][0] = (double)comp<T>(D.x[cur], n, 0)[ic];
        px[q][1] = (double)comp<T>(D.x[cur], n, 1)[ic];
        px[q][2] = (double)comp<T>(D.x[cur], n, 2)[ic];
        psp[q] = D.st[cur][ic] & 1;
    }
    if (t < nb) {
        double rec[RMP_SERIES_FIELDS];
        dimer_record(D.cp, rs, t, rec);
        for (int d = 0; d < 3; ++d) {
            sR[t][d] = colloid_image(rec[d], D.Ld[d]);
            sU[t][d] = rec[6 + d];
        }
        if (chunk == 0) {
            const int64_t k = A->n_samples;
            if (k < A->cap) {
                double* dst = A->series + (k * nb + t) * RMP_SERIES_FIELDS;
                for (int f = 0; f < RMP_SERIES_FIELDS; ++f) dst[f] = rec[f];
                if (t == 0) A->series_t[k] = rs->md_step;
            }
        }
    }
    // bounding box of the chunk's positions
    double bx[6];
    for (int d = 0; d < 3; ++d) {
        bx[d] = INFINITY;
        bx[3 + d] = -INFINITY;
    }
#pragma unroll
    for (int q = 0; q < PPT; ++q)
        if (pv[q])
            for (int d = 0; d < 3; ++d) {
                bx[d] = fmin(bx[d], px[q][d]);
                bx[3 + d] = fmax(bx[3 + d], px[q][d]);
            }
    for (int m = 1; m < 64; m <<= 1)
        for (int d = 0; d < 3; ++d) {
            bx[d] = fmin(bx[d], __shfl_xor(bx[d], m, 64));
            bx[3 + d] = fmax(bx[3 + d], __shfl_xor(bx[3 + d], m, 64));
        }
    if ((t & 63) == 0)
        for (int k = 0; k < 6; ++k) sBox[t >> 6][k] = bx[k];
    __syncthreads();
    if (chunk == 0 && t == 0) {
        if (A->n_samples < A->cap) A->n_samples += 1;
        else A->n_dropped += 1;
    }
    if (t < nb) {
        bool live = true;
        for (int d = 0; d < 3; ++d) {
            const double lo = fmin(fmin(sBox[0][d], sBox[1][d]), fmin(sBox[2][d], sBox[3][d]));
            const double hi = fmax(fmax(sBox[0][3 + d], sBox[1][3 + d]), fmax(sBox[2][3 + d], sBox[3][3 + d]));
            // periodic distance from the centre's images to [lo, hi]
            double dist = INFINITY;
            for (int k = -1; k <= 1; ++k) {
                const double c = sR[t][d] + (double)k * D.Ld[d];
                dist = fmin(dist, c < lo ? lo - c : (c > hi ? c - hi : 0.0));
            }
            if (dist >= A->cull_r) live = false;
        }
        sLive[t] = live ? 1 : 0;
    }
    __syncthreads();
    const int nz = A->nz, nr = A->nr;
    const double zmax = A->zmax, inv_dz = A->inv_dz, inv_dr = A->inv_dr, skip_r2 = A->skip_r2;
    const double fnz = (double)nz, fnr = (double)nr;
    uint64_t* hist = A->hist;
    for (int b = 0; b < nb; ++b) {
        if (!sLive[b]) continue;
        const double c0 = sR[b][0], c1 = sR[b][1], c2 = sR[b][2];
        const double u0 = sU[b][0], u1 = sU[b][1], u2 = sU[b][2];
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            if (!pv[q]) continue;
            const double r0 = min_image(px[q][0] - c0, D.Ld[0], D.halfL[0]);
            const double r1 = min_image(px[q][1] - c1, D.Ld[1], D.halfL[1]);
            const double r2 = min_image(px[q][2] - c2, D.Ld[2], D.halfL[2]);
            const double z = dot3(r0, r1, r2, u0, u1, u2);
            const double zs = (z + zmax) * inv_dz;
            if (!(zs >= 0.0 && zs < fnz)) continue;
            const double p0 = r0 - z * u0, p1 = r1 - z * u1, p2 = r2 - z * u2;
            const double pp = dot3(p0, p1, p2, p0, p1, p2);
            if (!(pp < skip_r2)) continue;
            const double rsc = sqrt(pp) * inv_dr;
            if (!(rsc < fnr)) continue;
            const int iz = (int)zs, ir = (int)rsc;
            atomicAdd((unsigned long long*)&hist[(((int64_t)b * 2 + psp[q]) * nz + iz) * nr + ir], 1ull);
        }
    }
}

// Mean-squared displacement of each dimer's centre of mass over the stored
// series: one thread per (dimer, lag), origins summed in order.
__global__ __launch_bounds__(256) void k_msd(Analysis* A, int32_t max_lag)
{
    const int nb = A->nb;
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= (int64_t)nb * (max_lag + 1)) return;
    const int b = (int)(g / (max_lag + 1));
    const int lag = (int)(g % (max_lag + 1));
    const int64_t T = A->n_samples;
    double out = 0.0;
    if (lag < T) {
        double acc = 0.0;
        for (int64_t t0 = 0; t0 + lag < T; ++t0) {
            const double* p = A->series + ((t0 + lag) * nb + b) * RMP_SERIES_FIELDS;
            const double* q = A->series + (t0 * nb + b) * RMP_SERIES_FIELDS;
            const double d0 = p[0] - q[0], d1 = p[1] - q[1], d2 = p[2] - q[2];
            acc += dot3(d0, d1, d2, d0, d1, d2);
        }
        out = acc / (double)(T - lag);
    }
    A->msd[(int64_t)b * A->cap + lag] = out;
}

// ----------------------------------------------------- explicit instances

#define RMP_INST(T)                                                              \
    template __global__ void k_init<T>(const RepDesc*);                          \
    template __global__ void k_init_sub<T>(const RepDesc*, const double*);       \
    template __global__ void k_list<T>(Work);                                    \
    template __global__ void k_stream_bin<T, 1>(Work, int);                      \
    template __global__ void k_stream_bin<T, 2>(Work, int);                      \
    template __global__ void k_stream_bin<T, 4>(Work, int);                      \
    template __global__ void k_scatter<T>(Work);                                 \
    template __global__ void k_collide_big<T, 0>(Work, int);                     \
    template __global__ void k_collide_big<T, 1>(Work, int);                     \
    template __global__ void k_collide<T, 0, 256, 2>(Work, int);                 \
    template __global__ void k_collide<T, 1, 256, 2>(Work, int);                 \
    template __global__ void k_collide<T, 0, 512, 2>(Work, int);                 \
    template __global__ void k_collide<T, 1, 512, 2>(Work, int);                 \
    template __global__ void k_collide<T, 0, 256, 1>(Work, int);                 \
    template __global__ void k_collide<T, 1, 256, 1>(Work, int);                 \
    template __global__ void k_collide<T, 0, 512, 1>(Work, int);                 \
    template __global__ void k_collide<T, 1, 512, 1>(Work, int);                 \
    template __global__ void k_observe<T>(Work, double*);                     \
    template __global__ void k_analysis<T>(Work);

RMP_INST(double)
RMP_INST(float)

}  // namespace rmp
