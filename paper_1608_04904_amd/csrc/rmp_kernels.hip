// gfx950 kernels of the MPCD+MD solvent path.
//
// One interval (paper, "Algorithms"): n_md velocity-Verlet steps with WCA
// colloid-solvent forces over a Verlet list built from the cell sort, exact
// RATTLE for dimers and catalytic conversion, then one MPCD collision on a
// randomly shifted grid with the RMPCD bulk reaction.  Kernels of one
// interval, in stream order:
//
//   k_stream       particles outside the Verlet list: n_md drifts held in
//                  registers, the cell of the coming collision and an atomic
//                  rank in it; the collision's random numbers per cell
//   k_chain        Verlet-list particles and colloids: n_md MD steps in
//                  persistent workgroups; colloid forces reduced with a fixed
//                  binary tree over list positions; inter-workgroup exchange
//                  per step when the list spans several workgroups; then the
//                  list particles' cells and ranks
//   k_scan_*       exclusive scan of the cell counts -> cell_start
//   k_cells        sparse boxes: the random numbers per cell
//   k_perm         array position of each particle to slot
//                  cell_start[key] + rank of the sort permutation
//   k_collide      per tile of cells: gather the records through the
//                  permutation, restore the stable (old-index) order inside
//                  each cell, FP64 centre-of-mass sums, rotation about a random
//                  axis (or Anderson thermostat), bulk B->A reaction,
//                  Verlet-list flags for the next interval, contiguous write
//                  of the cell-ordered records
//   k_close        compacted Verlet list, per-interval bookkeeping
//
// Data layout in HBM: one record per particle (position, velocity, id, state
// bits; 64 bytes in FP64, 32 in FP32), double-buffered across collisions, so
// that the sort moves only a 4-byte permutation and the collision gathers
// each particle with whole sectors.
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
        Rec<T> q{};
        for (int d = 0; d < 3; ++d) {
            T xv = (T)xi[d];
            if (xv >= (T)D.Ld[d]) xv = (T)0;    // FP32 rounding up to L
            q.x[d] = xv;
            q.v[d] = (T)(D.vscale * z[d]);
            sum[d] += (double)q.v[d];
        }
        q.id = (uint32_t)i;
        recs<T>(D, 0)[i] = q;
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
        T* v = recs<T>(D, 0)[i].v;
        for (int d = 0; d < 3; ++d) v[d] = (T)((double)v[d] - mean[d]);
    }
}

// ------------------------------------------------------- Verlet list build

// Stand-alone list flags (first interval, a new state, or a change of n_md);
// replicas whose list is valid for their n_md are left alone.
__device__ __forceinline__ bool list_is_valid(const RepDesc& D, const RepState* rs)
{
    return rs->list_nmd == (int64_t)D.n_md;
}

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
    if (list_is_valid(D, rs)) return;
    __shared__ double sXw[MAXC][3];
    __shared__ uint32_t sred[4];
    const int nc = cp->nc;
    const int t = threadIdx.x;
    if (t < nc)
        for (int d = 0; d < 3; ++d) sXw[t][d] = colloid_image(rs->X[t][d], D.Ld[d]);
    __syncthreads();
    const Rec<T>* rec = recs<T>(D, (int)(rs->coll_step & 1));
    uint64_t* lbits = list_bits(D, rs->coll_step);
    const int64_t n = D.n;
    const int64_t base = (int64_t)chunk * CHUNK;
    uint32_t cnt = 0;
    for (int j = t; j < CHUNK; j += 256) {
        const int64_t i = base + j;
        bool c = false;
        if (i < n) {
            const Rec<T>* r = rec + i;
            c = is_candidate(D, cp, nc, sXw, (uint8_t)r->st, r->x[0], r->x[1], r->x[2], r->v[0], r->v[1], r->v[2]);
        }
        const uint64_t m = __ballot(c);
        if ((t & 63) == 0) lbits[i >> 6] = m;
        cnt += c ? 1u : 0u;
    }
    uint32_t tot = block_sum_u32<256>(cnt, sred);
    if (t == 0) D.chunk_cnt[(int64_t)((rs->coll_step + 1) & 1) * D.n_chunks + chunk] = tot;
}

// Closes an interval (after_collision), or a stand-alone list build: the
// compacted Verlet list in array order, and per replica the list length and
// capacity check and, after a collision, the collision-step counter, the
// temperature, the reaction bookkeeping and the next grid shift.  One
// workgroup takes CLOSE_CH chunks, a wave each, and sums the counts of the
// chunks before them itself (where there are many chunks, only if its own have
// members: few do, the list gathers around the colloids), so no scan goes
// before.  Latency bounds it: what does not depend on the counts is loaded at
// the start.  With up to CLOSE_DIRECT workgroups the first one does the
// bookkeeping; with more, each sums its share of the tiles' partials and the
// last to arrive combines the shares in order; what it and the others exchange
// goes through atomics at device scope.  The counts are double-buffered by
// collision, since workgroups read each other's, and the list bits, since the
// streaming reads them after this launch: it clears the ones the next collision
// adds to.  (A scan by one workgroup and a launch that
// wrote the list after it: 60 + 9 us at 128^3, 10 + 6 at 32^3; now 40 and 12.)
constexpr int CLOSE_CH = CHUNK / 64;         // chunks per workgroup
constexpr int CLOSE_DIRECT = 64;             // (its chunks: one per thread of a workgroup)

template <class T>
__global__ __launch_bounds__(1024) void k_close(Work w, int after_collision)
{
    static_assert(CLOSE_CH == 16 && CHUNK == 1024, "a wave per chunk, 16 particles per lane");
    const int rep = find_rep(w.prefix, w.nrep, blockIdx.x);
    const int b = (int)blockIdx.x - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active) return;
    RepState* rs = D.rs;
    if (!after_collision && list_is_valid(D, rs)) return;
    __shared__ uint32_t sbuf[16], s_sum[16][2], s_cnt[16];
    __shared__ double dbuf[17 * 6];
    __shared__ int s_last;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int nch = D.n_chunks;
    const int nb = w.prefix[rep + 1] - w.prefix[rep];
    const bool counted = !after_collision || nb > CLOSE_DIRECT;
    // (coll_closing: the first workgroup may advance coll_step meanwhile)
    const int64_t coll = after_collision ? rs->coll_closing + 1 : rs->coll_step;
    const gptr<uint32_t> cnt = G(D.chunk_cnt) + (int64_t)((coll + 1) & 1) * nch;   // (the finished collision's parity)
    const gptr<uint32_t> nxt = G(D.chunk_cnt) + (int64_t)(coll & 1) * nch;
    const int c0 = b * CLOSE_CH;
    const int chunk = c0 + wave;
    const gptr<uint64_t> bits = G(list_bits(D, coll)) + (int64_t)chunk * (CHUNK / 64);
    const gptr<uint64_t> spent = G(list_bits(D, coll + 1)) + (int64_t)chunk * (CHUNK / 64);
    const uint64_t word = chunk < nch ? bits[lane >> 2] : 0ull;
    const uint32_t mine = chunk < nch ? cnt[chunk] : 0u;
    uint32_t pre = 0, total = 0;
    if (!counted) {
        total = t < nch ? cnt[t] : 0u;
        pre = t < c0 ? total : 0u;
    }
    // the tiles' partials: all of them, or this workgroup's share
    double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int64_t o_bulk = 0, o_cat = 0;
    double o_rxn = 0.0;
    if (after_collision && (counted || b == 0)) {
        const gptr<const double> tp = G((const double*)D.tpart);
        const int t0 = counted ? (int)((int64_t)D.n_tiles * b / nb) : 0;
        const int t1 = counted ? (int)((int64_t)D.n_tiles * (b + 1) / nb) : D.n_tiles;
        for (int k = t0 + t; k < t1; k += 1024)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += tp[(int64_t)k * 4 + e];
        for (int g = t; g < D.G; g += 1024) {
            v[4] += D.epart[(int64_t)g * 2 + 0];
            v[5] += D.epart[(int64_t)g * 2 + 1];
        }
        o_rxn = rs->e_rxn;
        o_bulk = rs->n_bulk;
        o_cat = rs->n_cat;
    }
    double shift[3];
    if (t == 1023 && (counted || b == 0)) shift_of(D.seed, coll, shift);
    if (lane == 0) {
        s_cnt[wave] = mine;
        if (chunk < nch) nxt[chunk] = 0u;
    }
    if (chunk < nch && lane < CHUNK / 64) spent[lane] = 0ull;
    if (__syncthreads_or(mine != 0u || !counted)) {
        if (counted) {
            for (int k = t; k < c0; k += 4 * 1024) {
                uint32_t q[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) q[u] = k + u * 1024 < c0 ? cnt[k + u * 1024] : 0u;
                pre += (q[0] + q[1]) + (q[2] + q[3]);
            }
            pre = block_sum_u32<1024>(pre, sbuf);
        } else {
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                pre += __shfl_xor(pre, m, 64);
                total += __shfl_xor(total, m, 64);
            }
            if (lane == 0) {
                s_sum[wave][0] = pre;
                s_sum[wave][1] = total;
            }
            __syncthreads();
            pre = total = 0;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                pre += s_sum[k][0];
                total += s_sum[k][1];
            }
        }
        for (int k = 0; k < wave; ++k) pre += s_cnt[k];
        if (mine != 0u) {
            // lane l: particles [16 l, 16 l + 16) of the chunk
            const int64_t i0 = (int64_t)chunk * CHUNK + lane * 16;
            const uint32_t all = (uint32_t)(word >> ((lane & 3) * 16)) & 0xffffu;
            uint32_t f = all;
            uint32_t x = (uint32_t)__popc(f);
            const uint32_t own = x;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t y = __shfl_up(x, d, 64);
                x += lane >= d ? y : 0u;
            }
            pre += x - own;
            for (; f; f &= f - 1u) {
                // beyond the list capacity (RMP_FLAG_LIST_OVERFLOW is set) the
                // particles are streamed freely so that every particle is still
                // binned exactly once
                if ((int64_t)pre >= (int64_t)D.cand_cap) {
                    typedef uint16_t __attribute__((may_alias)) bits16;
                    ((gptr<bits16>)bits)[lane] = (uint16_t)(all & ~f);
                    break;
                }
                D.cand_idx[pre] = (uint32_t)(i0 + __ffs(f) - 1);
                pre++;
            }
        }
    }
    if (counted && after_collision) {
        const double e4 = v[4], e5 = v[5];          // (whole in every workgroup)
        block_sum_n<1024, 6>(v, dbuf);
        // the share to the exchange array; the returned old values are waited
        // for, so that it is there before this workgroup is counted
        if (t == 0) {
            unsigned long long z = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                z |= __hip_atomic_exchange((unsigned long long*)D.gpart + (int64_t)b * 4 + e,
                                           (unsigned long long)__double_as_longlong(v[e]), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
            __asm__ __volatile__("" ::"v"((uint32_t)z), "v"((uint32_t)(z >> 32)) : "memory");
        }
        v[4] = e4;
        v[5] = e5;
    }
    if (counted) {
        if (t == 0) {
            // counted in two levels: many arrivals at one address are serial
            const int grp = b >> 6, ng = (nb + 63) >> 6;
            const uint32_t members = (uint32_t)(nb - (grp << 6) < 64 ? nb - (grp << 6) : 64);
            uint32_t* const done = D.done;
            bool l = __hip_atomic_fetch_add(done + 32 * (1 + grp), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                     members - 1u;
            if (l) {
                __hip_atomic_store(done + 32 * (1 + grp), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                l = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)ng - 1u;
                if (l) __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            s_last = l ? 1 : 0;
        }
        __syncthreads();
        if (s_last == 0) return;
        for (int k = t; k < nch; k += 4 * 1024) {
            uint32_t q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = k + u * 1024 < nch ? cnt[k + u * 1024] : 0u;
            total += (q[0] + q[1]) + (q[2] + q[3]);
        }
        total = block_sum_u32<1024>(total, sbuf);
    } else if (b != 0) {
        return;
    }
    if (after_collision) {
        if (counted) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = 0.0;
            for (int k = t; k < nb; k += 1024)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[e] += __longlong_as_double((long long)__hip_atomic_load(
                        (unsigned long long*)D.gpart + (int64_t)k * 4 + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        }
        for (int g = t; g < D.G; g += 1024) {
            D.epart[(int64_t)g * 2 + 0] = 0.0;
            D.epart[(int64_t)g * 2 + 1] = 0.0;
        }
        __syncthreads();
        block_sum_n<1024, 6>(v, dbuf);
        if (t == 0) {
            rs->T_sum = v[0];
            rs->T_cells = v[1];
            rs->e_rxn = o_rxn + (v[2] + v[4]);
            rs->n_bulk = o_bulk + (int64_t)v[3];
            rs->n_cat = o_cat + (int64_t)v[5];
        }
    } else {
        // a stand-alone list build follows init or set_state, where the step
        // counters may have moved backwards: clear the exchange words so no
        // stale epoch can match
        uint64_t* part = reinterpret_cast<uint64_t*>(D.partials);
        for (int64_t k = t; k < 2 * ((int64_t)D.G * ROWW + BCW); k += 1024) part[k] = 0ull;
    }
    if (t == 1023)
        for (int d = 0; d < 3; ++d) rs->shift[d] = shift[d];
    if (t == 0) {
        rs->coll_step = coll;
        rs->n_cand = total;
        if ((int64_t)total > (int64_t)D.cand_cap) rs->flags |= RMP_FLAG_LIST_OVERFLOW;
        rs->list_nmd = D.n_md;
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
    const gptr<const uint32_t> count = G((const uint32_t*)D.count);
    const int64_t c0 = (int64_t)blk * SCAN_BLK;
    uint32_t s = 0;
    for (int k = 0; k < SCAN_BLK / 1024; ++k) {
        int64_t c = c0 + (int64_t)threadIdx.x * (SCAN_BLK / 1024) + k;
        if (c < D.ncell) s += count[c];
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
    const gptr<const uint32_t> count = G((const uint32_t*)D.count);
    uint32_t pre = 0;
    if (direct) {
        // counts of cells [0, blk * SCAN_BLK): 4 loads in flight per thread
        const int64_t m = (int64_t)blk * SCAN_BLK;
        for (int64_t c = threadIdx.x; c < m; c += 4 * 1024) {
            uint32_t q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = c + u * 1024 < m ? count[c + u * 1024] : 0u;
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
        cnt[k] = c < D.ncell ? count[c] : 0u;
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

// The colloids whose list reach can meet a tile after the coming collision,
// for the tiles [tlo, thi): one wave, one colloid per lane.
__device__ __forceinline__ void tile_masks(const RepDesc& D, int64_t tlo, int64_t thi)
{
    const int lane = threadIdx.x & 63;
    const RepState* rs = D.rs;
    const ColloidParams* cp = D.cp;
    const int nc = cp->nc;
    if (nc == 0 || D.flow) return;
    const uint32_t L0 = (uint32_t)D.L[0], L1 = (uint32_t)D.L[1];
    for (int64_t tile = tlo; tile < thi; ++tile) {
        // the tile's box from its cells: a cell c of the grid shifted by
        // s in [0, 1)^3 holds the points with c + s <= x < c + 1 + s,
        // inside [c, c + 2) whatever the shift; cell offsets from the
        // first cell by minimum image, so a tile across the periodic
        // boundary stays compact
        const int64_t r0 = tile * D.tile_cells;
        const int64_t r1 = r0 + D.tile_cells < D.ncell ? r0 + D.tile_cells : D.ncell;
        const int ncl = (int)(r1 - r0);
        int ref[3], lo3[3] = {0, 0, 0}, hi3[3] = {0, 0, 0};
        const uint32_t first = (uint32_t)(D.hbits == KEY_ROW ? r0 : G(D.cell_of)[r0]);
        ref[0] = (int)(first % L0);
        ref[1] = (int)((first / L0) % L1);
        ref[2] = (int)(first / (L0 * L1));
        if (lane < ncl) {
            const uint32_t lin = (uint32_t)(D.hbits == KEY_ROW ? r0 + lane : G(D.cell_of)[r0 + lane]);
            const int cc[3] = {(int)(lin % L0), (int)((lin / L0) % L1), (int)(lin / (L0 * L1))};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                int o = cc[d] - ref[d];
                if (2 * o >= D.L[d]) o -= D.L[d];
                else if (2 * o < -D.L[d]) o += D.L[d];
                lo3[d] = hi3[d] = o;
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) wave_min_max_i(lo3[d], hi3[d]);
        bool near = false;
        if (lane < nc) {
            // colloid c can reach a particle of the tile only if its
            // reach sphere, widened by the largest speed after the
            // collision (|u| + |v - u| <= 3 vcap) times tau, meets the box
            // (minimum image per axis, margin far above rounding)
            const double reach = ((3.0 * D.vcap) * D.tau + cp->reachR[lane]) * (1.0 + 1e-6) + 1e-6;
            double r2 = 0.0;
            bool wide = !(reach < 1e200);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double blo = (double)lo3[d], bhi = (double)hi3[d] + 2.0;
                if (!(bhi - blo < 0.5 * D.Ld[d])) { wide = true; continue; }
                const double oc = min_image(colloid_image(rs->X[lane][d], D.Ld[d]) - (double)ref[d], D.Ld[d],
                                            D.halfL[d]);
                double dd = 1e300;
#pragma unroll
                for (int img = -1; img <= 1; ++img) {
                    const double ci = oc + (double)img * D.Ld[d];
                    double e = blo - ci > ci - bhi ? blo - ci : ci - bhi;
                    e = e > 0.0 ? e : 0.0;
                    dd = e < dd ? e : dd;
                }
                r2 += dd * dd;
            }
            near = wide || r2 < reach * reach;
        }
        const uint64_t m = __ballot(near);
        if (lane == 0) D.tilemask[tile] = (uint32_t)m;
    }
}

// (the workgroup size is a parameter of the instance: LDS for 256 threads left a
// compute unit five workgroups of 64, 128^3 with 8 dimers 2504 us an interval,
// now 1836)
template <class T, int PPT, bool FLOW, int NT>
__global__ __launch_bounds__(NT) void k_stream(Work w, int wg_per_chunk)
{
    stream_body<T, PPT, FLOW, NT>(w.desc, w.prefix, w.nrep, xcd_range(blockIdx.x, gridDim.x), wg_per_chunk);
}

// Sparse boxes: the coming collision's draws, a block of DRAW_CELLS cells per
// workgroup, and its tile masks, shared out over the replica's waves.
__global__ __launch_bounds__(256) void k_cells(Work w)
{
    const int rep = find_rep(w.prefix, w.nrep, blockIdx.x);
    const int blk = (int)blockIdx.x - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active) return;
    collision_draws(D, (int64_t)blk * DRAW_CELLS);
    const Share sh{(int64_t)blk * 4 + (threadIdx.x >> 6), (int64_t)(w.prefix[rep + 1] - w.prefix[rep]) * 4};
    tile_masks(D, sh.lo(D.n_tiles), sh.hi(D.n_tiles));
}

// Sort permutation of the coming collision: particle i goes to slot
// start[key] + rank.  Thread t of a workgroup holds particles t, t +
// blockDim.x, ... of its span (PPT of them).  The replica's workgroups share
// its tiles (colloid masks).
// `scan` (every grid of the launch has at most SCAN_BLK cells): no scan went
// before, and each workgroup sums the counts itself into LDS; the replica's
// first writes the cell starts for the collision.  A launch takes 4.4 us even
// when it does nothing (10^3 cells: scan and permutation 4.7 + 5.0, now 5.5).
template <int PPT, bool SCAN>
__global__ __launch_bounds__(256) void k_perm(Work w, int wg_per_chunk)
{
    const int b = xcd_range(blockIdx.x, gridDim.x);
    const int item = b / wg_per_chunk;
    const int sub = b - item * wg_per_chunk;
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int chunk = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active) return;
    const int64_t n = D.n;
    const gptr<const uint64_t> keyrank = G((const uint64_t*)D.keyrank);
    const gptr<const uint32_t> start = G((const uint32_t*)D.start);
    const gptr<uint32_t> perm = G(D.perm);
    const int span = CHUNK / wg_per_chunk;
    const int64_t base = (int64_t)chunk * CHUNK + (int64_t)sub * span;
    uint64_t kr[PPT];
    int64_t slot[PPT];
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const int64_t i = base + u * (int)blockDim.x + threadIdx.x;
        kr[u] = i < n ? keyrank[i] : 0ull;
    }
    if constexpr (SCAN) {
        __shared__ uint32_t s_start[SCAN_BLK];
        __shared__ uint32_t sbuf[4];
        const gptr<const uint32_t> count = G((const uint32_t*)D.count);
        constexpr int PER = SCAN_BLK / 256;
        const int nc = (int)D.ncell;
        const int per = (nc + 255) / 256;                 // cells per thread
        const int q0 = (int)threadIdx.x * per;
        uint32_t c[PER], loc = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) c[k] = k < per && q0 + k < nc ? count[q0 + k] : 0u;
#pragma unroll
        for (int k = 0; k < PER; ++k) loc += c[k];
        uint32_t total;
        uint32_t p = block_exscan_u32<256>(loc, sbuf, &total);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (k < per && q0 + k < nc) {
                s_start[q0 + k] = p;
                if (chunk == 0 && sub == 0) D.start[q0 + k] = p;
            }
            p += c[k];
        }
        if (chunk == 0 && sub == 0 && threadIdx.x == 0) D.start[nc] = total;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PPT; ++u) slot[u] = (int64_t)s_start[kr[u] >> 32] + (uint32_t)kr[u];
    } else {
#pragma unroll
        for (int u = 0; u < PPT; ++u) slot[u] = (int64_t)start[kr[u] >> 32] + (uint32_t)kr[u];
    }
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const int64_t i = base + u * (int)blockDim.x + threadIdx.x;
        if (i < n && slot[u] < n) perm[slot[u]] = (uint32_t)i;
    }
    const Share sh{(int64_t)chunk * wg_per_chunk + sub, (int64_t)D.n_chunks * wg_per_chunk};
    if (threadIdx.x < 64 && !D.sparse) tile_masks(D, sh.lo(D.n_tiles), sh.hi(D.n_tiles));
    if (sh.me == 0 && threadIdx.x == 0) D.rs->coll_closing = D.rs->coll_step;
    if (sh.me == 0 && (int)threadIdx.x < D.nc) {
        RepState* rs = D.rs;
        for (int d = 0; d < 3; ++d) rs->Xw[threadIdx.x][d] = colloid_image(rs->X[threadIdx.x][d], D.Ld[d]);
    }
}

// ------------------------------------------------------------- collision

// Verlet-list membership of the wave's slots: lane l holds slot o0 + l (o0
// uniform).  The bits go to their words (the wave's slots touch two at most)
// and their number to their chunks' counts, one atomic each, only where some
// slot is a member.  All 64 lanes must call it.
__device__ __forceinline__ void list_flags(const RepDesc& D, int64_t coll, int64_t o0, bool f)
{
    const uint64_t m = __ballot(f);
    if (m == 0ull) return;
    const int sh = (int)(o0 & 63);
    const uint64_t lo = m << sh, hi = sh ? m >> (64 - sh) : 0ull;
    if ((threadIdx.x & 63) == 0) {
        const int64_t w0 = o0 >> 6;
        const gptr<uint64_t> bits = G(list_bits(D, coll + 1));
        const gptr<uint32_t> cnt = G(D.chunk_cnt) + (int64_t)(coll & 1) * D.n_chunks;
        if (lo) {
            (void)__hip_atomic_fetch_or(bits + w0, lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            g_add(cnt + w0 / (CHUNK / 64), (uint32_t)__popcll(lo));
        }
        if (hi) {
            (void)__hip_atomic_fetch_or(bits + w0 + 1, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            g_add(cnt + (w0 + 1) / (CHUNK / 64), (uint32_t)__popcll(hi));
        }
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

// Sums over k = 0 .. nn - 1, one term after the other, of the M values that
// fill(k, o) gives: the workgroup puts the terms of `cap` k at a time into buf
// (M cap doubles of LDS), thread d < M adds those of value d and returns the sum.
template <int NT, int M, class F>
__device__ __forceinline__ double ordered_sums(double* buf, int cap, int nn, F fill)
{
    const int t = threadIdx.x;
    double sum = 0.0;
    for (int k0 = 0; k0 < nn; k0 += cap) {
        const int n = nn - k0 < cap ? nn - k0 : cap;
        __syncthreads();                             // (buf is free)
        for (int k = t; k < n; k += NT) {
            double o[M];
            fill(k0 + k, o);
#pragma unroll
            for (int d = 0; d < M; ++d) buf[d * cap + k] = o[d];
        }
        __syncthreads();
        if (t < M) {
            const double* p = buf + t * cap;
#pragma unroll 8
            for (int k = 0; k < n; ++k) sum = sum + p[k];
        }
    }
    return sum;
}

// One cell of the tile holding more particles than a collision group (beyond a
// wave's 128, in the workgroup form 512).  Its particles go to their output
// slots in the stable order, found by counting ranks of the old indices; then
// the sequential sums over them in that order, their terms staged in LDS; then
// every particle in place.  buf: LDS of 3 cap doubles, cap a multiple of 4; s_n
// holds the axis, s_u between plates the virtual momentum's normals (big_draws).
// Bound by the comparisons of the ranks and the chains of additions.  (One
// thread reading the records for the sums, the indices read from memory: 512
// cells of 200 in 32^3 cells, 711 us an interval, under the thermostat 5920; now
// 163 and 208.)
template <int RULE, bool FLOW>
__device__ __forceinline__ void big_draws(const RepDesc& D, int64_t coll, int64_t cell, double* s_u, double* s_n)
{
    if (threadIdx.x != 0) return;
    if (RULE == 0) marsaglia_axis<true>(D.seed, (uint64_t)coll, (uint64_t)cell, s_n);
    if (FLOW && D.walls) {
        uint64_t wv[4];
        philox<true>((uint64_t)coll, (uint64_t)cell, 0, D.seed, TAG_VIRT, wv);
        double z[3];
        normals3(wv, z);
        for (int d = 0; d < 3; ++d) s_u[d] = z[d];
    }
}

template <class T, int RULE, int NT, bool FLOW>
__device__ void collide_big_cell(const RepDesc& D, const ColloidParams* cp, int nc, const double (*s_Xw)[3],
                                 int64_t coll, int64_t cell, uint32_t q0, int nn, double* buf, int cap,
                                 double* s_u, double* s_n, int32_t* s_flip,
                                 double& t_sum, double& t_cells, double& du_sum, double& n_flip)
{
    RepState* rs = D.rs;
    const int t = threadIdx.x;
    const int cur = (int)(coll & 1), nxt = cur ^ 1;
    const double ca = D.ca, sa = D.sa, oma = 1.0 - D.ca;
    // the particles into the output slots, in stable order
    // (the collision then changes them in place)
    const Rec<T>* src = recs<T>(D, cur);
    Rec<T>* rec = recs<T>(D, nxt) + q0;
    const uint32_t* perm = D.perm + q0;
    constexpr int JP = 2;                            // particles a thread ranks at a time
    uint32_t* ix = reinterpret_cast<uint32_t*>(buf);
    for (int j0 = 0; j0 < nn; j0 += JP * NT) {
        uint32_t pj[JP];
        int r[JP];
#pragma unroll
        for (int u = 0; u < JP; ++u) {
            const int j = j0 + u * NT + t;
            pj[u] = j < nn ? perm[j] : 0u;
            r[u] = 0;
        }
        for (int k0 = 0; k0 < nn; k0 += 6 * cap) {
            const int n = nn - k0 < 6 * cap ? nn - k0 : 6 * cap;
            __syncthreads();                         // (buf is free)
            for (int k = t; k < ((n + 3) & ~3); k += NT) ix[k] = k < n ? perm[k0 + k] : 0xffffffffu;
            __syncthreads();
            for (int k = 0; k < n; k += 4) {
                const u32x4 q = *reinterpret_cast<const u32x4*>(ix + k);
#pragma unroll
                for (int u = 0; u < JP; ++u)
                    r[u] += (q.x < pj[u] ? 1 : 0) + (q.y < pj[u] ? 1 : 0) + (q.z < pj[u] ? 1 : 0) +
                            (q.w < pj[u] ? 1 : 0);
            }
        }
#pragma unroll
        for (int u = 0; u < JP; ++u)
            if (j0 + u * NT + t < nn) {
                rec[r[u]] = src[pj[u]];
            }
    }
    // a cell cut by a plate and under-filled has virtual particles, as in
    // k_collide, and no temperature
    bool virt = false;
    if (FLOW && D.walls && nn < D.wall_n0) {
        const int64_t cz = cell / ((int64_t)D.L[0] * D.L[1]);
        virt = cz == 0 || cz == D.L[2] - 1;
    }
    const double S = ordered_sums<NT, 3>(buf, cap, nn, [&](int k, double (&o)[3]) {
#pragma unroll
        for (int d = 0; d < 3; ++d) o[d] = (double)rec[k].v[d];
    });
    if (t < 3) {
        double um = S / (double)nn;
        if (FLOW && virt) {
            const double sd = sqrt((double)(D.wall_n0 - nn)) * D.vscale;
            um = (S + (sd * s_u[t])) / (double)D.wall_n0;
        }
        if (!isfinite(um)) atomicOr(&rs->flags, RMP_FLAG_NONFINITE);
        s_u[t] = um;
    }
    __syncthreads();
    if (!virt) {
        const double tsum = ordered_sums<NT, 1>(buf, cap, nn, [&](int k, double (&o)[1]) {
            const double w0 = (double)rec[k].v[0] - s_u[0], w1 = (double)rec[k].v[1] - s_u[1],
                         w2 = (double)rec[k].v[2] - s_u[2];
            o[0] = dot3(w0, w1, w2, w0, w1, w2);
        });
        if (t == 0) {
            t_sum += (D.mass * tsum) / (double)(nn - 1);
            t_cells += 1.0;
        }
    }
    if constexpr (RULE == 1) {
        const double G = ordered_sums<NT, 3>(buf, cap, nn, [&](int k, double (&o)[3]) {
            uint64_t wv[4]; double z[3];
            philox<true>((uint64_t)coll, rec[k].id, 0, D.seed, TAG_THERMO, wv);
            normals3(wv, z);
#pragma unroll
            for (int d = 0; d < 3; ++d) o[d] = D.vscale * z[d];
        });
        if (t < 3) s_n[t] = G / (double)nn;
    }
    if (t < 64) {
        // bulk reaction: the jb-th of the nB B particles, 64 particles at a time
        int flipk = -1;
        if (D.bulk_on) {
            auto species = [&](int k0) { return __ballot(k0 + t < nn && (rec[k0 + t < nn ? k0 + t : 0].st & 1u) != 0u); };
            int nB = 0;
            for (int k0 = 0; k0 < nn; k0 += 64) nB += __popcll(species(k0));
            if (nB > 0) {
                uint64_t wv[4];
                philox<true>((uint64_t)coll, (uint64_t)cell, 0, D.seed, TAG_BULK, wv);
                const double P = D.ptable[nB < RMP_PTABLE ? nB : RMP_PTABLE - 1];
                if (u01(wv[0]) < P) {
                    int jb = (int)(u01(wv[1]) * (double)nB);
                    if (jb >= nB) jb = nB - 1;
                    for (int k0 = 0; k0 < nn && flipk < 0; k0 += 64) {
                        uint64_t m = species(k0);
                        const int c = __popcll(m);
                        if (jb < c) {
                            for (; jb > 0; --jb) m &= m - 1ull;
                            flipk = k0 + __ffsll((long long)m) - 1;
                        }
                        jb -= c;
                    }
                }
            }
        }
        if (t == 0) *s_flip = flipk;
    }
    __syncthreads();
    const double u0 = s_u[0], u1 = s_u[1], u2 = s_u[2];
    const int flipk = *s_flip;
    for (int k0 = 0; k0 < nn; k0 += NT) {
        const int k = k0 + t;
        bool cnd = false;
        if (k < nn) {
            Rec<T>* q = &rec[k];
            const double vv0 = (double)q->v[0], vv1 = (double)q->v[1], vv2 = (double)q->v[2];
            uint32_t s = q->st;
            double v3[3];
            if constexpr (RULE == 0) {
                const double nax[3] = {s_n[0], s_n[1], s_n[2]};
                double rw[3];
                rotate(nax, ca, sa, oma, vv0 - u0, vv1 - u1, vv2 - u2, rw);
                v3[0] = u0 + rw[0]; v3[1] = u1 + rw[1]; v3[2] = u2 + rw[2];
            } else {
                uint64_t wv[4]; double z[3];
                philox<true>((uint64_t)coll, q->id, 0, D.seed, TAG_THERMO, wv);
                normals3(wv, z);
                v3[0] = u0 + ((D.vscale * z[0]) - s_n[0]);
                v3[1] = u1 + ((D.vscale * z[1]) - s_n[1]);
                v3[2] = u2 + ((D.vscale * z[2]) - s_n[2]);
            }
            const double x0 = (double)q->x[0], x1 = (double)q->x[1], x2 = (double)q->x[2];
            if (k == flipk) {
                du_sum += species_dU(D, cp, nc, s_Xw, x0, x1, x2, 1, 0);
                n_flip += 1.0;
                s = 0u;
            }
            const T vt[3] = {(T)v3[0], (T)v3[1], (T)v3[2]};
            cnd = is_candidate(D, cp, nc, s_Xw, (uint8_t)s, x0, x1, x2, (double)vt[0], (double)vt[1], (double)vt[2]);
            for (int d = 0; d < 3; ++d) q->v[d] = vt[d];
            q->st = s;
        }
        list_flags(D, coll, (int64_t)q0 + k0 + (t & ~63), cnd);
    }
    __syncthreads();
}

// The wave's records of slots [0, ns) to dst, by lane and 64 u: through buf (64
// records of LDS), so that four lanes (FP32: two) write one record and each
// store instruction a contiguous kilobyte.  The 16-byte words of record r are
// rotated within it by its number, which spreads both accesses over the
// banks.  The buffer's old contents may be read until the call.
template <class T, int PPT>
__device__ __forceinline__ void records_out(char* buf, gptr<Rec<T>> dst, int ns, const T (&x)[PPT][3],
                                            const T (&v)[PPT][3], const uint32_t (&id)[PPT], const uint32_t (&st)[PPT])
{
    constexpr int W = RecWords<T>::W;
    const int lane = threadIdx.x & 63;
    u32x4* b = reinterpret_cast<u32x4*>(buf);
    const gptr<u32x4> out = (gptr<u32x4>)dst;
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        if (u * 64 >= ns) break;
        RecWords<T> r;
        r.pack(x[u], v[u], id[u], st[u]);
        wave_sync();
#pragma unroll
        for (int k = 0; k < W; ++k) b[lds_word<W>(lane, k)] = r.w[k];
        wave_sync();
        const int nw = (ns - u * 64 < 64 ? ns - u * 64 : 64) * W;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const int p = k * 64 + lane;
            const u32x4 q = b[lds_word<W>(p / W, p % W)];
            if (p < nw) out[(int64_t)u * 64 * W + p] = q;
        }
    }
}

// tile-local cell of slot q (a map of the tile's leading slots; binary search
// over the cell starts of the group [ga, gb) past its end)
__device__ __forceinline__ int cell_of_slot(const uint32_t* s_start, const uint8_t* s_cellof, int cap, uint32_t q,
                                            int ga, int gb)
{
    if (q - s_start[0] < (uint32_t)cap) return s_cellof[q - s_start[0]];
    int lo = ga, hi = gb - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_start[mid] <= q) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// MPCD collision on one tile of cells of the shifted grid (sort ranks
// [c0, c0 + TC)).  The sort permutation lists the tile's particles in the
// contiguous slots [start[c0], start[c0 + TC)), cell by cell (in any order
// within a cell).  The tile's cells are cut, in order, into runs of whole cells
// of at most CAP = 64 PPT particles; wave w of the workgroup takes runs w, w +
// NT / 64, ...  A wave works on its own: no workgroup barrier, so the waves of
// a compute unit wait for memory at different times.  Per run, lane l holding
// the slots l and l + 64:
//   B  gather the records of the slots' particles (the index loads went out a
//      run earlier);
//   C  rank each particle by old index among its cell's slots (the stable
//      order) and put it to LDS at its rank's slot;
//   D  one lane per cell and component: sequential FP64 sums in the stable
//      order, centre-of-mass velocity; the particles' |v - u|^2; one lane per
//      cell: temperature term, bulk reaction decision;
//   E  rotate about the cell's axis, apply the reaction, decide the
//      Verlet-list membership, write the records (through LDS, four lanes a
//      record, so that they leave as whole lines).
// A cell beyond CAP is left to the end, when the workgroup collides it
// (collide_big_cell; a launch of its own for these cost 4.4 us an interval
// even where there are none).
// Bound by memory: the records once in and once out, 2.8 GB in FP64 for 20.97 M
// particles, 530 us at the rate of a copy, measured 630 to 665 (FP32 405 to 440,
// where the gather fetches three times the records).  Scattering
// the records into cell order first and reading them back cost 557 + 714.
constexpr int RUN_CELLS = 24;        // cells per run at most

// VW: the partial sums of reaction energy and flips, one for each wave of a
// workgroup; a lone wave keeps four, by run, as four waves would, and the
// temperature terms are summed by cell, so that a tile's sums are the same
// whichever of the two forms its launch takes
template <class T, int PPT, int RULE, int VW>
struct alignas(16) CollideWave {
    static constexpr int CAP = 64 * PPT;
    T x[3][CAP], v[3][CAP];                  // by slot
    union {
        double sq[CAP];                      // |v - u|^2 (then thermostat draws) by slot
        uint32_t old[CAP];                   // old index by arrival
    };
    uint32_t id[CAP];
    uint8_t st[CAP];
    double u[RUN_CELLS][3];                  // centre-of-mass velocity
    double n[RUN_CELLS][3];                  // rotation axis; under the thermostat the mean draw
    double du[VW][2];                        // reaction energy and flips
    int16_t flip[RUN_CELLS];
    uint8_t go[RUN_CELLS];
};

template <class T, int RULE, int NT, int PPT, bool FLOW>
__global__ __launch_bounds__(NT, sizeof(T) == 4 && RULE == 0 ? 5 : 4) void k_collide(Work w, int xcd_map)
{
    constexpr int CAP = 64 * PPT, NW = NT / 64;
    const int item = xcd_map ? xcd_range(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int rep = w.nrep == 1 ? 0 : find_rep(w.prefix, w.nrep, item);
    const int tile = w.nrep == 1 ? item : item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active || D.rule != RULE || D.dense || (D.flow != 0) != FLOW) return;
    constexpr int VW = NW == 1 ? 4 : 1;
    using Ctx = CollideWave<T, PPT, RULE, VW>;
    __shared__ Ctx s_w[NW];
    static_assert(sizeof(Ctx) - 176 >= 64 * sizeof(Rec<T>), "room for 64 records before du");
    __shared__ double s_ct[COLL_TCMAX];        // the cells' temperature terms
    __shared__ uint32_t s_start[COLL_TCMAX + 1];
    RepState* rs = D.rs;
    const ColloidParams* cp = D.cp;
    const int nc = D.nc;
    const int t = threadIdx.x, lane0 = t & 63;
    const int wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(t >> 6);
    Ctx& S = s_w[wave];
    const int TC = D.tile_cells;
    const int64_t c0 = (int64_t)tile * TC;
    const int ncl = (int)((c0 + TC < D.ncell ? c0 + TC : D.ncell) - c0);
    // lane l: first slot of cell l of the tile, and of the cell after it
    const uint32_t sl0 = G(D.start)[c0 + (lane0 < ncl ? lane0 : ncl)];
    const uint32_t tend = G(D.start)[c0 + ncl];
    const bool cull = RULE == 0 && nc > 0 && !FLOW;
    const uint32_t all_mask = nc >= 32 ? 0xffffffffu : ((1u << nc) - 1u);
    const uint32_t tmask = cull ? G(D.tilemask)[tile] : all_mask;
    const int64_t coll = rs->coll_step;
    const double (*Xw)[3] = rs->Xw;
    const int cur = (int)(coll & 1), nxt = cur ^ 1;
    uint32_t sl1 = __shfl_down(sl0, 1, 64);
    if (lane0 >= ncl - 1) sl1 = tend;
    if (t < ncl) G(D.count)[c0 + t] = 0u;      // for the next binning
    // cell starts: every wave writes the same values, and so may read them
    // after its own write
    if (lane0 < ncl) s_start[lane0] = sl0;
    if (lane0 == 0) {
        s_start[ncl] = tend;
#pragma unroll
        for (int q = 0; q < VW; ++q) S.du[q][0] = S.du[q][1] = 0.0;
    }

    const gptr<const Rec<T>> src = G((const Rec<T>*)recs<T>(D, cur));
    const gptr<Rec<T>> dst = G(recs<T>(D, nxt));
    const gptr<const uint32_t> perm = G((const uint32_t*)D.perm);
    const gptr<const double> axes = G((const double*)D.axes);
    const double ca = D.ca, sa = D.sa, oma = 1.0 - D.ca;

    int t_cells = 0;           // cells with a temperature term (uniform)
    uint64_t big = 0;          // cells beyond a run's capacity (the same in every wave)
    int ga = 0, nrun = 0;
    // this wave's next run: cells [a, a + nrc) of the tile, slots [q0, q0 + ns)
    int a = 0, nrc = 0, ns = 0;
    uint32_t q0 = 0;
    auto next_run = [&]() {
        while (ga < ncl) {
            // the longest run of cells from ga whose particles fit
            q0 = (uint32_t)__builtin_amdgcn_readlane((int)sl0, ga);
            const uint64_t fit =
                __ballot(lane0 >= ga && lane0 < ncl && lane0 < ga + RUN_CELLS && sl1 - q0 <= (uint32_t)CAP);
            if (fit == 0ull) {
                big |= 1ull << ga;     // one cell beyond the capacity
                ++ga;
                continue;
            }
            a = ga;
            nrc = __popcll(fit);
            ga += nrc;
            ns = (int)((uint32_t)__builtin_amdgcn_readlane((int)sl1, ga - 1) - q0);
            if ((nrun++ & (NW - 1)) == wave && ns > 0) return;
        }
        ns = 0;
    };
    uint32_t pj[PPT];          // array positions of the run's particles, loaded a run ahead
    auto load_perm = [&]() {
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int j = lane0 + u * 64;
            pj[u] = j < ns ? perm[q0 + j] : 0u;
        }
    };
    next_run();
    load_perm();
    while (ns > 0) {
        wave_sync();                                             // the last run's reads are done
        // an opaque copy per run: per-lane addresses are formed where they are
        // used; hoisted out of the loop they spilled, and their reloads waited
        // behind the stores in flight
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        // ---- B
        T xq[PPT][3], vq[PPT][3];
        uint32_t idq[PPT], stq[PPT], pc[PPT];
        int lc[PPT];                                             // cell of the slot, from a
        const int a0 = a, nr = nrc, n1 = ns, dq = (nrun - 1) & (VW - 1);
        const uint32_t q1 = q0;
#pragma unroll
        for (int u = 0; u < PPT; ++u) rec_load<T>(src + (int64_t)pj[u], xq[u], vq[u], idq[u], stq[u]);
        double ax[2] = {0.0, 0.0};
        if constexpr (RULE == 0)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (lane + 64 * q < 3 * nr) ax[q] = axes[3 * (c0 + a0) + lane + 64 * q];
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            pc[u] = pj[u];
            if (lane + u * 64 < n1) S.old[lane + u * 64] = pc[u];
        }
        // the run after this one
        next_run();
        load_perm();
        // cell of each slot: the run's cell boundaries at or below it (the
        // same by arrival and by slot: a cell's slots are one range)
#pragma unroll
        for (int u = 0; u < PPT; ++u) lc[u] = 0;
        for (int k = 1; k < nr; ++k) {
            const int bound = (int)((uint32_t)__builtin_amdgcn_readlane((int)sl0, a0 + k) - q1);
#pragma unroll
            for (int u = 0; u < PPT; ++u) lc[u] += lane + u * 64 >= bound ? 1 : 0;
        }
        wave_sync();
        // ---- C
        float gv2 = 0.0f;
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int j = lane + u * 64;
            if (j < n1) {
                const int cb = (int)(s_start[a0 + lc[u]] - q1), ce = (int)(s_start[a0 + lc[u] + 1] - q1);
                const uint32_t p = pc[u];
                const T (&xr)[3] = xq[u];
                const T (&vr)[3] = vq[u];
                int r = 0, q = cb;
                for (; q + 4 <= ce; q += 4)
                    r += (S.old[q] < p ? 1 : 0) + (S.old[q + 1] < p ? 1 : 0) + (S.old[q + 2] < p ? 1 : 0) +
                         (S.old[q + 3] < p ? 1 : 0);
                for (; q < ce; ++q) r += S.old[q] < p ? 1 : 0;
                const int sl = cb + r;
#pragma unroll
                for (int d = 0; d < 3; ++d) { S.x[d][sl] = xr[d]; S.v[d][sl] = vr[d]; }
                S.id[sl] = idq[u];
                S.st[sl] = (uint8_t)stq[u];
                if (cull) {
                    // largest |v|^2 rounded up in FP32, for the tile mask (inf
                    // or NaN: no cull)
                    const double vv = dot3((double)vr[0], (double)vr[1], (double)vr[2], (double)vr[0], (double)vr[1],
                                           (double)vr[2]);
                    const float f = vv <= 1e30 ? (float)vv * 1.000001f : 3e38f;
                    gv2 = f > gv2 ? f : gv2;
                }
            }
        }
        if constexpr (RULE == 0)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (lane + 64 * q < 3 * nr) (&S.n[0][0])[lane + 64 * q] = ax[q];
        uint32_t cmask = tmask;
        if (cull && cmask != all_mask && __ballot((double)gv2 > D.vcap * D.vcap) != 0ull) cmask = all_mask;
        wave_sync();
        // every particle by slot now (read back from LDS where it is needed)
        uint64_t mB[PPT];
#pragma unroll
        for (int u = 0; u < PPT; ++u) mB[u] = __ballot(lane + u * 64 < n1 && (S.st[lane + u * 64] & 1) != 0);
        // ---- D: sums by cell and component
        for (int q = lane; q < 3 * nr; q += 64) {
            const int k = q / 3, d = q - 3 * k;
            const int cb = (int)(s_start[a0 + k] - q1), ce = (int)(s_start[a0 + k + 1] - q1);
            const int nn = ce - cb;
            // Lamura et al. (2001): a cell of the first or last layer (cut by
            // a plate) with fewer than n0 particles holds n0 - n virtual ones
            // at rest on average; only their summed momentum enters, a normal
            // vector of variance (n0 - n) kT / m per component
            bool virt = false;
            uint64_t cell = 0;
            if (FLOW && D.walls && nn >= 1 && nn < D.wall_n0) {
                cell = (uint64_t)(D.hbits == KEY_ROW ? c0 + a0 + k : G(D.cell_of)[c0 + a0 + k]);
                const int64_t cz = (int64_t)cell / ((int64_t)D.L[0] * D.L[1]);
                virt = cz == 0 || cz == D.L[2] - 1;
            }
            double s = 0.0;
            for (int i = cb; i < ce; ++i) s = s + (double)S.v[d][i];
            double um;
            if (FLOW && virt) {
                uint64_t wv[4]; double z[3];
                philox<true>((uint64_t)coll, cell, 0, D.seed, TAG_VIRT, wv);
                normals3(wv, z);
                const double sd = sqrt((double)(D.wall_n0 - nn)) * D.vscale;
                um = (s + (sd * (d == 0 ? z[0] : d == 1 ? z[1] : z[2]))) / (double)D.wall_n0;
            } else {
                um = s / (double)nn;
            }
            const bool go = nn >= 2 || virt;
            // a non-finite centre-of-mass velocity would spread through its
            // cell: latched for the caller
            if (go && !isfinite(um)) atomicOr(&rs->flags, RMP_FLAG_NONFINITE);
            S.u[k][d] = um;
            if (d == 0) {
                S.go[k] = (uint8_t)((go ? 1 : 0) | (virt ? 2 : 0));
                S.flip[k] = -1;
            }
        }
        wave_sync();
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int sl = lane + u * 64;
            const double w0 = (double)S.v[0][sl] - S.u[lc[u]][0], w1 = (double)S.v[1][sl] - S.u[lc[u]][1],
                         w2 = (double)S.v[2][sl] - S.u[lc[u]][2];
            S.sq[sl] = dot3(w0, w1, w2, w0, w1, w2);
        }
        wave_sync();
        {
            bool tc = false, flips = false;
            if (lane < nr) {
                const int cb = (int)(s_start[a0 + lane] - q1), ce = (int)(s_start[a0 + lane + 1] - q1);
                double term = 0.0;
                if (S.go[lane] == 1) {
                    double tsum = 0.0;
                    for (int i = cb; i < ce; ++i) tsum = tsum + S.sq[i];
                    term = (D.mass * tsum) / (double)(ce - cb - 1);
                    tc = true;
                }
                s_ct[a0 + lane] = term;
                if (D.bulk_on) {
                    // the cell's B particles: bits [cb, ce) of the species masks
                    int nB = 0;
                    uint64_t mine[PPT];
#pragma unroll
                    for (int u = 0; u < PPT; ++u) {
                        const int l0 = cb - 64 * u > 0 ? cb - 64 * u : 0, l1 = ce - 64 * u < 64 ? ce - 64 * u : 64;
                        const uint64_t ones = l1 - l0 >= 64 ? ~0ull : ((1ull << ((l1 - l0) & 63)) - 1ull);
                        mine[u] = l1 > l0 ? mB[u] & (ones << (l0 & 63)) : 0ull;
                        nB += __popcll(mine[u]);
                    }
                    if (nB > 0) {
                        const double P = G(D.ptable)[nB < RMP_PTABLE ? nB : RMP_PTABLE - 1];
                        const gptr<const double> bulk = G((const double*)D.bulk) + 2 * (c0 + a0 + lane);
                        if (bulk[0] < P) {
                            int jb = (int)(bulk[1] * (double)nB);
                            if (jb >= nB) jb = nB - 1;
                            flips = true;
#pragma unroll
                            for (int u = 0; u < PPT; ++u)
                                for (uint64_t m = mine[u]; m; m &= m - 1ull)
                                    if (jb-- == 0) S.flip[lane] = (int16_t)(64 * u + __ffsll((long long)m) - 1);
                        }
                    }
                }
            }
            t_cells += __popcll(__ballot(tc));
            if (__ballot(flips) != 0ull) {
                // potential change of the flipped particles (one per cell at most)
                wave_sync();
                double du = 0.0, nf = 0.0;
                if (flips) {
                    const int sl = S.flip[lane];
                    du = species_dU(D, cp, nc, Xw, (double)S.x[0][sl], (double)S.x[1][sl], (double)S.x[2][sl], 1, 0);
                    nf = 1.0;
                }
                du = wave_tree_sum(du);
                nf = wave_tree_sum(nf);
                if (lane == 0) {
                    S.du[dq][0] += du;
                    S.du[dq][1] += nf;
                }
            }
        }
        // the velocity after the collision is u + (draw - mean draw) under the
        // thermostat: the draws by slot, their cell means by cell, component
        // by component
        double gd[RULE ? PPT : 1][3];
        if constexpr (RULE == 1) {
#pragma unroll
            for (int u = 0; u < PPT; ++u) {
#pragma unroll
                for (int d = 0; d < 3; ++d) gd[u][d] = 0.0;
                if (lane + u * 64 < n1) {
                    uint64_t wv[4]; double z[3];
                    philox<true>((uint64_t)coll, S.id[lane + u * 64], 0, D.seed, TAG_THERMO, wv);
                    normals3(wv, z);
#pragma unroll
                    for (int d = 0; d < 3; ++d) gd[u][d] = D.vscale * z[d];
                }
            }
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                wave_sync();
#pragma unroll
                for (int u = 0; u < PPT; ++u) S.sq[lane + u * 64] = gd[u][d];
                wave_sync();
                if (lane < nr) {
                    const int cb = (int)(s_start[a0 + lane] - q1), ce = (int)(s_start[a0 + lane + 1] - q1);
                    double g = 0.0;
                    for (int i = cb; i < ce; ++i) g = g + S.sq[i];
                    S.n[lane][d] = g / (double)(ce - cb);
                }
            }
        }
        wave_sync();
        // ---- E
        T xr[PPT][3], vr[PPT][3];
        uint32_t idr[PPT], so[PPT];
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int sl = lane + u * 64, k = lc[u];
            bool cnd = false;
            so[u] = idr[u] = 0u;
#pragma unroll
            for (int d = 0; d < 3; ++d) xr[u][d] = vr[u][d] = (T)0;
            if (sl < n1) {
#pragma unroll
                for (int d = 0; d < 3; ++d) { xr[u][d] = S.x[d][sl]; vr[u][d] = S.v[d][sl]; }
                idr[u] = S.id[sl];
                so[u] = S.st[sl];
                if ((S.go[k] & 1) != 0) {
                    const double u0 = S.u[k][0], u1 = S.u[k][1], u2 = S.u[k][2];
                    double v3[3];
                    if constexpr (RULE == 0) {
                        const double nax[3] = {S.n[k][0], S.n[k][1], S.n[k][2]};
                        double rw[3];
                        rotate(nax, ca, sa, oma, (double)vr[u][0] - u0, (double)vr[u][1] - u1, (double)vr[u][2] - u2, rw);
                        v3[0] = u0 + rw[0]; v3[1] = u1 + rw[1]; v3[2] = u2 + rw[2];
                    } else {
                        v3[0] = u0 + (gd[u][0] - S.n[k][0]);
                        v3[1] = u1 + (gd[u][1] - S.n[k][1]);
                        v3[2] = u2 + (gd[u][2] - S.n[k][2]);
                    }
#pragma unroll
                    for (int d = 0; d < 3; ++d) vr[u][d] = (T)v3[d];
                }
                if (S.flip[k] == sl) so[u] = 0u;
                cnd = !FLOW && is_candidate_masked(D, cp, cmask, Xw, (uint8_t)so[u], (double)xr[u][0], (double)xr[u][1],
                                          (double)xr[u][2], (double)vr[u][0], (double)vr[u][1], (double)vr[u][2]);
            }
            list_flags(D, coll, (int64_t)q1 + u * 64, cnd);
        }
        records_out<T, PPT>(reinterpret_cast<char*>(&S), dst + (int64_t)q1, n1, xr, vr, idr, so);
    }
    const int lane = lane0;
    // the tile's sums: the temperature terms over its cells (those of a run; the
    // others have none), the rest over the waves in order
    __shared__ double s_red[NW * VW][3];
    if (lane < VW) {
        s_red[wave * VW + lane][0] = lane == 0 ? (double)t_cells : 0.0;
        s_red[wave * VW + lane][1] = S.du[lane][0];
        s_red[wave * VW + lane][2] = S.du[lane][1];
    }
    if constexpr (NW > 1) __syncthreads();
    else wave_sync();
    double part = 0.0;
    if (wave == 0) {
        const uint32_t nn = sl1 - sl0;
        const double tsum = wave_tree_sum(lane < ncl && nn >= 2u && nn <= (uint32_t)CAP ? s_ct[lane] : 0.0);
        if (t == 0) part = tsum;
        else if (t < 4)
#pragma unroll
            for (int q = 0; q < NW * VW; ++q) part = part + s_red[q][t - 1];
    }
    if (big != 0ull) {
        // cells beyond a run's capacity, one after the other, by the workgroup
        // (their temperature, reaction energy and flips after the others')
        __shared__ double s_bu[3], s_bn[3], s_bred[(NT / 64 + 1) * 4], s_bsum[4];
        __shared__ int32_t s_bflip;
        // (the waves' runs are done: their LDS holds the terms)
        double* buf = reinterpret_cast<double*>(s_w);
        constexpr int BIG_CAP = (int)(sizeof(s_w) / 24) & ~3;
        double b_sum = 0.0, b_cells = 0.0, b_du = 0.0, b_flip = 0.0;
        for (uint64_t m = big; m; m &= m - 1) {
            const int k = __ffsll((long long)m) - 1;
            const int64_t cell = D.hbits == KEY_ROW ? c0 + k : D.cell_of[c0 + k];
            const uint32_t q0b = D.start[c0 + k];
            const int nn = (int)(D.start[c0 + k + 1] - q0b);
            big_draws<RULE, FLOW>(D, coll, cell, s_bu, s_bn);
            __syncthreads();
            collide_big_cell<T, RULE, NT, FLOW>(D, cp, nc, Xw, coll, cell, q0b, nn, buf, BIG_CAP, s_bu, s_bn, &s_bflip, b_sum,
                                          b_cells, b_du, b_flip);
        }
        double br[4] = {b_sum, b_cells, b_du, b_flip};
        block_sum_n<NT, 4>(br, s_bred);
        if (t == 0)
            for (int j = 0; j < 4; ++j) s_bsum[j] = br[j];
        __syncthreads();
        if (t < 4) part = part + s_bsum[t];
    }
    if (t < 4) G(D.tpart)[(int64_t)tile * 4 + t] = part;
}

// The same collision for dense systems (more than DENSE_RHO particles per
// cell), where a wave's 128 slots would hold too few whole cells.  The tile's
// cells are taken in groups whose particles fit the workgroup (NT threads
// holding PPT particles each); usually the whole tile is one group.  Phases as
// above, with workgroup barriers between them.
template <class T, int RULE, int NT, int PPT>
__global__ __launch_bounds__(NT, RULE ? 3 : 4) void k_collide_dense(Work w, int xcd_map)
{
    constexpr int CAP = NT * PPT;
    constexpr int FILLCAP = 2 * CAP;    // leading slots of the tile with their cell in s_cellof
    const int item = xcd_map ? xcd_range(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int rep = find_rep(w.prefix, w.nrep, item);
    const int tile = item - w.prefix[rep];
    const RepDesc& D = w.desc[rep];
    if (!D.active || D.rule != RULE || !D.dense) return;
    RepState* rs = D.rs;
    const ColloidParams* cp = D.cp;
    const int nc = cp->nc;
    const int t = threadIdx.x;
    const int lane = t & 63;

    __shared__ uint32_t s_start[COLL_TCMAX + 1];
    __shared__ uint8_t s_cellof[FILLCAP];
    __shared__ uint32_t s_perm[CAP];
    __shared__ T s_x[3][CAP];
    __shared__ T s_v[3][CAP];
    __shared__ uint32_t s_id[CAP];
    __shared__ double s_g[3][RULE ? CAP : 1];
    __shared__ uint8_t s_st[CAP];
    __shared__ double s_u[COLL_TCMAX][3], s_n[COLL_TCMAX][3];
    __shared__ double s_b[COLL_TCMAX][2];       // bulk-reaction uniforms
    __shared__ double s_z[COLL_TCMAX][3];       // virtual-momentum normal of a plate-layer cell
    __shared__ int32_t s_flip[COLL_TCMAX];
    __shared__ uint8_t s_go[COLL_TCMAX];
    __shared__ double s_Xw[MAXC][3];
    __shared__ uint64_t s_vmax2;       // max |v|^2 (bit patterns order like the values)
    __shared__ double sred[(NT / 64 + 1) * 4];

    const int64_t coll = rs->coll_step;
    const int cur = (int)(coll & 1), nxt = cur ^ 1;
    const int TC = D.tile_cells;
    const int64_t c0 = (int64_t)tile * TC;
    const int64_t c1 = (c0 + TC < D.ncell) ? c0 + TC : D.ncell;
    const int ncl = (int)(c1 - c0);
    // the colloid cull needs a bound on the speed after the collision:
    // the rotation gives one (below), the thermostat's fresh draws do not
    const bool cull = RULE == 0 && nc > 0 && !D.flow;

    // ---- A: cell starts (and the counters zeroed for the next binning); the
    //         cells' draws; colloid images
    for (int k = t; k <= ncl; k += NT) {
        s_start[k] = G(D.start)[c0 + k];
        if (k < ncl) G(D.count)[c0 + k] = 0;
    }
    if constexpr (RULE == 0)
        for (int q = t; q < 3 * ncl; q += NT) s_n[q / 3][q % 3] = G(D.axes)[3 * c0 + q];
    if (D.bulk_on)
        for (int q = t; q < 2 * ncl; q += NT) s_b[q / 2][q % 2] = G(D.bulk)[2 * c0 + q];
    if (D.walls) {
        // plates (flows have no colloids): the virtual-momentum normal of
        // every cell of the first and last layer, used if the cell turns
        // out to be cut and under-filled
        for (int lc = t; lc < ncl; lc += NT) {
            const int64_t cell = D.hbits == KEY_ROW ? c0 + lc : G(D.cell_of)[c0 + lc];
            const int64_t cz = cell / ((int64_t)D.L[0] * D.L[1]);
            if (cz == 0 || cz == D.L[2] - 1) {
                uint64_t wv[4]; double z[3];
                philox<true>((uint64_t)coll, (uint64_t)cell, 0, D.seed, TAG_VIRT, wv);
                normals3(wv, z);
                s_z[lc][0] = z[0]; s_z[lc][1] = z[1]; s_z[lc][2] = z[2];
            }
        }
    } else if (t < nc) {
        for (int d = 0; d < 3; ++d) s_Xw[t][d] = colloid_image(G(rs)->X[t][d], D.Ld[d]);
    }
    if (t < 64 && lane < ncl) {
        // tile-local cell of each of the tile's first FILLCAP slots (the
        // cells' slot ranges are contiguous and in order)
        const uint32_t base = G(D.start)[c0], a = G(D.start)[c0 + lane], b = G(D.start)[c0 + lane + 1];
        const uint32_t e = b - base < (uint32_t)FILLCAP ? b - base : (uint32_t)FILLCAP;
        for (uint32_t r = a - base; r < e; ++r) s_cellof[r] = (uint8_t)lane;
    }
    if (t == 64) s_vmax2 = 0ull;
    __syncthreads();

    const gptr<const Rec<T>> src = G((const Rec<T>*)recs<T>(D, cur));
    const gptr<Rec<T>> dst = G(recs<T>(D, nxt));
    const gptr<const uint32_t> perm = G((const uint32_t*)D.perm);
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
        // ---- B: records of the group's slots
        T xr[PPT][3], vr[PPT][3];
        uint32_t idr[PPT], pj[PPT], sr[PPT];
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int j = t + u * NT;
            pj[u] = j < ns ? perm[q0 + j] : 0u;
        }
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int j = t + u * NT;
            rec_load<T>(src + (int64_t)pj[u], xr[u], vr[u], idr[u], sr[u]);
            if (j < ns) s_perm[j] = pj[u];
        }
        __syncthreads();
        // ---- C: stable rank; the particle to LDS at the rank's slot
        double gv2 = 0.0;
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int j = t + u * NT;
            if (j < ns) {
                const int lc = cell_of_slot(s_start, s_cellof, FILLCAP, q0 + (uint32_t)j, ga, gb);
                const int cb = (int)(s_start[lc] - q0), ce = (int)(s_start[lc + 1] - q0);
                const uint32_t p = pj[u];
                int r = 0, q = cb;
                for (; q + 4 <= ce; q += 4)
                    r += (s_perm[q] < p ? 1 : 0) + (s_perm[q + 1] < p ? 1 : 0) + (s_perm[q + 2] < p ? 1 : 0) +
                         (s_perm[q + 3] < p ? 1 : 0);
                for (; q < ce; ++q) r += s_perm[q] < p ? 1 : 0;
                const int sl = cb + r;
#pragma unroll
                for (int d = 0; d < 3; ++d) { s_x[d][sl] = xr[u][d]; s_v[d][sl] = vr[u][d]; }
                s_id[sl] = idr[u];
                s_st[sl] = (uint8_t)sr[u];
                if constexpr (RULE == 1) {
                    uint64_t wv[4]; double z[3];
                    philox<true>((uint64_t)coll, idr[u], 0, D.seed, TAG_THERMO, wv);
                    normals3(wv, z);
                    s_g[0][sl] = D.vscale * z[0];
                    s_g[1][sl] = D.vscale * z[1];
                    s_g[2][sl] = D.vscale * z[2];
                }
                if (cull) {
                    // the largest speed vmax of the tile's particles, for the
                    // colloid cull: after the rotation a speed is at most
                    // |u| + |v - u| <= 3 vmax
                    const double vv = dot3((double)vr[u][0], (double)vr[u][1], (double)vr[u][2],
                                           (double)vr[u][0], (double)vr[u][1], (double)vr[u][2]);
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
        // ---- D: per cell (one thread each)
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
        __syncthreads();
        // ---- E: rotate (or thermostat), react, write, Verlet-list flag
        // the tile's mask holds up to the speed vcap; beyond it, and under the
        // thermostat's fresh draws, every colloid is tested
        const bool slow = __longlong_as_double((long long)s_vmax2) <= D.vcap * D.vcap;
        const uint32_t cmask = cull && slow ? G(D.tilemask)[tile] : (nc >= 32 ? 0xffffffffu : ((1u << nc) - 1u));
        int fl[PPT];               // slot of a flipped particle, or -1
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int sl = t + u * NT;
            bool cnd = false;
            fl[u] = -1;
            if (sl < ns) {
                const int cl = cell_of_slot(s_start, s_cellof, FILLCAP, q0 + (uint32_t)sl, ga, gb);
                double v3[3] = {(double)s_v[0][sl], (double)s_v[1][sl], (double)s_v[2][sl]};
                if (s_go[cl]) {
                    const double u0 = s_u[cl][0], u1 = s_u[cl][1], u2 = s_u[cl][2];
                    if constexpr (RULE == 0) {
                        const double nax[3] = {s_n[cl][0], s_n[cl][1], s_n[cl][2]};
                        double rw[3];
                        rotate(nax, ca, sa, oma, v3[0] - u0, v3[1] - u1, v3[2] - u2, rw);
                        v3[0] = u0 + rw[0]; v3[1] = u1 + rw[1]; v3[2] = u2 + rw[2];
                    } else {
                        v3[0] = u0 + (s_g[0][sl] - s_n[cl][0]);
                        v3[1] = u1 + (s_g[1][sl] - s_n[cl][1]);
                        v3[2] = u2 + (s_g[2][sl] - s_n[cl][2]);
                    }
                }
                uint32_t s = s_st[sl];
                if (s_flip[cl] == sl) {
                    fl[u] = sl;
                    n_flip += 1.0;
                    s = 0u;
                }
                const T xo[3] = {s_x[0][sl], s_x[1][sl], s_x[2][sl]};
                const T vo[3] = {(T)v3[0], (T)v3[1], (T)v3[2]};
                cnd = is_candidate_masked(D, cp, cmask, s_Xw, (uint8_t)s, (double)xo[0], (double)xo[1], (double)xo[2],
                                          (double)vo[0], (double)vo[1], (double)vo[2]);
                rec_store<T, RecWords<T>::W>(dst + ((int64_t)q0 + sl), xo, vo, s_id[sl], s);
            }
            list_flags(D, coll, (int64_t)q0 + u * NT + (t & ~63), cnd);
        }
        // the potential change of a flipped particle, in the same order per
        // thread, after the writes: inside their loop its colloid loop
        // raised the register peak beyond the budget (spills to scratch)
#pragma unroll
        for (int u = 0; u < PPT; ++u)
            if (fl[u] >= 0)
                du_sum += species_dU(D, cp, nc, s_Xw, (double)s_x[0][fl[u]], (double)s_x[1][fl[u]],
                                     (double)s_x[2][fl[u]], 1, 0);
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

// The cells that k_collide_dense found beyond a group's capacity (a bit per
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
    constexpr int BIG_CAP = 512;
    __shared__ __attribute__((aligned(16))) double s_buf[3 * BIG_CAP];
    const int item0 = blockIdx.x * 64;
    bool any = false;
    if (t < 64) {
        const int item = item0 + t;
        uint64_t m = 0;
        if (item < n_items) {
            const int rep = find_rep(w.prefix, w.nrep, item);
            const RepDesc& D = w.desc[rep];
            if (D.active && D.rule == RULE && D.dense) m = D.bigmask[item - w.prefix[rep]];
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
            big_draws<RULE, true>(D, coll, cell, s_u, s_n);
            __syncthreads();
            collide_big_cell<T, RULE, NT, true>(D, cp, nc, s_Xw, coll, cell, q0, nn, s_buf, BIG_CAP, s_u, s_n, &s_flip,
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
// state: where a copy of the replica's state goes (nullptr: nowhere); part and
// state may be host memory.
template <class T>
__global__ __launch_bounds__(256) void k_observe(Work w, double* part, RepState* state)
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
    if (state && chunk == 0) {
        static_assert(sizeof(RepState) % 8 == 0, "copied as 64-bit words");
        for (int k = threadIdx.x; k < (int)(sizeof(RepState) / 8); k += 256)
            ((uint64_t*)state)[k] = ((const uint64_t*)D.rs)[k];
    }
    double P0 = 0.0, P1 = 0.0, P2 = 0.0, ke = 0.0, nb = 0.0;
    for (int j = threadIdx.x; j < CHUNK; j += 256) {
        int64_t i = base + j;
        if (i >= n) break;
        const Rec<T>* q = recs<T>(D, cur) + i;
        const double v0 = q->v[0], v1 = q->v[1], v2 = q->v[2];
        P0 += v0; P1 += v1; P2 += v2;
        ke += dot3(v0, v1, v2, v0, v1, v2);
        nb += (double)(q->st & 1u);
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

// --------------------------------------------------- exchange with the host
// Fields of the records of buffer b as contiguous arrays, by the bits of
// `what`: 1 positions, 2 velocities (three arrays of doubles each, exact from
// FP32, rounded to it), one after the other in the other record buffer, whose
// contents are spent between intervals; 4 ids, then state bytes, in xchg; 8
// positions and velocities as stored instead of doubles.
template <class T>
__global__ __launch_bounds__(256) void k_fields_out(const RepDesc* Dp, int b, int what)
{
    const RepDesc& D = *Dp;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, n = D.n;
    if (i >= n) return;
    T x[3], v[3];
    uint32_t id, st;
    rec_load<T>((gptr<const Rec<T>>)(recs<T>(D, b) + i), x, v, id, st);
    if (what & 8) {
        T* q = reinterpret_cast<T*>(recs<T>(D, b ^ 1)) + i;
        for (int d = 0; d < 3; ++d, q += n) *q = x[d];
        for (int d = 0; d < 3; ++d, q += n) *q = v[d];
    }
    double* o = reinterpret_cast<double*>(recs<T>(D, b ^ 1)) + i;
    if (what & 1)
        for (int d = 0; d < 3; ++d, o += n) *o = (double)x[d];
    if (what & 2)
        for (int d = 0; d < 3; ++d, o += n) *o = (double)v[d];
    if (what & 4) {
        reinterpret_cast<uint32_t*>(D.xchg)[i] = id;
        (reinterpret_cast<uint8_t*>(D.xchg) + 4 * n)[i] = (uint8_t)st;
    }
}

template <class T>
__global__ __launch_bounds__(256) void k_fields_in(const RepDesc* Dp, int b, int what)
{
    const RepDesc& D = *Dp;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, n = D.n;
    if (i >= n) return;
    Rec<T>* r = recs<T>(D, b) + i;
    const double* o = reinterpret_cast<const double*>(recs<T>(D, b ^ 1)) + i;
    if (what & 1)
        for (int d = 0; d < 3; ++d, o += n) {
            const T xt = (T)*o;
            r->x[d] = (double)xt >= D.Ld[d] ? (T)0 : xt;    // FP32 rounding up to L
        }
    if (what & 2)
        for (int d = 0; d < 3; ++d, o += n) r->v[d] = (T)*o;
    if (what & 4) {
        r->id = reinterpret_cast<const uint32_t*>(D.xchg)[i];
        r->st = (reinterpret_cast<const uint8_t*>(D.xchg) + 4 * n)[i];
    }
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
        const Rec<T>* r = recs<T>(D, cur) + ic;
        px[q][0] = (double)r->x[0];
        px[q][1] = (double)r->x[1];
        px[q][2] = (double)r->x[2];
        psp[q] = (int)(r->st & 1u);
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
    template __global__ void k_close<T>(Work, int);                              \
    template __global__ void k_fields_out<T>(const RepDesc*, int, int);          \
    template __global__ void k_fields_in<T>(const RepDesc*, int, int);           \
    template __global__ void k_collide_big<T, 0>(Work, int);                     \
    template __global__ void k_collide_big<T, 1>(Work, int);                     \
    template __global__ void k_collide<T, 0, 64, 2, false>(Work, int); \
    template __global__ void k_collide<T, 0, 64, 2, true>(Work, int); \
    template __global__ void k_collide<T, 1, 64, 2, false>(Work, int); \
    template __global__ void k_collide<T, 1, 64, 2, true>(Work, int); \
    template __global__ void k_collide<T, 0, 64, 1, false>(Work, int); \
    template __global__ void k_collide<T, 0, 64, 1, true>(Work, int); \
    template __global__ void k_collide<T, 1, 64, 1, false>(Work, int); \
    template __global__ void k_collide<T, 1, 64, 1, true>(Work, int); \
    template __global__ void k_collide<T, 0, 256, 2, false>(Work, int); \
    template __global__ void k_collide<T, 0, 256, 2, true>(Work, int); \
    template __global__ void k_collide<T, 1, 256, 2, false>(Work, int); \
    template __global__ void k_collide<T, 1, 256, 2, true>(Work, int); \
    template __global__ void k_collide<T, 0, 512, 2, false>(Work, int); \
    template __global__ void k_collide<T, 0, 512, 2, true>(Work, int); \
    template __global__ void k_collide<T, 1, 512, 2, false>(Work, int); \
    template __global__ void k_collide<T, 1, 512, 2, true>(Work, int); \
    template __global__ void k_collide<T, 0, 256, 1, false>(Work, int); \
    template __global__ void k_collide<T, 0, 256, 1, true>(Work, int); \
    template __global__ void k_collide<T, 1, 256, 1, false>(Work, int); \
    template __global__ void k_collide<T, 1, 256, 1, true>(Work, int); \
    template __global__ void k_collide<T, 0, 512, 1, false>(Work, int); \
    template __global__ void k_collide<T, 0, 512, 1, true>(Work, int); \
    template __global__ void k_collide<T, 1, 512, 1, false>(Work, int); \
    template __global__ void k_collide<T, 1, 512, 1, true>(Work, int); \
    template __global__ void k_collide_dense<T, 0, 256, 2>(Work, int);           \
    template __global__ void k_collide_dense<T, 1, 256, 2>(Work, int);           \
    template __global__ void k_observe<T>(Work, double*, RepState*);                     \
    template __global__ void k_analysis<T>(Work);

template __global__ void k_perm<2, true>(Work, int);
template __global__ void k_perm<1, false>(Work, int);
template __global__ void k_perm<2, false>(Work, int);
template __global__ void k_perm<4, false>(Work, int);
RMP_INST(double)
RMP_INST(float)

}  // namespace rmp
