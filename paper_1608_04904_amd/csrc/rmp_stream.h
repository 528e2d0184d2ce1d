// Streaming of the particles outside the Verlet list, and the particle records
// it and the collision read and write.  The streaming is a kernel of its own
// and, in small launches, a part of the MD chain's launch.
#pragma once
#include "rmp_util.h"

namespace rmp {

// A record as 16-byte words (one global instruction each): FP64 (x0, x1),
// (x2, v0), (v1, v2), (id, st, 0, 0); FP32 (x0, x1, x2, v0), (v1, v2, id, st).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4 word16(double a, double b)
{
    return u32x4{(uint32_t)__double2loint(a), (uint32_t)__double2hiint(a), (uint32_t)__double2loint(b),
                 (uint32_t)__double2hiint(b)};
}
__device__ __forceinline__ double lo_d(u32x4 w) { return __hiloint2double((int)w.y, (int)w.x); }
__device__ __forceinline__ double hi_d(u32x4 w) { return __hiloint2double((int)w.w, (int)w.z); }

template <class T> struct RecWords;
template <> struct RecWords<double> {
    static constexpr int W = 4;
    u32x4 w[4];
    __device__ __forceinline__ void pack(const double (&x)[3], const double (&v)[3], uint32_t id, uint32_t st)
    {
        w[0] = word16(x[0], x[1]);
        w[1] = word16(x[2], v[0]);
        w[2] = word16(v[1], v[2]);
        w[3] = u32x4{id, st, 0u, 0u};
    }
    __device__ __forceinline__ void unpack(double (&x)[3], double (&v)[3], uint32_t& id, uint32_t& st) const
    {
        x[0] = lo_d(w[0]); x[1] = hi_d(w[0]); x[2] = lo_d(w[1]);
        v[0] = hi_d(w[1]); v[1] = lo_d(w[2]); v[2] = hi_d(w[2]);
        id = w[3].x; st = w[3].y;
    }
};
template <> struct RecWords<float> {
    static constexpr int W = 2;
    u32x4 w[2];
    __device__ __forceinline__ void pack(const float (&x)[3], const float (&v)[3], uint32_t id, uint32_t st)
    {
        w[0] = u32x4{__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(v[0])};
        w[1] = u32x4{__float_as_uint(v[1]), __float_as_uint(v[2]), id, st};
    }
    __device__ __forceinline__ void unpack(float (&x)[3], float (&v)[3], uint32_t& id, uint32_t& st) const
    {
        x[0] = __uint_as_float(w[0].x); x[1] = __uint_as_float(w[0].y); x[2] = __uint_as_float(w[0].z);
        v[0] = __uint_as_float(w[0].w); v[1] = __uint_as_float(w[1].x); v[2] = __uint_as_float(w[1].y);
        id = w[1].z; st = w[1].w;
    }
};

// Place of word k of record r in an LDS buffer of records: the words are
// rotated within a record by its number, which spreads an access by record
// and one by word over the banks.
template <int W>
__device__ __forceinline__ int lds_word(int r, int k)
{
    return r * W + (k ^ ((r >> (W == 4 ? 2 : 3)) & (W - 1)));
}

template <class T>
__device__ __forceinline__ void rec_load(gptr<const Rec<T>> r, T (&x)[3], T (&v)[3], uint32_t& id, uint32_t& st)
{
    RecWords<T> q;
    const gptr<const u32x4> p = (gptr<const u32x4>)r;
#pragma unroll
    for (int k = 0; k < RecWords<T>::W; ++k) q.w[k] = p[k];
    q.unpack(x, v, id, st);
}

// words [0, WORDS) of a record
template <class T, int WORDS>
__device__ __forceinline__ void rec_store(gptr<Rec<T>> r, const T (&x)[3], const T (&v)[3], uint32_t id, uint32_t st)
{
    RecWords<T> q;
    q.pack(x, v, id, st);
    const gptr<u32x4> p = (gptr<u32x4>)r;
#pragma unroll
    for (int k = 0; k < WORDS; ++k) p[k] = q.w[k];
}

// Per-cell random numbers of the coming collision, for the block of DRAW_CELLS
// sort ranks from lo: rotation axes and bulk-reaction uniforms.  Made by
// k_stream, which waits for its atomics anyway, because a wave's run of cells
// in the collision has a dozen only; in a sparse box, where that would leave
// many cells to few workgroups, by k_cells.  A Philox block takes 2000 cycles of a
// wave (64-bit products), so all lanes are kept at work: a workgroup does a
// whole block of cells, and the 5 % of the axes that both tries of their first
// Philox block miss are collected and tried again together.  (A share of the
// cells, 26 or 51, for each workgroup and waves repeating until their last
// lane had its axis: 128^3 FP64, 689 us for the streaming, now 633; FP32 451,
// now 410.)
constexpr int DRAW_CELLS = 256;

__device__ __forceinline__ void collision_draws(const RepDesc& D, int64_t lo)
{
    __shared__ uint32_t s_nq;
    __shared__ uint16_t s_q[DRAW_CELLS];
    const int t = threadIdx.x, bd = (int)blockDim.x;
    const uint64_t coll = (uint64_t)D.rs->coll_step;
    const int n = (int)(D.ncell - lo < DRAW_CELLS ? D.ncell - lo : DRAW_CELLS);
    if (t == 0) s_nq = 0u;
    __syncthreads();
    const gptr<double> axes = G(D.axes) + 3 * lo;
    const gptr<double> bulk = G(D.bulk) + 2 * lo;
    for (int k = t; k < n; k += bd) {
        const uint64_t cell = D.hbits == KEY_ROW ? (uint64_t)(lo + k) : (uint64_t)G(D.cell_of)[lo + k];
        if (D.rule == 0) {
            double a[3];
            if (marsaglia_axis<true>(D.seed, coll, cell, a, 0, 1)) {
                axes[3 * k] = a[0]; axes[3 * k + 1] = a[1]; axes[3 * k + 2] = a[2];
            } else {
                s_q[atomicAdd(&s_nq, 1u)] = (uint16_t)k;
            }
        }
        if (D.bulk_on) {
            uint64_t wv[4];
            philox<true>(coll, cell, 0, D.seed, TAG_BULK, wv);
            bulk[2 * k] = u01(wv[0]); bulk[2 * k + 1] = u01(wv[1]);
        }
    }
    __syncthreads();
    const int nq = (int)s_nq;
    for (int q = t; q < nq; q += bd) {
        const int k = s_q[q];
        const uint64_t cell = D.hbits == KEY_ROW ? (uint64_t)(lo + k) : (uint64_t)G(D.cell_of)[lo + k];
        double a[3];
        marsaglia_axis<true>(D.seed, coll, cell, a, 1);
        axes[3 * k] = a[0]; axes[3 * k + 1] = a[1]; axes[3 * k + 2] = a[2];
    }
    __syncthreads();
}

// Share of a replica's work list, cut over its particle workgroups
struct Share {
    int64_t me, all;
    __device__ int64_t lo(int64_t n) const { return n * me / all; }
    __device__ int64_t hi(int64_t n) const { return n * (me + 1) / all; }
};

// Streaming of the particles outside the Verlet list (flows: of all) over the
// interval, their cells in the coming collision and their ranks in them (any
// order: the collision restores the stable one).  Workgroup `sub` of a chunk
// covers particles [sub*span, (sub+1)*span) of it, span = blockDim.x * PPT;
// thread t holds particles t, t + blockDim.x, ... of its span, and every load
// is issued before the drifts.  The ranks are counted in LDS first, in a hash
// table of the workgroup's cell pairs (neighbours in the array go to a few rows
// of cells), and each pair takes one 64-bit atomic of both its counters: the
// atomics all go to memory, 0.2 a particle where one per run of equal keys in
// a wave made 0.5.  A list member's record, which the MD chain may be writing
// meanwhile, is loaded and not used: who is a member is read from the list bits,
// a word per wave.
// A wave reads and writes its 64 records through LDS so that each instruction
// covers a contiguous kilobyte (one lane a record: 80 us more).
// 20.97 M particles, 50 drifts: FP64 630 to 650 us, FP32 410 to 425.  The records, read whole
// and half written, are 2.0 and 1.0 GB, 380 and 190 us at the rate of a copy;
// with one drift instead of 50 it takes 540, and the draws for the cells cost
// about 30.
// b: the workgroup's place in the list of particle workgroups.
template <class T, int PPT, bool FLOW, int NT>
__device__ __forceinline__ void stream_body(const RepDesc* desc, const int32_t* prefix, int nrep, int b,
                                            int wg_per_chunk)
{
    constexpr int W = RecWords<T>::W;
    const int item = b / wg_per_chunk;
    const int sub = b - item * wg_per_chunk;
    const int rep = find_rep(prefix, nrep, item);
    const int chunk = item - prefix[rep];
    const RepDesc& D = desc[rep];
    if (!D.active || (D.flow != 0) != FLOW) return;
    const RepState* rs = D.rs;
    const gptr<Rec<T>> rec = G(recs<T>(D, (int)(rs->coll_step & 1)));
    const int64_t n = D.n;
    const int span = CHUNK / wg_per_chunk;
    const int64_t base = (int64_t)chunk * CHUNK + (int64_t)sub * span;
    const int lane = threadIdx.x & 63;
    __shared__ u32x4 s_rec[NT / 64][64 * W];       // a wave's 64 records
    u32x4* buf = s_rec[threadIdx.x >> 6];
    T x[PPT][3], v[PPT][3];
    bool go[PPT];
    uint32_t id[PPT], st[PPT];
    u32x4 in[PPT][W];
    uint64_t members[PPT];
    const gptr<const uint64_t> lbits = G((const uint64_t*)list_bits(D, rs->coll_step));
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const int64_t i0 = base + u * (int)blockDim.x + (threadIdx.x & ~63u);
        members[u] = FLOW ? 0ull : lbits[i0 >> 6];
        const int64_t left = (n - i0) * W;
        const gptr<const u32x4> p = (gptr<const u32x4>)rec + i0 * W;
#pragma unroll
        for (int k = 0; k < W; ++k) in[u][k] = k * 64 + lane < left ? p[k * 64 + lane] : u32x4{};
    }
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const int64_t i = base + u * (int)blockDim.x + threadIdx.x;
        RecWords<T> q;
        wave_sync();
#pragma unroll
        for (int k = 0; k < W; ++k) buf[lds_word<W>((k * 64 + lane) / W, (k * 64 + lane) % W)] = in[u][k];
        wave_sync();
#pragma unroll
        for (int k = 0; k < W; ++k) q.w[k] = buf[lds_word<W>(lane, k)];
        q.unpack(x[u], v[u], id[u], st[u]);
        go[u] = i < n && ((members[u] >> lane) & 1ull) == 0ull;
    }
    const double s[3] = {uniform_d(G(rs)->shift[0]), uniform_d(G(rs)->shift[1]), uniform_d(G(rs)->shift[2])};
    advance<T, PPT, FLOW>(D, x, v, go);
    // ranks among the workgroup's particles of each cell, by cell pair
    constexpr int SLOTS = 2 * NT * PPT;              // at most half filled
    constexpr uint32_t NONE = 0xffffffffu;
    __shared__ uint32_t s_pair[SLOTS], s_cnt[SLOTS][2];
    const int nslots = 2 * (int)blockDim.x * PPT;    // of this launch's workgroup size (a power of two)
    for (int k = threadIdx.x; k < nslots; k += (int)blockDim.x) {
        s_pair[k] = NONE;
        s_cnt[k][0] = s_cnt[k][1] = 0u;
    }
    __syncthreads();
    uint32_t key[PPT], rank[PPT];
    int slot[PPT];
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        key[u] = rank[u] = 0u;
        slot[u] = 0;
        if (go[u]) {
            key[u] = cell_key<FLOW>(D, (double)x[u][0], (double)x[u][1], (double)x[u][2], s);
            const uint32_t pair = key[u] >> 1;
            int q = (int)((pair * 0x9E3779B1u) >> 12) & (nslots - 1);
            while (true) {
                const uint32_t old = atomicCAS(&s_pair[q], NONE, pair);
                if (old == NONE || old == pair) break;
                q = (q + 1) & (nslots - 1);
            }
            slot[u] = q;
            rank[u] = atomicAdd(&s_cnt[q][key[u] & 1u], 1u);
        }
    }
    __syncthreads();
    // one 64-bit atomic per cell pair: both cells' counts
    constexpr int SPT = 2 * PPT;
    uint64_t got[SPT];
    bool have[SPT];
#pragma unroll
    for (int k = 0; k < SPT; ++k) {
        const int q = (int)threadIdx.x + k * (int)blockDim.x;
        const uint32_t pair = s_pair[q];
        have[k] = pair != NONE;
        got[k] = 0;
        if (have[k])
            got[k] = __hip_atomic_fetch_add((gptr<uint64_t>)G(D.count) + pair,
                                            (uint64_t)s_cnt[q][0] | ((uint64_t)s_cnt[q][1] << 32), __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const int64_t i0 = base + u * (int)blockDim.x + (threadIdx.x & ~63u);
        constexpr int WS = FLOW ? W : W / 2;         // a flow changes the velocity too
        const uint64_t m = __ballot(go[u]);
        RecWords<T> q;
        q.pack(x[u], v[u], id[u], st[u]);
        wave_sync();
#pragma unroll
        for (int k = 0; k < WS; ++k) buf[lds_word<W>(lane, k)] = q.w[k];
        wave_sync();
        const gptr<u32x4> p = (gptr<u32x4>)rec + i0 * W;
#pragma unroll
        for (int k = 0; k < WS; ++k) {
            const int r = (k * 64 + lane) / WS, part = (k * 64 + lane) % WS;
            if ((m >> r) & 1ull) p[r * W + part] = buf[lds_word<W>(r, part)];
        }
    }
    // the blocks of cells that fall to this workgroup
    if (!D.sparse) {
        const int64_t nblk = (D.ncell + DRAW_CELLS - 1) / DRAW_CELLS;
        const int64_t me = (int64_t)chunk * wg_per_chunk + sub, all = (int64_t)D.n_chunks * wg_per_chunk;
        for (int64_t j = (me * nblk + all - 1) / all; j < ((me + 1) * nblk + all - 1) / all; ++j)
            collision_draws(D, j * DRAW_CELLS);
    }
    // (a thread rewrites only the counts of its own slots, read above)
#pragma unroll
    for (int k = 0; k < SPT; ++k)
        if (have[k]) {
            const int q = (int)threadIdx.x + k * (int)blockDim.x;
            s_cnt[q][0] = (uint32_t)got[k];
            s_cnt[q][1] = (uint32_t)(got[k] >> 32);
        }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const int64_t i = base + u * (int)blockDim.x + threadIdx.x;
        if (go[u]) G(D.keyrank)[i] = ((uint64_t)key[u] << 32) | (s_cnt[slot[u]][key[u] & 1u] + rank[u]);
    }
}

}  // namespace rmp
