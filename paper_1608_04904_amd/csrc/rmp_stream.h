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

// Per-cell random numbers of the coming collision (sort ranks [lo, hi)):
// rotation axes (role 0) and bulk-reaction uniforms (role 1), one cell per
// lane.  Made by k_stream, with every lane at work, because a wave's run of
// cells in the collision has a dozen only; k_stream waits for its atomics
// anyway.
__device__ __forceinline__ void collision_draws(const RepDesc& D, int role, int64_t lo, int64_t hi)
{
    const int lane = threadIdx.x & 63;
    const RepState* rs = D.rs;
    const uint64_t coll = (uint64_t)rs->coll_step;
    if (role == 0 && D.rule == 0) {
        const gptr<double> axes = G(D.axes);
        for (int64_t r = lo + lane; r < hi; r += 64) {
            const uint64_t cell = D.hbits == KEY_ROW ? (uint64_t)r : (uint64_t)G(D.cell_of)[r];
            double a[3];
            marsaglia_axis<true>(D.seed, coll, cell, a);
            axes[3 * r] = a[0]; axes[3 * r + 1] = a[1]; axes[3 * r + 2] = a[2];
        }
    }
    if (role == 1 && D.bulk_on) {
        const gptr<double> bulk = G(D.bulk);
        for (int64_t r = lo + lane; r < hi; r += 64) {
            const uint64_t cell = D.hbits == KEY_ROW ? (uint64_t)r : (uint64_t)G(D.cell_of)[r];
            uint64_t wv[4];
            philox<true>(coll, cell, 0, D.seed, TAG_BULK, wv);
            bulk[2 * r] = u01(wv[0]); bulk[2 * r + 1] = u01(wv[1]);
        }
    }
}

// Share of a replica's work list, cut over its particle workgroups
struct Share {
    int64_t me, all;
    __device__ int64_t lo(int64_t n) const { return n * me / all; }
    __device__ int64_t hi(int64_t n) const { return n * (me + 1) / all; }
};

// Streaming of the particles outside the Verlet list (flows: of all) over the
// interval, their cells in the coming collision and their ranks in them (any
// order: the collision restores the stable one), with one returning atomic per
// run of equal keys in a wave.  Workgroup `sub` of a chunk covers particles
// [sub*span, (sub+1)*span) of it, span = blockDim.x * PPT; thread t holds
// particles t, t + blockDim.x, ... of its span: every load is issued before
// the drifts, every rank atomic before the first of them is waited for.  The
// atomics all go to memory, so this kernel keeps many waves (in the
// collision, at four waves per SIMD, their latency and the drifts showed in
// full).  A list member's record, which the MD chain on the side stream may be
// writing meanwhile, is loaded and not used but for the list bit, which stays
// set.  The replica's workgroups share its cells for the collision's draws.
// A wave reads and writes its 64 records through LDS so that each instruction
// covers a contiguous kilobyte (one lane a record: 783 us where this takes
// 706, 20.97 M particles in FP64; FP32 489).  Those 2.2 GB need 414 us at the
// rate of a copy; the rest is the rank atomics (a trial without them 450).
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
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const int64_t i0 = base + u * (int)blockDim.x + (threadIdx.x & ~63u);
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
        go[u] = i < n && (st[u] & ST_LIST) == 0u;
    }
    const double s[3] = {uniform_d(G(rs)->shift[0]), uniform_d(G(rs)->shift[1]), uniform_d(G(rs)->shift[2])};
    advance<T, PPT, FLOW>(D, x, v, go);
    uint32_t key[PPT];
    RankIssue ri[PPT];
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        key[u] = go[u] ? cell_key<FLOW>(D, (double)x[u][0], (double)x[u][1], (double)x[u][2], s) : 0u;
        ri[u] = wave_rank_issue(G(D.count), key[u], go[u]);
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
    const Share sh{(int64_t)chunk * wg_per_chunk + sub, (int64_t)D.n_chunks * wg_per_chunk};
    for (int role = threadIdx.x >> 6; role < 2; role += (int)(blockDim.x >> 6))
        collision_draws(D, role, sh.lo(D.ncell), sh.hi(D.ncell));
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const int64_t i = base + u * (int)blockDim.x + threadIdx.x;
        const uint32_t rank = wave_rank_finish(ri[u]);
        if (go[u]) G(D.keyrank)[i] = ((uint64_t)key[u] << 32) | rank;
    }
}

}  // namespace rmp
