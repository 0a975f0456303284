// kernels_small.hpp -- the coarse end of the V-cycle in one workgroup.
//
// All levels from the first one of at most 8 x 8 x 8 blocks of 2 x 2 x 2
// vertices (16^3 cells) down to the coarsest run inside a single workgroup;
// the coarsest level is solved exactly in float64 by a product with the
// inverse of its operator (formed once per coefficient set).  Levels may
// have different cell counts and spacings per axis.
//
// What bounds it: a chain of about 60 dependent steps on one CU, where the
// first level's half-sweeps are bound by that CU's arithmetic (512 threads
// of about 50 instructions, 400 cycles) and every other step by the latency
// of an LDS read.  Three choices keep the steps few and short:
//
//  - A thread owns a block of 2 x 2 x 2 vertices (Block3).  A half-sweep is
//    12 LDS reads, 28 multiply-adds and a barrier.  (With D, w and q read
//    from LDS as well, two vertices a thread, it took three times as long.)
//  - A coarse vertex 2X is the corner of block X, so the thread that owns the
//    block also restricts to X and prolongs from X .. X+1: no other index map.
//  - Every level below the first has at most 64 blocks and belongs to one
//    wave of its own (waves 8 and 9), whose steps need no barrier at all and
//    whose coefficients are in registers when the first level gets there.
//
// After a red-black sweep the residual of the colour updated last is zero
// (its update solved its own equations), so only the other colour's is
// formed and restricted.
//
// From the first level of at most 64 unknowns down the whole cycle is linear
// in its right-hand side: one matrix, formed once per coefficient set
// (k_small_cols), and one product per call (15 -> 12.6 us).
//
// Measured, 16^3 .. 2^3 levels, V(2,2): float32 25 -> 12.6 us per call,
// float64 15.3 us, where the 16^3 level took three launches of its own (pass,
// restriction, pass: 42 us) before an 11 us call for the levels below it;
// of a 12^3 level the same cost 12 launches of one operation each.  As the
// last workgroup of the restricting pass over 32^3 (BlockTailArgs), which
// hides its loads: 16.8 and 18.6 us for both.
#pragma once
#include "grid.hpp"
#include "kernels_basic.hpp"
#include "kernels_block.hpp"

namespace dmgs {

constexpr int kSmallMaxLevels = 4;      // levels of one call, the exactly solved one among them
constexpr int kSmallTop = 512;          // most blocks of the first level, one per thread of waves 0 .. 7
constexpr int kSmallThreads = kSmallTop + 64 * (kSmallMaxLevels - 2);
constexpr int kSmallCoarseMax = 64;     // most unknowns of the coarsest level

template <class T>
struct SmallLevel {
    int nc[3];     // cells per axis
    const T* D;    // level coefficient arrays, (nc+1) vertices per axis, z fastest
    const T* w;    // inverse diagonal (0 on the boundary), or mua (SmallArgs::from_mu)
    T s[3];        // per axis: 1 / (2 h^2) (arithmetic face mean) or 2 / h^2 (harmonic)
};

template <class T>
struct SmallArgs {
    int nlev;                          // levels handled (first small level .. coarsest)
    SmallLevel<T> lev[kSmallMaxLevels];
    const T* q;                        // right-hand side on the first small level
    T* u;                              // result on the first small level (boundary layer not written)
    const double* cinv;                // the last level's solution operator (m x m, row-major): the coarsest
                                       // operator's inverse, or the matrix of the cycle below it
    int ctrans;                        // apply its transpose
    int nu_pre, nu_post, order;
    int from_mu;                       // lev[].w holds mua: the inverse diagonal is formed here
};

// LDS layout of a level: octant o = 4 (x&1) + 2 (y&1) + (z&1) of block
// (x>>1, y>>1, z>>1) at off + o kSmallS + bx kSmallX + by kSmallY + bz.  The
// strides are those of the largest first level and the same for every level,
// so that all 24 neighbour addresses of a block are one register and
// instruction offsets; the 64 blocks of a wave are 64 consecutive words (a
// pitch of 9 instead of 8 put every second read in a two-way bank conflict).
// The vertex past a row's or plane's last block is on the boundary, and so
// is what lies there: an unused entry, or with 8 blocks the first vertex of
// the next row or plane.  Along x a plane of zeros follows.  The coarser
// levels share one more set of octants, each in a corner of it that the
// others leave free.
constexpr int kSmallNb = 8;                  // most blocks per axis (first level; half as many on the next, ...)
constexpr int kSmallY = kSmallNb, kSmallX = kSmallY * kSmallNb, kSmallS = kSmallX * (kSmallNb + 1);
constexpr int kSmallWords = 2 * 8 * kSmallS;
__host__ __device__ constexpr int small_off(int level) {
    return level == 0 ? 0 : 8 * kSmallS + (level == 1 ? 0 : 5 * kSmallX + (level == 2 ? 0 : 4 * kSmallY));
}
__device__ __forceinline__ int small_at(int off, int x, int y, int z) {
    return off + ((x & 1) * 4 + (y & 1) * 2 + (z & 1)) * kSmallS + (x >> 1) * kSmallX + (y >> 1) * kSmallY + (z >> 1);
}

template <class T>
constexpr size_t small_lds_bytes() {
    return kSmallWords * sizeof(T) + (kSmallCoarseMax + 1) * kSmallCoarseMax * sizeof(double);
}

// Whether levels nc[0 .. nlev-1] (cells per axis) fit the kernel.
inline bool small_fits(const int (*nc)[3], int nlev) {
    if (nlev < 1 || nlev > kSmallMaxLevels) return false;
    int64_t m = 1;
    for (int a = 0; a < 3; a++) {
        for (int i = 0; i < nlev; i++)
            if (nc[i][a] < 2 || nc[i][a] > (2 * kSmallNb >> i) || (i > 0 && nc[i - 1][a] != 2 * nc[i][a])) return false;
        m *= nc[nlev - 1][a] - 1;
    }
    return m <= kSmallCoarseMax;
}

// Order this wave's LDS operations among its lanes (they execute in order;
// the fences only stop the compiler from moving them).
__device__ __forceinline__ void small_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// How a call gets its right-hand side and where its result goes.
//   kSmallPlain  a.q, a.u
//   kSmallTail   the same as the last workgroup of the launch that restricts
//                to a.q: loads the coefficients first, then waits for the
//                count of finished workgroups at `done` to reach `need`
//                (small_wait; when that gives up the result is NaN)
//   kSmallCols   workgroup j solves for unit vector j of the first level's
//                unknowns and writes column j of the cycle's matrix (m x m,
//                row-major) to `mat`
enum SmallMode { kSmallPlain = 0, kSmallTail = 1, kSmallCols = 2 };

// The wait of a launch's last workgroup (grouped: of each member's) for the
// `need` workgroups before it, which wait for nothing.  An XCD takes a launch's
// workgroups in order, so on the waiter's own XCD they were dispatched before
// it, and elsewhere they wait at most for CUs: those of work that ends, or of
// other waiters.  A launch has at most kGroupMax waiters, one a CU; only if
// waiters held every CU of two XCDs (64) could launches hold each other up.
// So the wait is bounded: after `spins` looks (seconds, where the others take
// microseconds) it marks the count, so that the plan's later launches do not
// wait either, and returns false; the result is then NaN, which tolerance
// solves report as a non-finite residual.  Otherwise the count is back at 0
// when the launch ends.
constexpr unsigned kTailSpins = 1u << 22, kTailGaveUp = 1u << 31;
__device__ __forceinline__ bool small_wait(unsigned* done, unsigned need, unsigned spins) {
    __shared__ bool met;
    if (threadIdx.x == 0) {
        unsigned seen = 0;   // need, or kTailGaveUp and more
        for (unsigned i = 0; i < spins && seen < need; i++) {
            if (i > 0) __builtin_amdgcn_s_sleep(1);
            seen = __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        met = seen == need;
        if (met) __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else __hip_atomic_fetch_or(done, kTailGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return met;
}
// ... and what the other workgroups do once their stores are issued: the
// restricted values are stored past the caches (block3_body with COHERENT),
// so each wave only waits for its own stores to complete.
__device__ __forceinline__ void small_arrive(unsigned* done) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

template <class T, bool HARM, int MODE, int NT = kSmallThreads>
__device__ __forceinline__ void small_vcycle_body(const SmallArgs<T>& a, unsigned* done = nullptr, unsigned need = 0,
                                                  unsigned spins = 0, double* mat = nullptr) {
    extern __shared__ __align__(16) unsigned char block_smem[];
    T* const base = reinterpret_cast<T*>(block_smem);
    const int tid = threadIdx.x, L = a.nlev;
    const int first = a.order ? 1 : 0;       // colour of the first half-sweep
    // this wave's level: 0 for waves 0 .. 7, 1 and 2 for waves 8 and 9
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ml = wave < kSmallTop / 64 ? 0 : wave - kSmallTop / 64 + 1;
    const bool mine = ml < L - 1;             // a smoothed level
    const SmallLevel<T>& lv = a.lev[mine ? ml : 0];
    const int nb0 = lv.nc[0] / 2, nb1 = lv.nc[1] / 2, nb2 = lv.nc[2] / 2;   // blocks per axis
    // blocks on the lanes of 8 x 8 x 8 (level 0) or 4 x 4 x 4 (one wave)
    const int sb = ml == 0 ? 3 : 2, mb = (1 << sb) - 1;
    const int bz = tid & mb, by = (tid >> sb) & mb, bx = (tid >> (2 * sb)) & mb;
    const bool act = mine && bx < nb0 && by < nb1 && bz < nb2;
    using B3 = Block3<T, kSmallS, kSmallX, kSmallY>;
    constexpr int S = kSmallS;
    const int idx = small_off(ml) + bx * kSmallX + by * kSmallY + bz;     // own octant o: base[idx + o S]
    // the coarsest operator's inverse (transposed)
    double* const sinv = reinterpret_cast<double*>(block_smem + kSmallWords * sizeof(T));
    const int cx = a.lev[L - 1].nc[0] - 1, cy = a.lev[L - 1].nc[1] - 1, cz = a.lev[L - 1].nc[2] - 1;
    const int m = cx * cy * cz;
    if (MODE != kSmallCols && L == 1) {   // nothing to smooth: u = A^-1 q straight from memory
        const bool met = MODE != kSmallTail || small_wait(done, need, spins);
        if (tid < m) {
            const int n1 = cy + 2, n2 = cz + 2;
            auto gid = [&](int c) { return ((1 + c / (cy * cz)) * n1 + 1 + (c / cz) % cy) * n2 + 1 + c % cz; };
            double acc = met ? 0.0 : __builtin_nan("");
            for (int c = 0; c < m; c++) acc += a.cinv[a.ctrans ? c * m + tid : tid * m + c] *
                       (double)__hip_atomic_load(a.q + gid(c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            a.u[gid(tid)] = (T)acc;
        }
        return;
    }

    B3 P;   // the block's state

    // own D, w and q; own D and the D past the end of each axis to the
    // octants, the neighbours' D from them; the coarsest inverse
    const int n1 = lv.nc[1] + 1, n2 = lv.nc[2] + 1;
    const int v0 = ((2 * bx) * n1 + 2 * by) * n2 + 2 * bz;   // the corner
    auto vert = [&](int o) { return v0 + (o >> 2) * n1 * n2 + ((o >> 1) & 1) * n2 + (o & 1); };
    const int ev[3] = {n1 * n2, n2, 1};
    const bool edge[3] = {act && bx == nb0 - 1, act && by == nb1 - 1, act && bz == nb2 - 1};
    struct Pair {   // two vertices along z, aligned as one
        T a, b;
    };
    auto load = [&](const T* p, bool on, T none, T* v) {
#pragma unroll
        for (int o = 0; o < 8; o += 2) {
            const Pair t = on ? *reinterpret_cast<const Pair*>(p + vert(o)) : Pair{none, none};
            v[o] = t.a;
            v[o + 1] = t.b;
        }
    };
    {
        // every global load before the first use of one
        T D[8], De[3][4];
        load(lv.D, act, T(1), D);
        load(lv.w, act, T(0), P.w);
        if (MODE == kSmallPlain) load(a.q, act && ml == 0, T(0), P.q);
#pragma unroll
        for (int ax = 0; ax < 3; ax++)
#pragma unroll
            for (int o = 0; o < 8; o++)
                if (o & B3::bit(ax)) De[ax][B3::inner(ax, o)] = edge[ax] ? lv.D[vert(o) + ev[ax]] : T(0);
        for (int i = tid; i < kSmallWords; i += NT) base[i] = T(0);
        for (int i = tid; i < m * m; i += NT) sinv[a.ctrans ? i : (i % m) * m + i / m] = a.cinv[i];
        __syncthreads();
#pragma unroll
        for (int ax = 0; ax < 3; ax++)
#pragma unroll
            for (int o = 0; o < 8; o++)
                if ((o & B3::bit(ax)) && edge[ax]) base[idx + B3::outer(ax, o)] = De[ax][B3::inner(ax, o)];
        // the D of the low y and z faces is nobody's neighbour but boundary
        // vertices' (their entries may be an edge's)
#pragma unroll
        for (int o = 0; o < 8; o++)
            if (act && (by > 0 || (o & 2)) && (bz > 0 || (o & 1))) base[idx + o * S] = D[o];
        __syncthreads();
        P.template coefs<HARM>(base, idx, D, lv.s);
        if (a.from_mu) {
#pragma unroll
            for (int o = 0; o < 8; o++) {
                const bool in = act && (bx > 0 || (o & 4)) && (by > 0 || (o & 2)) && (bz > 0 || (o & 1));
                P.w[o] = in ? T(1) / P.diag(o, P.w[o]) : T(0);
            }
        }
    }
    __syncthreads();
    // the vertices past the end are boundary: 0 from here on
#pragma unroll
    for (int ax = 0; ax < 3; ax++)
#pragma unroll
        for (int o = 0; o < 8; o++)
            if ((o & B3::bit(ax)) && edge[ax]) base[idx + B3::outer(ax, o)] = T(0);

    if (MODE == kSmallTail) {
        const bool met = small_wait(done, need, spins);
#pragma unroll
        for (int o = 0; o < 8; o++) {
            P.q[o] = act && ml == 0 ? __hip_atomic_load(a.q + vert(o), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : T(0);
            P.q[o] = met ? P.q[o] : T(__builtin_nan(""));
        }
    } else if (MODE == kSmallCols) {
        // unknowns of the first level in x, y, z order
#pragma unroll
        for (int o = 0; o < 8; o++) {
            const int x = 2 * bx + (o >> 2), y = 2 * by + ((o >> 1) & 1), z = 2 * bz + (o & 1);
            const int id = ((x - 1) * (lv.nc[1] - 1) + y - 1) * (lv.nc[2] - 1) + z - 1;
            P.q[o] = ml == 0 && P.w[o] != T(0) && id == (int)blockIdx.x ? T(1) : T(0);
        }
    }

    auto half_of = [&](int c) {
        if (c) P.template half<1, false>(base, idx);
        else P.template half<0, false>(base, idx);
    };
    // level 0 is shared by waves 0 .. 7: its steps end with a workgroup
    // barrier, which every wave joins; the other levels are one wave's
    auto sync = [&](int l) {
        if (l == 0) __syncthreads();
        else if (ml == l) small_wave_sync();
    };
    auto sweeps = [&](int l, int count, bool skip1) {
        const bool run = ml == l && act;
        for (int c = 0; c < 2 * count; c++) {
            if (skip1 && c == 0) continue;
            if (run) half_of((c & 1) ? 1 - first : first);
            sync(l);
        }
    };

    for (int l = 0; l < L - 1; l++) {   // down: every level starts from a zero iterate
        const bool run = ml == l && act;
        if (run) {
            // right-hand side; from zero the first half-sweep is u = w q on
            // the first colour
#pragma unroll
            for (int o = 0; o < 8; o++) {
                if (l > 0) P.q[o] = base[idx + o * S];
                P.u[o] = (a.nu_pre > 0 && B3::colour(o) == first) ? P.w[o] * P.q[o] : T(0);
            }
            B3::publish(base, idx, P.u);
        }
        sync(l);
        sweeps(l, a.nu_pre, true);
        // defect of the first colour, 0 for the other (of both when nothing
        // was smoothed: there it is q), 0 on the boundary (w = 0)
        T r[8] = {};
        if (run) {
            if (a.nu_pre == 0) {
#pragma unroll
                for (int o = 0; o < 8; o++) r[o] = P.w[o] == T(0) ? T(0) : P.q[o];
            } else if (first) {
                P.template residual<1>(base, idx, r);
            } else {
                P.template residual<0>(base, idx, r);
            }
        }
        sync(l);
        if (run) B3::publish(base, idx, r);
        sync(l);
        // restriction to the corner X = (bx, by, bz), interior: octant o
        // of block X and, where its bit is set, of the block before
        if (run && bx > 0 && by > 0 && bz > 0) {
            T s = first ? B3::template weighted<1>(base, idx) : B3::template weighted<0>(base, idx);
            if (a.nu_pre == 0) s += first ? B3::template weighted<0>(base, idx) : B3::template weighted<1>(base, idx);
            base[small_at(small_off(l + 1), bx, by, bz)] = s * T(1.0 / 64.0);
        }
        __syncthreads();
    }
    if (wave == 0) {   // the last level: u = C q on the interior unknowns (x, y, z order), one a lane
        const int at = small_at(small_off(L - 1), 1 + tid / (cy * cz), 1 + (tid / cz) % cy, 1 + tid % cz);
        double* const sq = sinv + kSmallCoarseMax * kSmallCoarseMax;
        if (tid < m) sq[tid] = (double)base[at];
        small_wave_sync();
        if (tid < m) {
            double acc = 0.0;
#pragma unroll 8
            for (int c = 0; c < m; c++) acc += sinv[c * m + tid] * sq[c];
            base[at] = (T)acc;
        }
    }
    __syncthreads();
    for (int l = L - 2; l >= 0; l--) {  // up
        const bool run = ml == l && act;
        if (run) {
            // trilinear correction from X .. X+1; the next half-sweep reads
            // the second colour only, with no post-smoothing both are published
            T E[8];
#pragma unroll
            for (int o = 0; o < 8; o++) E[o] = base[small_at(small_off(l + 1), bx + (o >> 2), by + ((o >> 1) & 1), bz + (o & 1))];
#pragma unroll
            for (int o = 0; o < 8; o++)
                if (P.w[o] != T(0)) P.u[o] += B3::corrected(E, o);
            B3::publish(base, idx, P.u);
        }
        sync(l);
        sweeps(l, a.nu_post, false);
        if (l > 0) __syncthreads();   // the finer level's waves read the result
    }
    if (ml == 0 && act) {
#pragma unroll
        for (int o = 0; o < 8; o++) {
            if (P.w[o] == T(0)) continue;   // boundary entries stay 0
            if (MODE == kSmallCols) {
                const int x = 2 * bx + (o >> 2), y = 2 * by + ((o >> 1) & 1), z = 2 * bz + (o & 1);
                const int id = ((x - 1) * (lv.nc[1] - 1) + y - 1) * (lv.nc[2] - 1) + z - 1;
                mat[(int64_t)id * gridDim.x + blockIdx.x] = (double)P.u[o];
            } else {
                a.u[vert(o)] = P.u[o];
            }
        }
    }
}

template <class T, bool HARM>
__global__ __launch_bounds__(kSmallThreads) void k_small_vcycle(SmallArgs<T> a) {
    small_vcycle_body<T, HARM, kSmallPlain>(a);
}

// The matrix of the cycle from a level of at most kSmallCoarseMax unknowns
// down (once per coefficient set): the cycle is linear and starts from zero,
// so that level and everything below it is one product with this matrix (and
// the transposed cycle's with its transpose).  A level of 4^3 and the 2^3
// below it took 40 % of the chain of steps for 28 unknowns.
template <class T, bool HARM>
__global__ __launch_bounds__(kSmallThreads) void k_small_cols(SmallArgs<T> a, double* mat) {
    small_vcycle_body<T, HARM, kSmallCols>(a, nullptr, 0, 0, mat);
}

// Grouped form: one workgroup per member.
template <class T, bool HARM>
__global__ __launch_bounds__(kSmallThreads) void k_small_grp(const Group<SmallArgs<T>>* g) {
    int bid;
    const int m = group_member(g, &bid);
    if (bid < 0) return;
    small_vcycle_body<T, HARM, kSmallPlain>(g->a[m]);
}

// The block pass that restricts to the coarse kernel's first level, with that
// kernel as the launch's last workgroup: its coefficients are loaded while the
// others work, and the gap between two launches is gone.
template <class T>
struct BlockTailArgs {
    Block3Args<T> b;
    SmallArgs<T> s;
    unsigned* done;   // 0 between launches
    int nb;           // workgroups of the block pass
    unsigned spins;   // bound of the last workgroup's wait
};

template <int MODE, bool GEN>
constexpr int block_tail_threads() {
    return Block3Shape<MODE, GEN>::NT > kSmallThreads ? Block3Shape<MODE, GEN>::NT : kSmallThreads;
}
template <class T, int MODE, bool GEN>
constexpr size_t block_tail_lds() {
    return block3_lds<T, MODE, GEN>() > small_lds_bytes<T>() ? block3_lds<T, MODE, GEN>() : small_lds_bytes<T>();
}

template <class T, int MODE, bool HARM, bool GEN>
__device__ __forceinline__ void block_tail_body(const BlockTailArgs<T>& a, int bid) {
    if (bid < a.nb) {
        block3_body<T, MODE, HARM, GEN, true>(a.b, bid);
        small_arrive(a.done);
    } else {
        small_vcycle_body<T, HARM, kSmallTail, block_tail_threads<MODE, GEN>()>(a.s, a.done, (unsigned)a.nb, a.spins);
    }
}

template <class T, int MODE, bool HARM, bool GEN>
__global__ __launch_bounds__((block_tail_threads<MODE, GEN>())) void k_block_tail(BlockTailArgs<T> a) {
    block_tail_body<T, MODE, HARM, GEN>(a, blockIdx.x);
}

template <class T, int MODE, bool HARM>
__global__ __launch_bounds__((block_tail_threads<MODE, false>())) void k_block_tail_grp(const Group<BlockTailArgs<T>>* g) {
    int bid;
    const int m = group_member(g, &bid);
    if (bid < 0) return;
    block_tail_body<T, MODE, HARM, false>(g->a[m], bid);
}

}  // namespace dmgs
