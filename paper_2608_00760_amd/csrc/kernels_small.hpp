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
//  - A thread owns a block of 2 x 2 x 2 vertices (even corner) and keeps
//    their iterate, right-hand side, inverse diagonal and all 36 face
//    coefficients in registers.  Half of every vertex's neighbours are then
//    the thread's own; the others are read from LDS, three per update, where
//    the iterate lies by octant (position in the block) so that the lanes of
//    a wave read consecutive words.  A half-sweep is 12 LDS reads, 28
//    multiply-adds and a barrier.  (With D, w and q read from LDS as well,
//    two vertices a thread, a half-sweep took three times as long.)
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
// Measured, 16^3 .. 2^3 levels, V(2,2): float32 25 -> 15 us per call,
// float64 18 us, where the 16^3 level took three launches of its own (pass,
// restriction, pass: 42 us) before an 11 us call for the levels below it;
// of a 12^3 level the same cost 12 launches of one operation each.
#pragma once
#include "grid.hpp"
#include "kernels_basic.hpp"

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
    const double* cinv;                // inverse of the coarsest operator (m x m)
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
    return kSmallWords * sizeof(T) + kSmallCoarseMax * kSmallCoarseMax * sizeof(double);
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

template <class T, bool HARM>
__device__ __forceinline__ void small_vcycle_body(const SmallArgs<T>& a) {
    extern __shared__ __align__(16) unsigned char small_smem[];
    T* const base = reinterpret_cast<T*>(small_smem);
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
    constexpr int S = kSmallS, stepB[3] = {kSmallX, kSmallY, 1};         // to the next octant; block per axis
    const int idx = small_off(ml) + bx * kSmallX + by * kSmallY + bz;     // own octant o: base[idx + o S]
    // the coarsest operator's inverse (transposed)
    double* const sinv = reinterpret_cast<double*>(small_smem + kSmallWords * sizeof(T));
    const int cx = a.lev[L - 1].nc[0] - 1, cy = a.lev[L - 1].nc[1] - 1, cz = a.lev[L - 1].nc[2] - 1;
    const int m = cx * cy * cz;
    if (L == 1) {   // nothing to smooth: u = A^-1 q straight from memory
        if (tid < m) {
            const int n1 = cy + 2, n2 = cz + 2;
            auto gid = [&](int c) { return ((1 + c / (cy * cz)) * n1 + 1 + (c / cz) % cy) * n2 + 1 + c % cz; };
            double acc = 0.0;
            for (int c = 0; c < m; c++) acc += a.cinv[tid * m + c] * (double)a.q[gid(c)];
            a.u[gid(tid)] = (T)acc;
        }
        return;
    }

    // state of the block: octant o has bit 2 for x, 1 for y, 0 for z
    T u[8], q[8], w[8];
    T ci[3][4];    // faces inside the block per axis, by the other two bits
    T co[3][8];    // faces to the neighbouring blocks, by octant
    auto inner = [](int ax, int o) { return ax == 0 ? o & 3 : ax == 1 ? (o >> 2) * 2 + (o & 1) : o >> 1; };
    constexpr int bitOf[3] = {4, 2, 1};

    // own D, w and q; own D and the D past the end of each axis to the
    // octants, the neighbours' D from them; the coarsest inverse
    const int n1 = lv.nc[1] + 1, n2 = lv.nc[2] + 1;
    const int v0 = ((2 * bx) * n1 + 2 * by) * n2 + 2 * bz;   // the corner
    auto vert = [&](int o) { return v0 + (o >> 2) * n1 * n2 + ((o >> 1) & 1) * n2 + (o & 1); };
    const int ev[3] = {n1 * n2, n2, 1};
    const bool edge[3] = {act && bx == nb0 - 1, act && by == nb1 - 1, act && bz == nb2 - 1};
    {
        // every global load before the first use of one
        T D[8], De[3][4];
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
        load(lv.D, act, T(1), D);
        load(lv.w, act, T(0), w);
        load(a.q, act && ml == 0, T(0), q);
#pragma unroll
        for (int ax = 0; ax < 3; ax++)
#pragma unroll
            for (int o = 0; o < 8; o++)
                if (o & bitOf[ax]) De[ax][inner(ax, o)] = edge[ax] ? lv.D[vert(o) + ev[ax]] : T(0);
        for (int i = tid; i < kSmallWords; i += kSmallThreads) base[i] = T(0);
        for (int i = tid; i < m * m; i += kSmallThreads) sinv[(i % m) * m + i / m] = a.cinv[i];
        __syncthreads();
#pragma unroll
        for (int ax = 0; ax < 3; ax++)
#pragma unroll
            for (int o = 0; o < 8; o++)
                if ((o & bitOf[ax]) && edge[ax]) base[idx + (o ^ bitOf[ax]) * S + stepB[ax]] = De[ax][inner(ax, o)];
        // the D of the low y and z faces is nobody's neighbour but boundary
        // vertices' (their entries may be an edge's)
#pragma unroll
        for (int o = 0; o < 8; o++)
            if (act && (by > 0 || (o & 2)) && (bz > 0 || (o & 1))) base[idx + o * S] = D[o];
        __syncthreads();
        auto fc = [&](int ax, T Da, T Db) -> T {
            if (HARM) return (Da * Db) / (Da + Db) * lv.s[ax];
            return (Da + Db) * lv.s[ax];
        };
#pragma unroll
        for (int ax = 0; ax < 3; ax++)
#pragma unroll
            for (int o = 0; o < 8; o++) {
                const int p = o ^ bitOf[ax];
                const int j = idx + p * S + ((o & bitOf[ax]) ? stepB[ax] : -stepB[ax]);
                co[ax][o] = fc(ax, D[o], act ? base[j] : T(0));
                if (!(o & bitOf[ax])) ci[ax][inner(ax, o)] = fc(ax, D[o], D[p]);
            }
        if (a.from_mu) {
#pragma unroll
            for (int o = 0; o < 8; o++) {
                T d = w[o];
#pragma unroll
                for (int ax = 0; ax < 3; ax++) d += ci[ax][inner(ax, o)] + co[ax][o];
                const bool in = (bx > 0 || (o & 4)) && (by > 0 || (o & 2)) && (bz > 0 || (o & 1));
                w[o] = in && act ? T(1) / d : T(0);
            }
        }
    }
    __syncthreads();
    // the vertices past the end are boundary: 0 from here on
#pragma unroll
    for (int ax = 0; ax < 3; ax++)
#pragma unroll
        for (int o = 0; o < 8; o++)
            if ((o & bitOf[ax]) && edge[ax]) base[idx + (o ^ bitOf[ax]) * S + stepB[ax]] = T(0);

    // q + sum_j c_ij u_j at the octants of one colour (the Gauss-Seidel value
    // is w times it); a colour's octants have one bit parity (the corner's
    // coordinates are even).  All LDS reads are issued before the first is
    // used: left to itself the compiler interleaves them with the sums and
    // waits for the LDS four times over.
    auto numer = [&](auto Cc, T* s) {
        constexpr int C = decltype(Cc)::value;
        T nb[8][3];
#pragma unroll
        for (int o = 0; o < 8; o++)
            if ((__builtin_popcount(o) & 1) == C)
#pragma unroll
                for (int ax = 0; ax < 3; ax++)
                    nb[o][ax] = base[idx + (o ^ bitOf[ax]) * S + ((o & bitOf[ax]) ? stepB[ax] : -stepB[ax])];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int o = 0; o < 8; o++)
            if ((__builtin_popcount(o) & 1) == C) {
                s[o] = q[o];
#pragma unroll
                for (int ax = 0; ax < 3; ax++) s[o] += ci[ax][inner(ax, o)] * u[o ^ bitOf[ax]];
#pragma unroll
                for (int ax = 0; ax < 3; ax++) s[o] += co[ax][o] * nb[o][ax];
            }
    };
    auto half = [&](auto Cc) {
        constexpr int C = decltype(Cc)::value;
        T v[8];
        numer(Cc, v);
#pragma unroll
        for (int o = 0; o < 8; o++)
            if ((__builtin_popcount(o) & 1) == C) {
                u[o] = v[o] * w[o];
                base[idx + o * S] = u[o];
            }
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    auto half_of = [&](int c) {
        if (c) half(C1());
        else half(C0());
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
                if (l > 0) q[o] = base[idx + o * S];
                u[o] = (a.nu_pre > 0 && (__builtin_popcount(o) & 1) == first) ? w[o] * q[o] : T(0);
            }
#pragma unroll
            for (int o = 0; o < 8; o++) base[idx + o * S] = u[o];
        }
        sync(l);
        sweeps(l, a.nu_pre, true);
        // defect of the first colour, 0 for the other (of both when nothing
        // was smoothed: there it is q), 0 on the boundary (w = 0)
        auto defect = [&](auto Cc) {
            constexpr int C = decltype(Cc)::value;
            T r[8] = {};
            if (run) {
                numer(Cc, r);
#pragma unroll
                for (int o = 0; o < 8; o++)
                    if ((__builtin_popcount(o) & 1) == C) r[o] = w[o] == T(0) ? T(0) : r[o] - u[o] / w[o];
            }
            sync(l);
            if (run) {
#pragma unroll
                for (int o = 0; o < 8; o++) base[idx + o * S] = r[o];
            }
        };
        if (a.nu_pre == 0) {
            sync(l);
            if (run) {
#pragma unroll
                for (int o = 0; o < 8; o++) base[idx + o * S] = w[o] == T(0) ? T(0) : q[o];
            }
        } else if (first) {
            defect(C1());
        } else {
            defect(C0());
        }
        sync(l);
        // restriction to the corner X = (bx, by, bz), interior: octant o
        // of block X and, where its bit is set, of the block before
        if (run && bx > 0 && by > 0 && bz > 0) {
            auto sum = [&](auto Cc) -> T {   // over the octants of one colour
                constexpr int C = decltype(Cc)::value;
                T v[8][8], s = T(0);
#pragma unroll
                for (int o = 0; o < 8; o++)
#pragma unroll
                    for (int k = 0; k < 8; k++)
                        if ((__builtin_popcount(o) & 1) == C && !(k & ~o))
                            v[o][k] = base[idx + o * S - ((k & 4) ? stepB[0] : 0) - ((k & 2) ? stepB[1] : 0) -
                                           ((k & 1) ? stepB[2] : 0)];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int o = 0; o < 8; o++) {
                    T t = T(0);
#pragma unroll
                    for (int k = 0; k < 8; k++)
                        if ((__builtin_popcount(o) & 1) == C && !(k & ~o)) t += v[o][k];
                    if ((__builtin_popcount(o) & 1) == C) s += t * T(8 >> __builtin_popcount(o));
                }
                return s;
            };
            T s = first ? sum(C1()) : sum(C0());
            if (a.nu_pre == 0) s += first ? sum(C0()) : sum(C1());
            base[small_at(small_off(l + 1), bx, by, bz)] = s * T(1.0 / 64.0);
        }
        __syncthreads();
    }
    if (tid < m) {   // coarsest level: u = A^-1 q on the interior unknowns (x, y, z order)
        auto vid = [&](int c) { return small_at(small_off(L - 1), 1 + c / (cy * cz), 1 + (c / cz) % cy, 1 + c % cz); };
        double acc = 0.0;
        for (int c = 0; c < m; c++) acc += sinv[c * m + tid] * (double)base[vid(c)];
        small_wave_sync();
        base[vid(tid)] = (T)acc;
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
            for (int o = 0; o < 8; o++) {
                T s = T(0);
#pragma unroll
                for (int k = 0; k < 8; k++)
                    if (!(k & ~o)) s += E[k];
                if (w[o] != T(0)) u[o] += s * T(1.0 / (1 << __builtin_popcount(o)));
            }
#pragma unroll
            for (int o = 0; o < 8; o++) base[idx + o * S] = u[o];
        }
        sync(l);
        sweeps(l, a.nu_post, false);
        if (l > 0) __syncthreads();   // the finer level's waves read the result
    }
    if (ml == 0 && act) {
#pragma unroll
        for (int o = 0; o < 8; o++)
            if (w[o] != T(0)) a.u[vert(o)] = u[o];   // boundary entries stay 0
    }
}

template <class T, bool HARM>
__global__ __launch_bounds__(kSmallThreads) void k_small_vcycle(SmallArgs<T> a) {
    small_vcycle_body<T, HARM>(a);
}

// Grouped form: one workgroup per member.
template <class T, bool HARM>
__global__ __launch_bounds__(kSmallThreads) void k_small_grp(const Group<SmallArgs<T>>* g) {
    int bid;
    const int m = group_member(g, &bid);
    if (bid < 0) return;
    small_vcycle_body<T, HARM>(g->a[m]);
}

}  // namespace dmgs
