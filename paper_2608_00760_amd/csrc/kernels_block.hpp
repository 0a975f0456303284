// kernels_block.hpp -- smoothing phases in register blocks of 2 x 2 x 2
// vertices: the block itself (also the coarse kernel's), and whole phases of
// a mid-size level in one launch.
#pragma once
#include <type_traits>

#include "kernels_stream.hpp"

namespace dmgs {

// A thread owns the block with even corner (2 bx, 2 by, 2 bz): octant o =
// 4 (x&1) + 2 (y&1) + (z&1).  Iterate, right-hand side, inverse diagonal and
// all 36 face coefficients stay in registers for a whole phase; half of every
// vertex's neighbours are the thread's own, the other three are read from
// LDS, where the iterate lies by octant (base[idx + o S], X and Y to the next
// block along x and y, 1 along z) so that consecutive lanes read consecutive
// words.  A vertex's colour is its octant's bit parity.  Vertices that must
// not change (grid boundary, outside) have w = 0.
template <class T, int S, int X, int Y>
struct Block3 {
    T u[8], q[8], w[8];
    T ci[3][4];    // faces inside the block per axis, by the other two bits
    T co[3][8];    // faces to the neighbouring blocks, by octant

    __device__ static constexpr int bit(int ax) { return 4 >> ax; }
    __device__ static constexpr int step(int ax) { return ax == 0 ? X : ax == 1 ? Y : 1; }
    __device__ static constexpr int inner(int ax, int o) {
        return ax == 0 ? o & 3 : ax == 1 ? (o >> 2) * 2 + (o & 1) : o >> 1;
    }
    __device__ static constexpr int colour(int o) { return __builtin_popcount(o) & 1; }
    // LDS entry, from idx, of octant o's neighbour outside the block along ax
    __device__ static constexpr int outer(int ax, int o) { return (o ^ bit(ax)) * S + ((o & bit(ax)) ? step(ax) : -step(ax)); }

    __device__ __forceinline__ static void publish(T* base, int idx, const T* v) {
#pragma unroll
        for (int o = 0; o < 8; o++) base[idx + o * S] = v[o];
    }
    // face coefficients from the block's D and its neighbours' (published);
    // s: 1 / (2 h^2) per axis (arithmetic face mean) or 2 / h^2 (harmonic)
    template <bool HARM>
    __device__ __forceinline__ void coefs(const T* base, int idx, const T* D, const T* s) {
        auto fc = [&](int ax, T a, T b) -> T { return HARM ? (a * b) / (a + b) * s[ax] : (a + b) * s[ax]; };
#pragma unroll
        for (int ax = 0; ax < 3; ax++)
#pragma unroll
            for (int o = 0; o < 8; o++) {
                co[ax][o] = fc(ax, D[o], base[idx + outer(ax, o)]);
                if (!(o & bit(ax))) ci[ax][inner(ax, o)] = fc(ax, D[o], D[o ^ bit(ax)]);
            }
    }
    // diagonal of octant o's equation with mua m
    __device__ __forceinline__ T diag(int o, T m) const {
        T d = m;
#pragma unroll
        for (int ax = 0; ax < 3; ax++) d += ci[ax][inner(ax, o)] + co[ax][o];
        return d;
    }
    // q + sum_j c_ij u_j at the octants of colour C (the Gauss-Seidel value
    // is w times it).  All LDS reads are issued before the first is used:
    // left to itself the compiler interleaves them with the sums and waits
    // for the LDS four times over.
    template <int C>
    __device__ __forceinline__ void numer(const T* base, int idx, T* s) const {
        T nb[8][3];
#pragma unroll
        for (int o = 0; o < 8; o++)
            if (colour(o) == C)
#pragma unroll
                for (int ax = 0; ax < 3; ax++) nb[o][ax] = base[idx + outer(ax, o)];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int o = 0; o < 8; o++)
            if (colour(o) == C) {
                s[o] = q[o];
#pragma unroll
                for (int ax = 0; ax < 3; ax++) s[o] += ci[ax][inner(ax, o)] * u[o ^ bit(ax)];
#pragma unroll
                for (int ax = 0; ax < 3; ax++) s[o] += co[ax][o] * nb[o][ax];
            }
    }
    // Gauss-Seidel update of colour C from numer's sums, published; vertices
    // with w = 0 keep their value (FIXED) or become 0
    template <int C, bool FIXED>
    __device__ __forceinline__ void update(T* base, int idx, const T* s) {
#pragma unroll
        for (int o = 0; o < 8; o++)
            if (colour(o) == C) {
                const T t = s[o] * w[o];
                u[o] = FIXED && w[o] == T(0) ? u[o] : t;
                base[idx + o * S] = u[o];
            }
    }
    template <int C, bool FIXED>
    __device__ __forceinline__ void half(T* base, int idx) {
        T s[8];
        numer<C>(base, idx, s);
        update<C, FIXED>(base, idx, s);
    }
    // residual of colour C, 0 where w = 0, and 0 for the other colour (whose
    // equations a sweep that ended with it has solved)
    template <int C>
    __device__ __forceinline__ void residual(const T* base, int idx, T* r) const {
        numer<C>(base, idx, r);
#pragma unroll
        for (int o = 0; o < 8; o++) r[o] = colour(o) != C || w[o] == T(0) ? T(0) : r[o] - u[o] / w[o];
    }
    // 64 x the full weighting to the block's corner of the published values
    // of colour C: octant o of this block and, where its bit is set, of the
    // block before
    template <int C>
    __device__ __forceinline__ static T weighted(const T* base, int idx) {
        T v[8][8], s = T(0);
#pragma unroll
        for (int o = 0; o < 8; o++)
#pragma unroll
            for (int k = 0; k < 8; k++)
                if (colour(o) == C && !(k & ~o))
                    v[o][k] = base[idx + o * S - ((k & 4) ? X : 0) - ((k & 2) ? Y : 0) - (k & 1)];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int o = 0; o < 8; o++)
            if (colour(o) == C) {
                T t = T(0);
#pragma unroll
                for (int k = 0; k < 8; k++)
                    if (!(k & ~o)) t += v[o][k];
                s += t * T(8 >> __builtin_popcount(o));
            }
        return s;
    }
    // trilinear correction of octant o from the coarse values E at the
    // block's corner and the next ones
    __device__ __forceinline__ static T corrected(const T* E, int o) {
        T s = T(0);
#pragma unroll
        for (int k = 0; k < 8; k++)
            if (!(k & ~o)) s += E[k];
        return s * T(1.0 / (1 << __builtin_popcount(o)));
    }
};

// ---------------------------------------------------------------------------
// Phases of a mid-size level: one workgroup per tile, the tile and a ring
// around it (the box) as NB^3 blocks of one thread each.
//   kB3PreZero  two red-black sweeps from zero, u and the restricted defect
//   kB3Pre      the same from u_in
//   kB3Zero     two sweeps from zero, u only (float32; tiles of 10^3, starting
//               at odd coordinates, in boxes of 16^3)
//   kB3Sweep    two sweeps from u_in, u only; optionally (a.partial) the
//               squared residual of u_in, on the tile's first colour
//   kB3Defect   the restricted defect of u_in, whose last half-sweep updated
//               the second colour
//   kB3Post     u_in plus the trilinear correction, two sweeps, u
//   kB3PostEpi  kB3Post on a general grid of at most one round of workgroups,
//               with the likelihood epilogue of the result: rhobar = mua w
//               (mua u - d) (0 on the boundary) and per-workgroup sums of
//               w (mua u - d)^2 and of w > 0
// Every block of the box is updated in every half-sweep; a vertex j rings
// inside the box then has the sequential sweeps' value after half-sweep j.
// What is formed nearer to the edge, from neighbours the box does not hold,
// is never read by what is kept: a wrong value moves in by one ring per
// half-sweep, and vertices that must not change are selected, not multiplied.
// Rings: four half-sweeps need 4 (3 from zero, where the first reads no
// neighbour); the defect of a coarse vertex 2X needs u final two vertices
// away.  Tiles are 8^3 with boxes of 16^3 (sweeps, correction), 18^3 (from
// zero: tiles start at odd coordinates, so the box reaches 5 vertices on
// either side) and 20^3 (float32 with the coarse kernel behind it; other
// levels, and float64, whose 1000 blocks exceed the registers of a CU, run
// kB3Sweep and kB3Defect instead); the defect's box of 16^3 gives 6^3 coarse
// vertices.
//
// Bound by latency (load, faces, four half-sweeps, store) and, from a few
// workgroups per CU on, by the arithmetic of the whole box: 8 to 16 times
// the tile's vertices, which is why larger levels march instead.  Measured
// (pre- / post-smoothing): float32 64^3 8.0 + 4.7 / 8.3 us, 32^3 6.2 / 5.3 us (with
// the fields in LDS and two coefficients read per neighbour 21.3 / 13.9 and
// 9.6 / 8.8 us); float64 48^3 9.3 / 7.4 us, 24^3 7.7 / 7.0 us (marching passes
// with the separate restriction 24 / 21 and 22 / 20 us); the paper's
// 128 x 64 x 64 grid 29 + 10 / 27 us (one operation per launch: 47 / 44 us).
enum Block3Mode { kB3PreZero = 0, kB3Pre = 1, kB3Sweep = 2, kB3Defect = 3, kB3Post = 4, kB3PostEpi = 5, kB3Zero = 6 };

template <class T>
struct Block3Args {
    const T* u_in;
    T* u_out;
    const T* q;
    const T* D;
    const T* w;        // inverse diagonal (0 on the boundary); GEN: mua
    const T* ec;       // coarse correction (kB3Post)
    T* qc;             // restricted defect (coarse interior written)
    double* partial;   // per-workgroup sums: kB3Sweep of squares (or null); kB3PostEpi two a workgroup, by kind
    double* norm;      // kB3Sweep with partial: their sum, by the last workgroup ...
    unsigned* done;    // ... counted here (null: not summed)
    int n[3];          // cells per axis
    int nt[3];         // tiles per axis
    T s[3];            // per axis: 1 / (2 h^2) or 2 / h^2 (harmonic)
    int order;         // colour of the first half-sweep
    const double *ed, *ew;   // kB3PostEpi: data, inverse variances
    double* rhobar;          // ... and dH/drho
    T* tape;                 // TAPE: the iterate after half-sweep j at tape + j tape_step (interior written);
    int64_t tape_step;       // u_out is not written
};

template <int MODE, bool GEN>
struct Block3Shape {
    static constexpr int NB = MODE == kB3PreZero ? 9 : MODE == kB3Pre ? 10 : 8;     // blocks per axis
    static constexpr int TILE = MODE == kB3Defect ? 12 : MODE == kB3Zero ? 10 : 8;   // fine vertices per tile and axis
    static constexpr int ORG = MODE == kB3Pre ? -6 : MODE == kB3Defect ? 0 : MODE == kB3Zero ? -2 : -4;   // box origin from TILE * tile
    static constexpr int LO = MODE == kB3PreZero ? 5 : MODE == kB3Pre ? 6 : MODE == kB3Zero ? 3 : 4;      // tile in the box
    static constexpr int HI = LO + (MODE == kB3Zero ? 10 : 8);
    static constexpr int CLO = MODE == kB3Defect ? 1 : 3, CHI = 7;                   // blocks whose corners are restricted to
    // general grids form w from the faces, which a sweep from zero needs on
    // the box's last vertices too: D one vertex past them, in a pad
    static constexpr bool EDGE = GEN && MODE == kB3PreZero;
    static constexpr int Y = NB + EDGE, X = Y * Y, S = X * Y;
    static constexpr int NT = (NB * NB * NB + 63) / 64 * 64;
    __host__ static int tiles(int N) {
        return MODE == kB3PreZero || MODE == kB3Zero ? (N - 1 + TILE - 1) / TILE
               : MODE == kB3Defect                     ? std::max(1, (N / 2 - 1 + 5) / 6)
                                                       : (N + 7) / 8;
    }
};

template <class T, int MODE, bool GEN>
constexpr size_t block3_lds() { return (size_t)8 * Block3Shape<MODE, GEN>::S * sizeof(T); }

// COHERENT: qc is stored past the caches, for a reader in the same launch.
// TAPE: every half-sweep's state is kept (the unrolled adjoint's record).
template <class T, int MODE, bool HARM, bool GEN, bool COHERENT = false, bool TAPE = false>
__device__ __forceinline__ void block3_body(const Block3Args<T>& a, const int bid) {
    using Sh = Block3Shape<MODE, GEN>;
    constexpr int NB = Sh::NB, S = Sh::S, X = Sh::X, Y = Sh::Y;
    constexpr bool ZERO = MODE == kB3PreZero || MODE == kB3Zero;
    extern __shared__ __align__(16) unsigned char block_smem[];
    T* const base = reinterpret_cast<T*>(block_smem);
    using B3 = Block3<T, S, X, Y>;
    B3 P;
    const int tid = threadIdx.x;
    const bool act = tid < NB * NB * NB;
    const int lz = tid % NB, ly = (tid / NB) % NB, lx = act ? tid / (NB * NB) : 0;
    const int idx = lx * X + ly * Y + lz;
    const int t = xcd_remap(bid, a.nt[0] * a.nt[1] * a.nt[2]);
    const int bx = t / (a.nt[1] * a.nt[2]), by = (t / a.nt[2]) % a.nt[1], bz = t % a.nt[2];
    const int g[3] = {bx * Sh::TILE + Sh::ORG + 2 * lx, by * Sh::TILE + Sh::ORG + 2 * ly, bz * Sh::TILE + Sh::ORG + 2 * lz};
    const int n1 = a.n[1] + 1, n2 = a.n[2] + 1;
    // per axis and bit: inside the grid, an interior coordinate, in the tile
    bool in[3][2], inner[3][2], tile[3][2];
    const int l3[3] = {2 * lx, 2 * ly, 2 * lz};
#pragma unroll
    for (int ax = 0; ax < 3; ax++)
#pragma unroll
        for (int k = 0; k < 2; k++) {
            in[ax][k] = g[ax] + k >= 0 && g[ax] + k <= a.n[ax];
            inner[ax][k] = g[ax] + k > 0 && g[ax] + k < a.n[ax];
            tile[ax][k] = l3[ax] + k >= Sh::LO && l3[ax] + k < Sh::HI;
        }
    auto of = [](const bool (&f)[3][2], int o) { return f[0][o >> 2] && f[1][(o >> 1) & 1] && f[2][o & 1]; };

    {
        // two vertices along z per load; outside the grid a clamped read,
        // replaced below; at z = n the pair read is (n - 1, n)
        struct Pair {
            T a, b;
        };
        int row[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int x = min(max(g[0] + (k >> 1), 0), a.n[0]), y = min(max(g[1] + (k & 1), 0), a.n[1]);
            row[k] = (x * n1 + y) * n2 + min(max(g[2], 0), a.n[2] - 1);
        }
        const bool last = g[2] == a.n[2];
        auto load = [&](const T* p, T* v) {
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const Pair r = *reinterpret_cast<const Pair*>(p + row[k]);
                v[2 * k] = last ? r.b : r.a;
                v[2 * k + 1] = r.b;
            }
        };
        T D[8], De[3][4];
        load(a.D, D);
        load(a.w, P.w);
        load(a.q, P.q);
        if (!ZERO) load(a.u_in, P.u);
        if (Sh::EDGE) {
            const int l[3] = {lx, ly, lz};
#pragma unroll
            for (int ax = 0; ax < 3; ax++)
#pragma unroll
                for (int o = 0; o < 8; o++) {
                    if (!(o & B3::bit(ax))) continue;
                    const int x = min(max(g[0] + (o >> 2) + (ax == 0), 0), a.n[0]);
                    const int y = min(max(g[1] + ((o >> 1) & 1) + (ax == 1), 0), a.n[1]);
                    const int z = min(max(g[2] + (o & 1) + (ax == 2), 0), a.n[2]);
                    De[ax][B3::inner(ax, o)] = act && l[ax] == NB - 1 ? a.D[(x * n1 + y) * n2 + z] : T(0);
                }
        }
        if (MODE == kB3Post || MODE == kB3PostEpi) {
            const int c0 = a.n[0] / 2, c1 = a.n[1] / 2, c2 = a.n[2] / 2;
            const int zc = g[2] >> 1, zr = min(max(zc, 0), c2 - 1);
            T E[8];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int x = min(max((g[0] >> 1) + (k >> 1), 0), c0), y = min(max((g[1] >> 1) + (k & 1), 0), c1);
                const Pair r = *reinterpret_cast<const Pair*>(a.ec + (x * (c1 + 1) + y) * (c2 + 1) + zr);
                E[2 * k] = zc == c2 ? r.b : r.a;
                E[2 * k + 1] = r.b;
            }
#pragma unroll
            for (int o = 0; o < 8; o++) P.u[o] += of(inner, o) ? B3::corrected(E, o) : T(0);
        }
        if (act) B3::publish(base, idx, D);
        if (Sh::EDGE) {
            const int l[3] = {lx, ly, lz};
#pragma unroll
            for (int ax = 0; ax < 3; ax++)
#pragma unroll
                for (int o = 0; o < 8; o++)
                    if ((o & B3::bit(ax)) && act && l[ax] == NB - 1) base[idx + B3::outer(ax, o)] = De[ax][B3::inner(ax, o)];
        }
        __syncthreads();
        P.template coefs<HARM>(base, idx, D, a.s);
#pragma unroll
        for (int o = 0; o < 8; o++) {
            if (GEN) P.w[o] = T(1) / P.diag(o, P.w[o]);
            P.w[o] = of(inner, o) ? P.w[o] : T(0);
            P.q[o] = of(in, o) ? P.q[o] : T(0);
            if (ZERO) P.u[o] = of(inner, o) && B3::colour(o) == a.order ? P.w[o] * P.q[o] : T(0);
            else P.u[o] = of(in, o) ? P.u[o] : T(0);
        }
        __syncthreads();
        if (act) B3::publish(base, idx, P.u);
        __syncthreads();
    }
    auto residual = [&](T* r) {
        if (a.order) P.template residual<1>(base, idx, r);
        else P.template residual<0>(base, idx, r);
    };
    double part = 0.0;
    if (MODE == kB3Sweep && a.partial) {
        double acc = 0.0;
        if (act) {
            T r[8];
            residual(r);
#pragma unroll
            for (int o = 0; o < 8; o++) acc += of(tile, o) ? (double)r[o] * (double)r[o] : 0.0;
        }
        part = block_sum(acc);
    }
    if (MODE != kB3Defect) {
        auto store = [&](T* out) {
            if (!act) return;
            const int v0 = (g[0] * n1 + g[1]) * n2 + g[2];
#pragma unroll
            for (int o = 0; o < 8; o++)
                if (of(tile, o) && of(inner, o)) out[v0 + ((o >> 2) * n1 + ((o >> 1) & 1)) * n2 + (o & 1)] = P.u[o];
        };
        if (TAPE && MODE == kB3PreZero) store(a.tape);
        // the first half-sweep from zero was u = w q
        for (int j = ZERO ? 1 : 0; j < 4; j++) {
            if (act) {
                if ((j & 1) ? !a.order : a.order) P.template half<1, true>(base, idx);
                else P.template half<0, true>(base, idx);
            }
            if (TAPE) store(a.tape + j * a.tape_step);
            __syncthreads();
        }
        if (!TAPE) store(a.u_out);
    }
    if (MODE == kB3Sweep && a.partial) {
        if (a.done) sum_arrived(part, a.partial, bid, (unsigned)(a.nt[0] * a.nt[1] * a.nt[2]), a.done, a.norm);
        else if (tid == 0) a.partial[bid] = part;
    }
    if constexpr (MODE == kB3PostEpi) {
        double acc = 0.0, cnt = 0.0;
        if (act) {
            const int v0 = (g[0] * n1 + g[1]) * n2 + g[2];
            // the last tile of an axis takes the grid's last vertices too
            const int b3[3] = {bx, by, bz};
#pragma unroll
            for (int ax = 0; ax < 3; ax++)
#pragma unroll
                for (int k = 0; k < 2; k++)
                    if (g[ax] + k == a.n[ax] && b3[ax] == a.nt[ax] - 1) tile[ax][k] = true;
#pragma unroll
            for (int o = 0; o < 8; o++) {
                if (!of(tile, o) || !of(in, o)) continue;
                const int v = v0 + ((o >> 2) * n1 + ((o >> 1) & 1)) * n2 + (o & 1);
                if (!of(inner, o)) {
                    a.rhobar[v] = 0.0;
                    continue;
                }
                const double m = a.w[v], wv = a.ew[v], res = m * P.u[o] - a.ed[v];
                a.rhobar[v] = m * wv * res;
                acc += wv * res * res;
                cnt += wv > 0.0 ? 1.0 : 0.0;
            }
        }
        const double sa = block_sum(acc), sc = block_sum(cnt);
        if (tid == 0) {
            a.partial[bid] = sa;
            a.partial[gridDim.x + bid] = sc;
        }
    }
    if (MODE == kB3PreZero || MODE == kB3Pre || MODE == kB3Defect) {
        T r[8];
        if (act) residual(r);
        __syncthreads();
        if (act) B3::publish(base, idx, r);
        __syncthreads();
        const bool mine = act && lx >= Sh::CLO && lx < Sh::CHI && ly >= Sh::CLO && ly < Sh::CHI && lz >= Sh::CLO && lz < Sh::CHI;
        if (mine && inner[0][0] && inner[1][0] && inner[2][0]) {   // a coarse interior vertex
            const T s = a.order ? B3::template weighted<1>(base, idx) : B3::template weighted<0>(base, idx);
            T* const qv = a.qc + ((g[0] >> 1) * (a.n[1] / 2 + 1) + (g[1] >> 1)) * (a.n[2] / 2 + 1) + (g[2] >> 1);
            if (COHERENT) __hip_atomic_store(qv, s * T(1.0 / 64.0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else *qv = s * T(1.0 / 64.0);
        }
    }
}

template <class T, int MODE, bool HARM, bool GEN>
__global__ __launch_bounds__((Block3Shape<MODE, GEN>::NT)) void k_block3(Block3Args<T> a) {
    block3_body<T, MODE, HARM, GEN>(a, blockIdx.x);
}

template <int MODE, bool HARM>
__global__ __launch_bounds__((Block3Shape<MODE, false>::NT)) void k_block3_tape(Block3Args<double> a) {
    block3_body<double, MODE, HARM, false, false, true>(a, blockIdx.x);
}

template <class T, int MODE, bool HARM>
__global__ __launch_bounds__((Block3Shape<MODE, false>::NT)) void k_block3_grp(const Group<Block3Args<T>>* g) {
    int bid;
    const int m = group_member(g, &bid);
    if (bid < 0) return;
    block3_body<T, MODE, HARM, false>(g->a[m], bid);
}

}  // namespace dmgs
