// kernels_2d.hpp -- kernels of the two-dimensional (five-point) variant.
//
// Grid: N cells per axis, (N+1)^2 vertices, x slowest, y fastest,
// v = x*(N+1) + y; interior vertices have both coordinates in [1, N-1].
// The operator is the two-dimensional form of Eq. (maineq):
//   (A u)_i = sum over the 4 neighbours j of c_ij (u_i - u_j) + mua_i u_i,
//   c_ij = D_f / h^2 with the arithmetic (or harmonic) face mean,
// red = (x + y) even, restriction (1/16)(1,2,1) x (1,2,1), bilinear
// prolongation, coefficients coarsened by full weighting (injection on the
// boundary) -- the readings of the three-dimensional solver.
//
// Every kernel here is float64 and memory-bound.  Kernels that read
// neighbouring rows take one item per thread over a grid of whole blocks
// rounded up to a multiple of 8, remapped so that each XCD walks a
// contiguous band of rows (the rows it reads twice stay in its L2).
#pragma once
#include "grid.hpp"
#include "kernels_basic.hpp"

namespace dmgs {

__device__ __forceinline__ bool interior2(int N, int x, int y) { return x > 0 && x < N && y > 0 && y < N; }

__device__ __forceinline__ int64_t item_of_thread2() {
    return (int64_t)xcd_tile(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
}

// ---------------------------------------------------------------------------
// Coefficients.

__global__ void k2_validate(const double* __restrict__ D, const double* __restrict__ mu, int N, int* __restrict__ bad) {
    const int n = N + 1;
    const int64_t nv = (int64_t)n * n;
    int b = 0;
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < nv; v += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(v / n), y = (int)(v % n);
        if (!coef_ok(D[v], mu[v], interior2(N, x, y))) b = 1;
    }
    if (b) atomicOr(bad, 1);
}

__global__ void k2_exp_validate(const double* __restrict__ logD, const double* __restrict__ logmu,
                                double* __restrict__ D, double* __restrict__ mu, int N, int* __restrict__ bad) {
    const int n = N + 1;
    const int64_t nv = (int64_t)n * n;
    int b = 0;
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < nv; v += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(v / n), y = (int)(v % n);
        const double d = exp(logD[v]), m = exp(logmu[v]);
        D[v] = d;
        mu[v] = m;
        if (!coef_ok(d, m, interior2(N, x, y))) b = 1;
    }
    if (b) atomicOr(bad, 1);
}

// sum over a, b in {-1, 0, 1} of (2 - |a|)(2 - |b|) f[2X + a, 2Y + b] / 16
__device__ __forceinline__ double full_weight2(const double* __restrict__ f, int nf, int X, int Y) {
    double s = 0.0;
    for (int a = -1; a <= 1; a++) {
        const double* row = f + (int64_t)(2 * X + a) * nf + 2 * Y;
        s += (double)(2 - abs(a)) * (row[-1] + 2.0 * row[0] + row[1]);
    }
    return s * (1.0 / 16.0);
}

__global__ void k2_coarsen_coef(const double* __restrict__ fD, const double* __restrict__ fmu, double* __restrict__ cD,
                                double* __restrict__ cmu, int Nf) {
    const int Nc = Nf / 2, nf = Nf + 1, nc = Nc + 1;
    const int64_t v = item_of_thread2();
    if (v >= (int64_t)nc * nc) return;
    const int X = (int)(v / nc), Y = (int)(v % nc);
    if (!interior2(Nc, X, Y)) {
        const int64_t i = (int64_t)(2 * X) * nf + 2 * Y;
        cD[v] = fD[i];
        cmu[v] = fmu[i];
        return;
    }
    cD[v] = full_weight2(fD, nf, X, Y);
    cmu[v] = full_weight2(fmu, nf, X, Y);
}

// ---------------------------------------------------------------------------
// The cycle.

// u = 0 on interior vertices, g on the boundary.
__global__ void k2_init_iterate(double* __restrict__ u, int N, double g) {
    const int n = N + 1;
    const int64_t nv = (int64_t)n * n;
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < nv; v += (int64_t)gridDim.x * blockDim.x)
        u[v] = interior2(N, (int)(v / n), (int)(v % n)) ? 0.0 : g;
}

// One red (colour 0) or black (colour 1) half-sweep in place (Sec. 2.2):
// u_i = (q_i + sum_j c_ij u_j) / (sum_j c_ij + mua_i) on the interior
// vertices of the colour.  Item t = row (x - 1) * (N/2) + j is the j-th
// vertex of the colour in row x; N is even on every level that smooths.
template <bool HARM>
__global__ void k2_half_sweep(double* __restrict__ u, const double* __restrict__ q, const double* __restrict__ D,
                              const double* __restrict__ mu, int N, Stencil<double> s, int colour) {
    const int S = N / 2;
    const int64_t t = item_of_thread2();
    if (t >= (int64_t)(N - 1) * S) return;
    const int x = 1 + (int)(t / S);
    const int y = (((colour - x) & 1) ? 1 : 2) + 2 * (int)(t % S);
    if (y >= N) return;
    const int n = N + 1;
    const int64_t i = (int64_t)x * n + y;
    const double Di = D[i];
    const double cxm = face<HARM>(Di, D[i - n], s), cxp = face<HARM>(Di, D[i + n], s);
    const double cym = face<HARM>(Di, D[i - 1], s), cyp = face<HARM>(Di, D[i + 1], s);
    u[i] = (q[i] + cxm * u[i - n] + cxp * u[i + n] + cym * u[i - 1] + cyp * u[i + 1]) / (cxm + cxp + cym + cyp + mu[i]);
}

// q - A u at the interior vertex i = (x, y) (row stride n).
template <bool HARM>
__device__ __forceinline__ double defect2_at(const double* __restrict__ u, const double* __restrict__ q,
                                             const double* __restrict__ D, const double* __restrict__ mu, int64_t i,
                                             int n, const Stencil<double>& s) {
    const double Di = D[i], ui = u[i];
    return q[i] - (mu[i] * ui + face<HARM>(Di, D[i - n], s) * (ui - u[i - n]) + face<HARM>(Di, D[i + n], s) * (ui - u[i + n]) +
                   face<HARM>(Di, D[i - 1], s) * (ui - u[i - 1]) + face<HARM>(Di, D[i + 1], s) * (ui - u[i + 1]));
}

// qc = R (q - A u) (Sec. 2.3.2 and Eq. (rest)): one coarse vertex per
// thread, its nine fine defects formed on the fly (0 on the coarse boundary).
template <bool HARM>
__global__ void k2_defect_restrict(const double* __restrict__ u, const double* __restrict__ q,
                                   const double* __restrict__ D, const double* __restrict__ mu, int Nf,
                                   Stencil<double> s, double* __restrict__ qc) {
    const int Nc = Nf / 2, nf = Nf + 1, nc = Nc + 1;
    const int64_t v = item_of_thread2();
    if (v >= (int64_t)nc * nc) return;
    const int X = (int)(v / nc), Y = (int)(v % nc);
    if (!interior2(Nc, X, Y)) {
        qc[v] = 0.0;
        return;
    }
    double acc = 0.0;
    for (int a = -1; a <= 1; a++) {
        const int64_t i = (int64_t)(2 * X + a) * nf + 2 * Y;
        const double row = defect2_at<HARM>(u, q, D, mu, i - 1, nf, s) + 2.0 * defect2_at<HARM>(u, q, D, mu, i, nf, s) +
                           defect2_at<HARM>(u, q, D, mu, i + 1, nf, s);
        acc += (double)(2 - abs(a)) * row;
    }
    qc[v] = acc * (1.0 / 16.0);
}

// u += I ec on fine interior vertices (Sec. 2.3.3, bilinear).
__global__ void k2_prolong_add(const double* __restrict__ ec, double* __restrict__ u, int Nf) {
    const int nf = Nf + 1, nc = Nf / 2 + 1;
    const int64_t v = item_of_thread2();
    if (v >= (int64_t)nf * nf) return;
    const int x = (int)(v / nf), y = (int)(v % nf);
    if (!interior2(Nf, x, y)) return;
    const int X0 = x >> 1, X1 = (x + 1) >> 1, Y0 = y >> 1, Y1 = (y + 1) >> 1;
    const double* r0 = ec + (int64_t)X0 * nc;
    const double* r1 = ec + (int64_t)X1 * nc;
    double e;
    if (X0 == X1) e = (Y0 == Y1) ? r0[Y0] : 0.5 * (r0[Y0] + r0[Y1]);
    else if (Y0 == Y1) e = 0.5 * (r0[Y0] + r1[Y0]);
    else e = 0.25 * (r0[Y0] + r1[Y0] + r0[Y1] + r1[Y1]);
    u[v] += e;
}

// Exact solve on the coarsest level (N in {2, 3}: at most 4 unknowns), the
// boundary values of u moved to the right-hand side; one thread, Cholesky.
template <bool HARM>
__global__ void k2_exact(const double* __restrict__ q, double* __restrict__ u, const double* __restrict__ D,
                         const double* __restrict__ mu, int N, Stencil<double> s) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    const int n = N + 1, m1 = N - 1, m = m1 * m1;
    double A[4][4], b[4];
    for (int r = 0; r < m; r++)
        for (int c = 0; c < m; c++) A[r][c] = 0.0;
    for (int x = 1; x < N; x++)
        for (int y = 1; y < N; y++) {
            const int t = (x - 1) * m1 + (y - 1);
            const int i = x * n + y;
            A[t][t] = mu[i];
            b[t] = q[i];
            const int nb[4][2] = {{x - 1, y}, {x + 1, y}, {x, y - 1}, {x, y + 1}};
            for (int e = 0; e < 4; e++) {
                const int xa = nb[e][0], ya = nb[e][1], j = xa * n + ya;
                const double c = face<HARM>(D[i], D[j], s);
                A[t][t] += c;
                if (interior2(N, xa, ya)) A[t][(xa - 1) * m1 + (ya - 1)] -= c;
                else b[t] += c * u[j];
            }
        }
    for (int j = 0; j < m; j++) {
        double d = A[j][j];
        for (int p = 0; p < j; p++) d -= A[j][p] * A[j][p];
        d = sqrt(d);
        A[j][j] = d;
        for (int i = j + 1; i < m; i++) {
            double acc = A[i][j];
            for (int p = 0; p < j; p++) acc -= A[i][p] * A[j][p];
            A[i][j] = acc / d;
        }
    }
    for (int i = 0; i < m; i++) {
        double acc = b[i];
        for (int p = 0; p < i; p++) acc -= A[i][p] * b[p];
        b[i] = acc / A[i][i];
    }
    for (int i = m - 1; i >= 0; i--) {
        double acc = b[i];
        for (int p = i + 1; p < m; p++) acc -= A[p][i] * b[p];
        b[i] = acc / A[i][i];
    }
    for (int x = 1; x < N; x++)
        for (int y = 1; y < N; y++) u[x * n + y] = b[(x - 1) * m1 + (y - 1)];
}

// partial[block] = sum over the block's interior vertices of (q - A u)^2.
template <bool HARM>
__global__ void k2_resid_sq(const double* __restrict__ u, const double* __restrict__ q, const double* __restrict__ D,
                            const double* __restrict__ mu, int N, Stencil<double> s, double* __restrict__ partial) {
    const int n = N + 1;
    const int64_t nv = (int64_t)n * n;
    double acc = 0.0;
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < nv; v += (int64_t)gridDim.x * blockDim.x) {
        if (!interior2(N, (int)(v / n), (int)(v % n))) continue;
        const double r = defect2_at<HARM>(u, q, D, mu, v, n, s);
        acc += r * r;
    }
    const double b = block_sum(acc);
    if (threadIdx.x == 0) partial[blockIdx.x] = b;
}

// ---------------------------------------------------------------------------
// Derivatives (the adjoint-state formulas of the three-dimensional solver
// with four neighbours).

// rhs = dq - (dA) rho on interior vertices, 0 on the boundary; dA along
// dlogD (face values) and dlogmu (dmua = mua dlogmu).  dq, dlogD or dlogmu
// may be null (zero).
__global__ void k2_tangent_rhs(const double* __restrict__ rho, const double* __restrict__ dq,
                               const double* __restrict__ dlogD, const double* __restrict__ dlogmu,
                               const double* __restrict__ D, const double* __restrict__ mu, int N, double inv_h2,
                               int harmonic, double* __restrict__ rhs) {
    const int n = N + 1;
    const int64_t i = item_of_thread2();
    if (i >= (int64_t)n * n) return;
    const int x = (int)(i / n), y = (int)(i % n);
    if (!interior2(N, x, y)) {
        rhs[i] = 0.0;
        return;
    }
    const int off[4] = {n, -n, 1, -1};
    const double ri = rho[i], Di = D[i];
    double acc = dlogmu ? mu[i] * dlogmu[i] * ri : 0.0;
    if (dlogD) {
        const double dDi = Di * dlogD[i];
        for (int e = 0; e < 4; e++) {
            const int64_t j = i + off[e];
            const double Dj = D[j], dDj = Dj * dlogD[j];
            double dDf;
            if (harmonic) {
                const double sum = Di + Dj;
                dDf = 2.0 * (Dj * Dj * dDi + Di * Di * dDj) / (sum * sum);
            } else {
                dDf = 0.5 * (dDi + dDj);
            }
            acc += dDf * inv_h2 * (ri - rho[j]);
        }
    }
    rhs[i] = (dq ? dq[i] : 0.0) - acc;
}

// g_logmua = -mua lam rho (interior, 0 on the boundary);
// g_logD_v = -sum over faces (v, j) with an interior endpoint of
// dD_f/dlogD_v (lam_v - lam_j)(rho_v - rho_j) / h^2, lam = 0 on the boundary.
__global__ void k2_coef_grads(const double* __restrict__ rho, const double* __restrict__ lam,
                              const double* __restrict__ D, const double* __restrict__ mu, int N, double inv_h2,
                              int harmonic, double* __restrict__ gD, double* __restrict__ gmu) {
    const int n = N + 1;
    const int64_t v = item_of_thread2();
    if (v >= (int64_t)n * n) return;
    const int x = (int)(v / n), y = (int)(v % n);
    const bool vin = interior2(N, x, y);
    const double lv = vin ? lam[v] : 0.0, rv = rho[v], Dv = D[v];
    if (gmu) gmu[v] = vin ? -mu[v] * lv * rv : 0.0;
    if (!gD) return;
    double acc = 0.0;
    const int o[4][2] = {{1, 0}, {-1, 0}, {0, 1}, {0, -1}};
    for (int e = 0; e < 4; e++) {
        const int xa = x + o[e][0], ya = y + o[e][1];
        if (xa < 0 || xa > N || ya < 0 || ya > N) continue;
        const bool jin = interior2(N, xa, ya);
        if (!vin && !jin) continue;
        const int64_t j = (int64_t)xa * n + ya;
        const double lj = jin ? lam[j] : 0.0, Dj = D[j];
        double dcdv;
        if (harmonic) {
            const double sum = Dv + Dj;
            dcdv = 2.0 * Dj * Dj * Dv / (sum * sum);
        } else {
            dcdv = 0.5 * Dv;
        }
        acc += dcdv * (lv - lj) * (rv - rho[j]);
    }
    gD[v] = -acc * inv_h2;
}

}  // namespace dmgs

namespace dmgs {

// ---------------------------------------------------------------------------
// Two red-black sweeps per pass, out of place (u_in -> u_out).
//
// One wave per tile of TILE interior columns [ts, ts + TILE); lane t holds
// the column pair (yb + 2t, yb + 2t + 1), yb = ts - RING, so a wave covers
// the tile and a ring of RING columns on each side (TILE = 128 - 2 RING).
// A chunk of rows [xa, xb) is marched one row per step; the four colour
// updates of the two sweeps run as a pipeline: at step s, stage j (j =
// 1..4) updates row s - j + 1, which then sees its neighbours exactly as the
// sequential order leaves them (a stage never changes the other colour).
// Stage j is applied on the tile plus a ring of RING - j columns
// (neighbouring tiles recompute these), and its rows reach RING - j beyond
// the chunk, so the output rows depend only on rows [xa - RING, xb + RING)
// of u_in.  Each lane keeps eight rows of its two columns (u, D, q, mua) in
// a register ring indexed by row & 7 (the march is unrolled by 8, so ring
// slots are compile-time); in-row neighbours of the other column come from
// the adjacent lane by a shuffle.  A row is loaded three steps before the
// first stage reads it and enters its ring slot at the end of the step.
// Only interior vertices of the tile are written; u_out's boundary keeps
// its values.  Rows: with O = RING - 1, chunk 0 is [1, O + chunk) and chunk
// c > 0 is [O + c chunk, O + (c + 1) chunk), cut at N (chunk a multiple of
// 8, so that every march starts at a multiple of 8).
//
// PROLONG (post-smoothing): the pass smooths u_in + I ec (Sec. 2.3.3,
// bilinear, ec on the next coarser level with a zero boundary); the
// correction of a row is added at the step before its first use, from
// coarse values loaded with the row.
//
// DEFECT (pre-smoothing): RING = 5, so the final values are known on the
// tile plus a ring of 1 and on one row beyond the chunk; at step s, once
// row s - 3 is final, the pass also writes the defect r = q - A u of row
// s - 4 on the tile (Sec. 2.3.2), for the restriction to read.
template <bool DEFECT> struct Sweep2Shape2 {
    static constexpr int RING = DEFECT ? 5 : 4, TILE = 2 * kWave - 2 * RING;
};
constexpr int kTile2 = Sweep2Shape2<false>::TILE, kTile2D = Sweep2Shape2<true>::TILE;

template <bool HARM, bool PROLONG, bool DEFECT = false>
__global__ __launch_bounds__(256) void k2_sweep2(const double* __restrict__ uin, double* __restrict__ uout,
                                                 const double* __restrict__ q, const double* __restrict__ D,
                                                 const double* __restrict__ mu, const double* __restrict__ ec,
                                                 double* __restrict__ rout, int N, Stencil<double> st,
                                                 int first_colour, int chunk, int ntiles, int nchunks) {
    static_assert(!(PROLONG && DEFECT), "the defect is formed after pre-smoothing only");
    constexpr int RING = Sweep2Shape2<DEFECT>::RING, TILE = Sweep2Shape2<DEFECT>::TILE, O = RING - 1;
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int tile = wave % ntiles, ch = wave / ntiles;
    if (ch >= nchunks) return;   // whole waves exit
    const int n = N + 1;
    const int ts = 1 + tile * TILE;
    const int yb = ts - RING;
    const int ya = yb + 2 * lane, yo = ya + 1;   // this lane's columns
    const int xa = ch == 0 ? 1 : O + ch * chunk, xb = min(N, O + (ch + 1) * chunk);
    // rows and columns outside the grid are read clamped to its edge: no
    // update that is kept reads them (an updated interior vertex has all its
    // neighbours in the grid), and unconditional loads let the compiler wait
    // for each row's loads alone
    const int yca = min(max(ya, 0), N), yco = min(max(yo, 0), N);

    double ua[8], uo[8], da[8], dd[8], qa[8], qo[8], ma[8], mo[8];
    // coarse values of the correction: rows X0 = r >> 1 and X1 = (r + 1) >> 1,
    // columns C0 = ya >> 1 and C0 + 1
    double e00[8], e01[8], e10[8], e11[8];
    const int Nc = N >> 1, nc = Nc + 1;
    // (clamped separately: on the left edge the lane of columns (-1, 0) must
    // take column 0 of ec, which is 0, for y = 0)
    const int C0 = min(max(ya >> 1, 0), Nc), C1 = min(max((ya >> 1) + 1, 0), Nc);
    struct Row {
        double ua, uo, da, dd, qa, qo, ma, mo, e00, e01, e10, e11;
    };
    // 32-bit element offsets (a grid has at most 16385^2 < 2^32 vertices)
    auto fetch_row = [&](int r) __attribute__((always_inline)) {
        Row t;
        const uint32_t b = (uint32_t)min(max(r, 0), N) * (uint32_t)n;
        t.ua = uin[b + yca];
        t.uo = uin[b + yco];
        t.da = D[b + yca];
        t.dd = D[b + yco];
        t.qa = q[b + yca];
        t.qo = q[b + yco];
        t.ma = mu[b + yca];
        t.mo = mu[b + yco];
        t.e00 = t.e01 = t.e10 = t.e11 = 0.0;
        if (PROLONG) {
            const int rc = min(max(r, 0), N);
            const uint32_t b0 = (uint32_t)(rc >> 1) * (uint32_t)nc, b1 = (uint32_t)min((rc + 1) >> 1, Nc) * (uint32_t)nc;
            t.e00 = ec[b0 + C0];
            t.e01 = ec[b0 + C1];
            t.e10 = ec[b1 + C0];
            t.e11 = ec[b1 + C1];
        }
        return t;
    };
    auto store_row = [&](const Row& t, int sl) __attribute__((always_inline)) {
        ua[sl] = t.ua; uo[sl] = t.uo; da[sl] = t.da; dd[sl] = t.dd;
        qa[sl] = t.qa; qo[sl] = t.qo; ma[sl] = t.ma; mo[sl] = t.mo;
        if (PROLONG) { e00[sl] = t.e00; e01[sl] = t.e01; e10[sl] = t.e10; e11[sl] = t.e11; }
    };
    // u += I ec on row r (the bilinear weights of k2_prolong_add; the
    // boundary gets 0, as ec vanishes there)
    auto correct_row = [&](int r, int sl) __attribute__((always_inline)) {
        if (!PROLONG) return;
        const bool rodd = r & 1;
        const double c0 = rodd ? 0.5 * (e00[sl] + e10[sl]) : e00[sl];
        const double c1 = rodd ? 0.5 * (e01[sl] + e11[sl]) : e01[sl];
        const double cm = rodd ? 0.25 * (e00[sl] + e10[sl] + e01[sl] + e11[sl]) : 0.5 * (e00[sl] + e01[sl]);
        // ya even: ya on C0, yo between C0 and C1; ya odd: the reverse
        const bool aodd = ya & 1;
        ua[sl] += aodd ? cm : c0;
        uo[sl] += aodd ? c1 : cm;
    };
    // colour c on row r (slot sl, rows r -1 / r + 1 in slots sm / sp), on the
    // tile plus a ring of `ring` columns
    auto stage = [&](int r, int sl, int sm, int sp, int c, int ring) __attribute__((always_inline)) {
        // the pair column of the colour (wave-uniform): odd -> yo, else ya;
        // every ring entry is updated through value selects, so the ring
        // stays in registers
        const bool odd = (c - r - yb) & 1;
        const double su = odd ? ua[sl] : uo[sl], sd = odd ? da[sl] : dd[sl];   // the pair's other column
        const int src = odd ? min(lane + 1, kWave - 1) : max(lane - 1, 0);
        const double un = __shfl(su, src, kWave), dn = __shfl(sd, src, kWave);   // the adjacent lane's
        const double ul = odd ? su : un, ur = odd ? un : su;
        const double dl = odd ? sd : dn, dr = odd ? dn : sd;
        const double Di = odd ? dd[sl] : da[sl];
        const double cxm = face<HARM>(Di, odd ? dd[sm] : da[sm], st), cxp = face<HARM>(Di, odd ? dd[sp] : da[sp], st);
        const double cym = face<HARM>(Di, dl, st), cyp = face<HARM>(Di, dr, st);
        const double um = odd ? uo[sm] : ua[sm], up = odd ? uo[sp] : ua[sp];
        const double qi = odd ? qo[sl] : qa[sl], mi = odd ? mo[sl] : ma[sl];
        const double v = (qi + cxm * um + cxp * up + cym * ul + cyp * ur) / (cxm + cxp + cym + cyp + mi);
        const int y = odd ? yo : ya;
        const bool act = r >= 1 && r <= N - 1 && y >= max(1, ts - ring) && y <= min(N - 1, ts + TILE - 1 + ring);
        ua[sl] = (act && !odd) ? v : ua[sl];
        uo[sl] = (act && odd) ? v : uo[sl];
    };
    // defect of row r (slot sl, final rows r -1 / r + 1 in slots sm / sp) on
    // the tile, in the order of defect2_at
    auto defect_row = [&](int r, int sl, int sm, int sp) __attribute__((always_inline)) {
        const double uL = __shfl_up(uo[sl], 1, kWave), dL = __shfl_up(dd[sl], 1, kWave);       // column ya - 1
        const double uR = __shfl_down(ua[sl], 1, kWave), dR = __shfl_down(da[sl], 1, kWave);   // column yo + 1
        if (r < xa || r >= xb) return;
        const uint32_t b = (uint32_t)r * (uint32_t)n;
        const double Da = da[sl], u_a = ua[sl];
        const double Do = dd[sl], u_o = uo[sl];
        const double ra = qa[sl] - (ma[sl] * u_a + face<HARM>(Da, da[sm], st) * (u_a - ua[sm]) +
                                    face<HARM>(Da, da[sp], st) * (u_a - ua[sp]) + face<HARM>(Da, dL, st) * (u_a - uL) +
                                    face<HARM>(Da, Do, st) * (u_a - u_o));
        const double ro = qo[sl] - (mo[sl] * u_o + face<HARM>(Do, dd[sm], st) * (u_o - uo[sm]) +
                                    face<HARM>(Do, dd[sp], st) * (u_o - uo[sp]) + face<HARM>(Do, Da, st) * (u_o - u_a) +
                                    face<HARM>(Do, dR, st) * (u_o - uR));
        if (ya >= ts && ya < ts + TILE && ya <= N - 1) rout[b + ya] = ra;
        if (yo >= ts && yo < ts + TILE && yo <= N - 1) rout[b + yo] = ro;
    };
    const int c1 = first_colour, c2 = 1 - first_colour;
    const int sb = (xa - O) & ~7;   // first step, a multiple of 8 (chunk 0 starts a few harmless steps early)
    const int se = xb + O;          // one past the last step
    // rows sb - 4 .. sb + 2 before the first step
#pragma unroll
    for (int k = -4; k <= 2; k++) store_row(fetch_row(sb + k), k & 7);
#pragma unroll
    for (int k = -4; k <= 0; k++) correct_row(sb + k, k & 7);
    for (int s8 = sb; s8 < se; s8 += 8) {
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int s = s8 + k;
            const Row next = fetch_row(s + 3);   // enters slot (k + 3) & 7 (row s - 5's) at the end of the step
            correct_row(s + 1, (k + 1) & 7);   // first read by stage 1 below
            stage(s, k & 7, (k - 1) & 7, (k + 1) & 7, c1, RING - 1);
            stage(s - 1, (k - 1) & 7, (k - 2) & 7, k & 7, c2, RING - 2);
            stage(s - 2, (k - 2) & 7, (k - 3) & 7, (k - 1) & 7, c1, RING - 3);
            stage(s - 3, (k - 3) & 7, (k - 4) & 7, (k - 2) & 7, c2, RING - 4);
            const int r = s - 3;
            if (r >= xa && r < xb) {
                const uint32_t b = (uint32_t)r * (uint32_t)n;
                const int sl = (k - 3) & 7;
                if (ya >= ts && ya < ts + TILE && ya <= N - 1) uout[b + ya] = ua[sl];
                if (yo >= ts && yo < ts + TILE && yo <= N - 1) uout[b + yo] = uo[sl];
            }
            if (DEFECT) defect_row(s - 4, (k - 4) & 7, (k - 5) & 7, (k - 3) & 7);
            store_row(next, (k + 3) & 7);
        }
    }
}

// qc = R r on coarse interior vertices from a fine defect r written by a
// DEFECT pass (0 on the coarse boundary): (1/16)(1,2,1) x (1,2,1), summed
// in the order of k2_defect_restrict.
__global__ void k2_restrict_r(const double* __restrict__ r, double* __restrict__ qc, int Nf) {
    const int Nc = Nf / 2, nf = Nf + 1, nc = Nc + 1;
    const int64_t v = item_of_thread2();
    if (v >= (int64_t)nc * nc) return;
    const int X = (int)(v / nc), Y = (int)(v % nc);
    if (!interior2(Nc, X, Y)) {
        qc[v] = 0.0;
        return;
    }
    double acc = 0.0;
    for (int a = -1; a <= 1; a++) {
        const double* row = r + (int64_t)(2 * X + a) * nf + 2 * Y;
        acc += (double)(2 - abs(a)) * (row[-1] + 2.0 * row[0] + row[1]);
    }
    qc[v] = acc * (1.0 / 16.0);
}

}  // namespace dmgs

namespace dmgs {

// qc = R (q - A u) streamed along fine rows (Sec. 2.3.2 and Eq. (rest)).
// One wave per tile of kTileR = 62 coarse columns [Ys, Ys + 62): lane t
// holds the fine column pair (2Y, 2Y + 1) of coarse column Y = Ys - 1 + t
// (lanes 0 and 63 are halo lanes).  Each fine defect is formed once; a
// fine row gives the horizontal sums h_x(Y) = r(x, 2Y-1) + 2 r(x, 2Y) +
// r(x, 2Y+1) (one shuffle), and coarse row X is (h_{2X-1} + 2 h_{2X} +
// h_{2X+1}) / 16, the order in which k2_defect_restrict sums.  A chunk of
// coarse rows [Xa, Xb) (Xa = 1 + c cx, cx a multiple of 4) marches fine
// rows 2Xa - 2 ... 2Xb - 1 in steps of 8 with rows in a register ring
// (row x in slot x & 7), each loaded three steps before the step that
// forms its defect.  Only coarse interior vertices are written.
constexpr int kTileR = 62;

template <bool HARM>
__global__ __launch_bounds__(256) void k2_defect_restrict_rows(const double* __restrict__ u, const double* __restrict__ q,
                                                               const double* __restrict__ D,
                                                               const double* __restrict__ mu, int Nf,
                                                               Stencil<double> st, double* __restrict__ qc, int cx,
                                                               int ntiles, int nchunks) {
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int tile = wave % ntiles, ch = wave / ntiles;
    if (ch >= nchunks) return;   // whole waves exit
    const int Nc = Nf / 2, nf = Nf + 1, nc = Nc + 1;
    const int Ys = 1 + tile * kTileR;
    const int Y = Ys - 1 + lane;
    const int ye = 2 * Y, yo = ye + 1;                     // this lane's fine columns
    const int yce = min(max(ye, 0), Nf), yco = min(max(yo, 0), Nf);   // clamped reads (kept defects never need them)
    const int Xa = 1 + ch * cx, Xb = min(Nc, Xa + cx);
    const bool wr = lane >= 1 && lane <= kTileR && Y <= Nc - 1;

    double ue[8], uo[8], de[8], dd[8], qe[8], qo[8], me[8], mo[8];
    auto load_row = [&](int x, int sl) __attribute__((always_inline)) {
        const uint32_t b = (uint32_t)min(max(x, 0), Nf) * (uint32_t)nf;
        ue[sl] = u[b + yce];
        uo[sl] = u[b + yco];
        de[sl] = D[b + yce];
        dd[sl] = D[b + yco];
        qe[sl] = q[b + yce];
        qo[sl] = q[b + yco];
        me[sl] = mu[b + yce];
        mo[sl] = mu[b + yco];
    };
    // h_x for row x (slot sl; rows x -1 / x + 1 in slots sm / sp)
    auto hsum = [&](int sl, int sm, int sp) __attribute__((always_inline)) {
        const double uoL = __shfl_up(uo[sl], 1, kWave), doL = __shfl_up(dd[sl], 1, kWave);     // column 2Y - 1
        const double ueR = __shfl_down(ue[sl], 1, kWave), deR = __shfl_down(de[sl], 1, kWave); // column 2Y + 2
        const double Dei = de[sl], uei = ue[sl];
        const double re = qe[sl] - (me[sl] * uei + face<HARM>(Dei, de[sm], st) * (uei - ue[sm]) +
                                    face<HARM>(Dei, de[sp], st) * (uei - ue[sp]) + face<HARM>(Dei, doL, st) * (uei - uoL) +
                                    face<HARM>(Dei, dd[sl], st) * (uei - uo[sl]));
        const double Doi = dd[sl], uoi = uo[sl];
        const double ro = qo[sl] - (mo[sl] * uoi + face<HARM>(Doi, dd[sm], st) * (uoi - uo[sm]) +
                                    face<HARM>(Doi, dd[sp], st) * (uoi - uo[sp]) + face<HARM>(Doi, de[sl], st) * (uoi - uei) +
                                    face<HARM>(Doi, deR, st) * (uoi - ueR));
        const double roL = __shfl_up(ro, 1, kWave);   // r(x, 2Y - 1)
        return roL + 2.0 * re + ro;
    };
    const int x0 = 2 * Xa - 2;            // a multiple of 8
    const int xe = 2 * Xb;                // one past the last fine row, 2 Xb - 1
#pragma unroll
    for (int k = -1; k <= 2; k++) load_row(x0 + k, k & 7);
    double carry = 0.0, hmid = 0.0;
    for (int x8 = x0; x8 < xe; x8 += 8) {
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int x = x8 + k;
            load_row(x + 3, (k + 3) & 7);
            const double h = hsum(k & 7, (k - 1) & 7, (k + 1) & 7);
            if ((k & 1) == 0) {
                hmid = h;                 // x = 2X
            } else {                      // x = 2X + 1 closes coarse row X
                const int X = x >> 1;
                if (wr && X >= Xa && X < Xb) qc[(uint32_t)X * (uint32_t)nc + Y] = (carry + 2.0 * hmid + h) * (1.0 / 16.0);
                carry = h;
            }
        }
    }
}

}  // namespace dmgs

namespace dmgs {

// ---------------------------------------------------------------------------
// Blocks of 2 x 2 vertices in registers, shared by the two kernels below.
//
// A thread owns the block with even corner (2 bx, 2 by): quadrant o = 2 (x&1)
// + (y&1).  Its iterate, right-hand side, inverse diagonal and 12 face
// coefficients stay in registers for a whole smoothing phase, so an update
// reads only the two neighbours in other blocks, from LDS, where the iterate
// lies by quadrant (consecutive lanes read consecutive words).  A vertex's
// colour is its quadrant's bit parity.  Vertices that must not change (grid
// boundary, outside) have w = 0.
struct Pair2 {   // two vertices along y, aligned as one
    double a, b;
};

struct Block2 {
    double u[4], q[4], w[4];
    double cx[2], cy[2];     // faces inside the block: along x (by y bit), along y (by x bit)
    double ox[4], oy[4];     // faces to the neighbouring blocks, by quadrant

    // Face coefficients from the block's D (published at base[idx + o S])
    // and the neighbours' in LDS, and w = 1 / (their sum + mua) where keep.
    template <bool HARM, int S, int X>
    __device__ __forceinline__ void coefs(const double* base, int idx, const double* D, const double* mu, const bool* keep,
                                          const Stencil<double>& st) {
        double nx[4], ny[4];
#pragma unroll
        for (int o = 0; o < 4; o++) {
            nx[o] = base[idx + (o ^ 2) * S + ((o & 2) ? X : -X)];
            ny[o] = base[idx + (o ^ 1) * S + ((o & 1) ? 1 : -1)];
        }
#pragma unroll
        for (int o = 0; o < 4; o++) {
            ox[o] = face<HARM>(D[o], nx[o], st);
            oy[o] = face<HARM>(D[o], ny[o], st);
            if (!(o & 2)) cx[o & 1] = face<HARM>(D[o], D[o ^ 2], st);
            if (!(o & 1)) cy[o >> 1] = face<HARM>(D[o], D[o ^ 1], st);
        }
#pragma unroll
        for (int o = 0; o < 4; o++) {
            const double d = ((ox[o] + cx[o & 1]) + (oy[o] + cy[o >> 1])) + mu[o];
            w[o] = keep[o] ? 1.0 / d : 0.0;
        }
    }
    // q + sum_j c_ij u_j at the two quadrants of colour C
    template <int C, int S, int X>
    __device__ __forceinline__ void numer(const double* base, int idx, double* v) const {
        double nx[4], ny[4];
#pragma unroll
        for (int o = 0; o < 4; o++)
            if ((__builtin_popcount(o) & 1) == C) {
                nx[o] = base[idx + (o ^ 2) * S + ((o & 2) ? X : -X)];
                ny[o] = base[idx + (o ^ 1) * S + ((o & 1) ? 1 : -1)];
            }
        __builtin_amdgcn_sched_barrier(0);   // issue every read before the first is waited for
#pragma unroll
        for (int o = 0; o < 4; o++)
            if ((__builtin_popcount(o) & 1) == C)
                v[o] = ((q[o] + cx[o & 1] * u[o ^ 2]) + cy[o >> 1] * u[o ^ 1]) + (ox[o] * nx[o] + oy[o] * ny[o]);
    }
    // Gauss-Seidel update of colour C, published; vertices with w = 0 keep
    // their value (FIXED) or become 0
    template <int C, int S, int X, bool FIXED>
    __device__ __forceinline__ void half(double* base, int idx) {
        double v[4];
        numer<C, S, X>(base, idx, v);
#pragma unroll
        for (int o = 0; o < 4; o++)
            if ((__builtin_popcount(o) & 1) == C) {
                const double t = v[o] * w[o];
                u[o] = FIXED && w[o] == 0.0 ? u[o] : t;
                base[idx + o * S] = u[o];
            }
    }
    // after a sweep that ended with the other colour: residual of colour C
    // (the other's is 0), 0 where w = 0; all four published
    template <int C, int S, int X>
    __device__ __forceinline__ void residual(const double* base, int idx, double* r) const {
        numer<C, S, X>(base, idx, r);
#pragma unroll
        for (int o = 0; o < 4; o++)
            r[o] = (__builtin_popcount(o) & 1) != C || w[o] == 0.0 ? 0.0 : r[o] - u[o] / w[o];
    }
    // full weighting to the block's corner of what all blocks published:
    // quadrant o of this block and, where its bit is set, of the one before
    template <int S, int X>
    __device__ __forceinline__ static double restricted(const double* base, int idx) {
        const double a0 = base[idx], a1 = base[idx + S], b1 = base[idx + S - 1], a2 = base[idx + 2 * S],
                     b2 = base[idx + 2 * S - X], a3 = base[idx + 3 * S], b3 = base[idx + 3 * S - 1],
                     c3 = base[idx + 3 * S - X], d3 = base[idx + 3 * S - X - 1];
        return (4.0 * a0 + 2.0 * ((a1 + b1) + (a2 + b2)) + ((a3 + b3) + (c3 + d3))) * (1.0 / 16.0);
    }
};

// ---------------------------------------------------------------------------
// The coarse end of a two-dimensional V-cycle in one workgroup: levels
// ks .. L-1 (N_ks <= kSmall2MaxN).  The correction of level ks starts from 0
// with a zero boundary (a coarse correction); nu_pre sweeps, defect and
// restriction, the next level, prolongation and correction, nu_post sweeps;
// the coarsest level is solved exactly.
//
// Bound by latency: a chain of about 100 dependent steps.  The first level
// has at most 32 x 32 blocks, one per thread; the second's (at most 256)
// belong to waves 0 .. 3 as well, every further level's (at most 64) to one
// wave of its own, whose steps need no barrier.
//
// 64 cells: with all fields in LDS and one vertex of a colour per thread the
// levels 32^2 .. 2^2 took 81 us a call and 64^2 two launches of 13 and 16 us.
constexpr int kSmall2MaxN = 64, kSmall2MaxLevels = 6;

// Inverse of the coarsest operator (N in {2, 3}: 1 or 4 unknowns, padded to
// 4 with the identity), by Gauss-Jordan in one thread, once per coefficient
// set.
template <bool HARM>
__global__ void k2_coarse_inverse(const double* __restrict__ D, const double* __restrict__ mu, int N, Stencil<double> st,
                                  double* __restrict__ inv) {
    if (threadIdx.x != 0) return;
    const int n = N + 1, m1 = N - 1, m = m1 * m1;
    double M[4][4], R[4][4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
#pragma unroll
        for (int c = 0; c < 4; c++) {
            M[t][c] = t == c ? 1.0 : 0.0;
            R[t][c] = t == c ? 1.0 : 0.0;
        }
        if (t < m) {
            const int x = 1 + t / m1, y = 1 + t % m1, v = x * n + y;
            const double cxm = face<HARM>(D[v], D[v - n], st), cxp = face<HARM>(D[v], D[v + n], st);
            const double cym = face<HARM>(D[v], D[v - 1], st), cyp = face<HARM>(D[v], D[v + 1], st);
            M[t][t] = mu[v] + ((cxm + cxp) + (cym + cyp));
            if (m == 4) {   // unknowns (1,1), (1,2), (2,1), (2,2)
                M[t][t ^ 2] = -((t & 2) ? cxm : cxp);
                M[t][t ^ 1] = -((t & 1) ? cym : cyp);
            }
        }
    }
#pragma unroll
    for (int p = 0; p < 4; p++) {
        const double ip = 1.0 / M[p][p];
#pragma unroll
        for (int c = 0; c < 4; c++) {
            M[p][c] *= ip;
            R[p][c] *= ip;
        }
#pragma unroll
        for (int t = 0; t < 4; t++) {
            if (t == p) continue;
            const double f = M[t][p];
#pragma unroll
            for (int c = 0; c < 4; c++) {
                M[t][c] -= f * M[p][c];
                R[t][c] -= f * R[p][c];
            }
        }
    }
#pragma unroll
    for (int t = 0; t < 16; t++) inv[t] = R[t >> 2][t & 3];
}

struct Small2Args {
    const double* q;                          // right-hand side of level ks
    double* u;                                // its correction (interior written)
    const double* D[kSmall2MaxLevels];
    const double* mu[kSmall2MaxLevels];
    Stencil<double> st[kSmall2MaxLevels];
    int N[kSmall2MaxLevels];
    int nl;                                   // levels ks .. L-1
    const double* cinv;                       // inverse of the coarsest operator (4 x 4, padded with the identity)
    int nu_pre, nu_post, first;               // first: colour of the first half-sweep
};

// LDS: quadrant o of block (bx, by) at off + o kS2S + bx kS2X + by.  What
// lies past a row's last block is on the boundary (an unused entry, or the
// next row's first vertex), a row of zeros follows the last.  The coarser
// levels share one more set of quadrants, each in a corner of it.
constexpr int kS2X = 32, kS2S = kS2X * 33, kS2Words = 2 * 4 * kS2S;
__host__ __device__ constexpr int small2_off(int level) {
    return level == 0 ? 0 : 4 * kS2S + (level == 1 ? 0 : level == 2 ? 20 : level == 3 ? 10 * kS2X + 20 : level == 4 ? 16 * kS2X + 20 : 20 * kS2X + 20);
}
__device__ __forceinline__ int small2_at(int off, int x, int y) {
    return off + (2 * (x & 1) + (y & 1)) * kS2S + (x >> 1) * kS2X + (y >> 1);
}
constexpr size_t kSmall2Lds = (kS2Words + 16) * sizeof(double);

template <bool HARM>
__global__ __launch_bounds__(1024) void k2_small_vcycle(Small2Args a) {
    extern __shared__ double lds2[];
    double* const base = lds2;
    double* const sinv = lds2 + kS2Words;    // inverse of the coarsest operator, at most 4 x 4
    const int tid = threadIdx.x, L = a.nl, first = a.first;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // this thread's blocks: A of level 0, B of level lb
    const int lb = wave < 4 ? 1 : wave - 2;
    const int sb = lb == 1 ? 4 : lb == 2 ? 3 : lb == 3 ? 2 : 1;
    const int ax = tid >> 5, ay = tid & 31;
    const int bx = (lb == 1 ? tid : tid & 63) >> sb, by = tid & ((1 << sb) - 1);
    const bool actA = ax < a.N[0] / 2 && ay < a.N[0] / 2;
    const bool hasB = lb < L - 1;
    const int lB = hasB ? lb : 0;
    const bool actB = hasB && bx < a.N[lB] / 2 && by < a.N[lB] / 2;
    const int idA = small2_off(0) + ax * kS2X + ay, idB = small2_off(lB) + (hasB ? bx * kS2X + by : 0);
    Block2 A, B;
    {
        // D, mua and q of both blocks, and the D past the end of each axis
        auto load = [&](const double* p, int N, int x, int y, bool on, double none, double* v) {
#pragma unroll
            for (int o = 0; o < 4; o += 2) {
                const Pair2 t = on ? *reinterpret_cast<const Pair2*>(p + (2 * x + (o >> 1)) * (N + 1) + 2 * y) : Pair2{none, none};
                v[o] = t.a;
                v[o + 1] = t.b;
            }
        };
        auto edges = [&](const double* p, int N, int x, int y, bool on, double* e) {
            const int n = N + 1;
#pragma unroll
            for (int k = 0; k < 2; k++) {
                e[k] = on && x == N / 2 - 1 ? p[N * n + 2 * y + k] : 0.0;
                e[2 + k] = on && y == N / 2 - 1 ? p[(2 * x + k) * n + N] : 0.0;
            }
        };
        double DA[4], mA[4], eA[4], DB[4], mB[4], eB[4];
        load(a.D[0], a.N[0], ax, ay, actA, 1.0, DA);
        load(a.mu[0], a.N[0], ax, ay, actA, 1.0, mA);
        load(a.q, a.N[0], ax, ay, actA, 0.0, A.q);
        edges(a.D[0], a.N[0], ax, ay, actA, eA);
        load(a.D[lB], a.N[lB], bx, by, actB, 1.0, DB);
        load(a.mu[lB], a.N[lB], bx, by, actB, 1.0, mB);
        edges(a.D[lB], a.N[lB], bx, by, actB, eB);
        for (int i = tid; i < kS2Words; i += 1024) base[i] = 0.0;
        if (tid < 16) sinv[tid] = a.cinv[tid];
        __syncthreads();
        auto put = [&](int id, int N, int x, int y, bool on, const double* D, const double* e) {
            // the low y faces' D is only boundary vertices' neighbour
#pragma unroll
            for (int o = 0; o < 4; o++)
                if (on && (y > 0 || (o & 1))) base[id + o * kS2S] = D[o];
#pragma unroll
            for (int k = 0; k < 2; k++) {
                if (on && x == N / 2 - 1) base[id + k * kS2S + kS2X] = e[k];
                if (on && y == N / 2 - 1) base[id + 2 * k * kS2S + 1] = e[2 + k];
            }
        };
        put(idA, a.N[0], ax, ay, actA, DA, eA);
        put(idB, a.N[lB], bx, by, actB, DB, eB);
        __syncthreads();
        auto keep = [&](int x, int y, bool on, bool* k) {
#pragma unroll
            for (int o = 0; o < 4; o++) k[o] = on && (x > 0 || (o & 2)) && (y > 0 || (o & 1));
        };
        bool kA[4], kB[4];
        keep(ax, ay, actA, kA);
        keep(bx, by, actB, kB);
        A.coefs<HARM, kS2S, kS2X>(base, idA, DA, mA, kA, a.st[0]);
        if (hasB) B.coefs<HARM, kS2S, kS2X>(base, idB, DB, mB, kB, a.st[lB]);
        __syncthreads();
        // the vertices past the end are boundary: 0 from here on
        const double zero[4] = {0.0, 0.0, 0.0, 0.0};
        put(idA, a.N[0], ax, ay, actA, zero, zero);
        put(idB, a.N[lB], bx, by, actB, zero, zero);
    }
    // levels 0 and 1 are shared by several waves: their steps end with a
    // workgroup barrier, which every wave joins
    auto sync = [&](int l) {
        if (l <= 1) {
            __syncthreads();
        } else if (lb == l) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    };
    auto sweeps = [&](int l, bool run, Block2& P, int id, int count, bool skip1) {
        for (int c = 0; c < 2 * count; c++) {
            if (skip1 && c == 0) continue;
            if (run) {
                if (((c & 1) ? 1 - first : first)) P.half<1, kS2S, kS2X, false>(base, id);
                else P.half<0, kS2S, kS2X, false>(base, id);
            }
            sync(l);
        }
    };
    auto down = [&](int l, bool run, Block2& P, int id, int x, int y) {
        if (run) {
            // from zero the first half-sweep is u = w q on the first colour
#pragma unroll
            for (int o = 0; o < 4; o++) {
                if (l > 0) P.q[o] = base[id + o * kS2S];
                P.u[o] = (a.nu_pre > 0 && (__builtin_popcount(o) & 1) == first) ? P.w[o] * P.q[o] : 0.0;
            }
#pragma unroll
            for (int o = 0; o < 4; o++) base[id + o * kS2S] = P.u[o];
        }
        sync(l);
        sweeps(l, run, P, id, a.nu_pre, true);
        double r[4] = {};
        if (run) {
            if (a.nu_pre == 0) {
#pragma unroll
                for (int o = 0; o < 4; o++) r[o] = P.w[o] == 0.0 ? 0.0 : P.q[o];
            } else if (first) {
                P.residual<1, kS2S, kS2X>(base, id, r);
            } else {
                P.residual<0, kS2S, kS2X>(base, id, r);
            }
        }
        sync(l);
        if (run) {
#pragma unroll
            for (int o = 0; o < 4; o++) base[id + o * kS2S] = r[o];
        }
        sync(l);
        if (run && x > 0 && y > 0)
            base[small2_at(small2_off(l + 1), x, y)] = Block2::restricted<kS2S, kS2X>(base, id);
        __syncthreads();
    };
    auto up = [&](int l, bool run, Block2& P, int id, int x, int y) {
        if (run) {
            double E[4];
#pragma unroll
            for (int o = 0; o < 4; o++) E[o] = base[small2_at(small2_off(l + 1), x + (o >> 1), y + (o & 1))];
            const double e[4] = {E[0], 0.5 * (E[0] + E[1]), 0.5 * (E[0] + E[2]), 0.25 * ((E[0] + E[2]) + (E[1] + E[3]))};
#pragma unroll
            for (int o = 0; o < 4; o++) {
                if (P.w[o] != 0.0) P.u[o] += e[o];
                base[id + o * kS2S] = P.u[o];
            }
        }
        sync(l);
        sweeps(l, run, P, id, a.nu_post, false);
        if (l > 1) __syncthreads();   // the finer level's waves read the result
    };
    down(0, actA, A, idA, ax, ay);
    for (int l = 1; l < L - 1; l++) down(l, actB && lb == l, B, idB, bx, by);
    {
        const int N = a.N[L - 1], m1 = N - 1, m = m1 * m1, off = small2_off(L - 1);
        if (tid < m) {
            double acc = 0.0;
            for (int c = 0; c < m; c++) acc += sinv[4 * tid + c] * base[small2_at(off, 1 + c / m1, 1 + c % m1)];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            base[small2_at(off, 1 + tid / m1, 1 + tid % m1)] = acc;
        }
        __syncthreads();
    }
    for (int l = L - 2; l >= 1; l--) up(l, actB && lb == l, B, idB, bx, by);
    up(0, actA, A, idA, ax, ay);
    if (actA) {
#pragma unroll
        for (int o = 0; o < 4; o++)
            if (A.w[o] != 0.0) a.u[(2 * ax + (o >> 1)) * (a.N[0] + 1) + 2 * ay + (o & 1)] = A.u[o];
    }
}

// ---------------------------------------------------------------------------
// A whole smoothing phase of a mid-size level in one launch: one workgroup
// per tile, the tile and a ring around it as NB x NB register blocks.
//   MODE 0 / 1 (pre-smoothing from u_in / from zero): two red-black sweeps
//     from a ring of 6 leave u final on the tile plus a ring of 2; the pass
//     writes u on the tile and the restricted defect qc = R (q - A u) of its
//     coarse vertices.
//   MODE 2 (post-smoothing): u_in + I ec (bilinear, the weights of
//     k2_prolong_add), two sweeps from a ring of 4, u on the tile.
// Every block of the box is updated in all four half-sweeps.  A vertex j
// rings inside the box has the sequential sweeps' value after half-sweep j;
// what is formed nearer to the edge, from neighbours the box does not hold,
// is finite and read by nothing that is kept.  Only interior grid vertices
// are updated or written.
//
// Bound by latency up to 512^2 (one round of workgroups: load, four
// half-sweeps, store) and above by the loads of the box.  Measured
// (pre- / post-smoothing): 128^2 .. 512^2 5 us each, 1024^2 13 / 13 us, 4096^2
// 172 / 151 us (3.9 / 4.4 TB/s of one read of u, q, D, mua and one write of u).
// Holding u, q, D and mua in LDS and dividing by the diagonal in every update
// took 14 / 17 us at 128^2 .. 512^2 and 35 / 40 us at 1024^2; the row-marching
// passes 84 / 62 us at 2048^2 and 242 / 192 us at 4096^2 (with the separate
// restriction).
//
// 22 x 22 blocks: with 32 x 32 (1.5 instead of 1.9 times the tile loaded, 1024
// threads) too few workgroups share a CU to overlap one's loads with
// another's half-sweeps, 14 -> 17 us at 1024^2 and 172 -> 233 us at 4096^2.
constexpr int kNb2 = 22;
constexpr int kB2X = kNb2 + 2, kB2S = kB2X * (kNb2 + 2);        // LDS strides: one unused block on every side
constexpr int kB2Threads = (kNb2 * kNb2 + 63) / 64 * 64;
__host__ __device__ constexpr int block2_ring(int mode) { return mode == 2 ? 4 : 6; }
__host__ __device__ constexpr int block2_tile(int mode) { return 2 * kNb2 - 2 * block2_ring(mode); }

template <bool HARM, int MODE>
__global__ __launch_bounds__(kB2Threads) void k2_block_pass(
    const double* __restrict__ uin, double* __restrict__ uout, const double* __restrict__ q, const double* __restrict__ D,
    const double* __restrict__ mu, const double* __restrict__ ec, double* __restrict__ qc, int N, Stencil<double> st,
    int first, int ntx) {
    constexpr int kB2 = block2_tile(MODE), kH2 = block2_ring(MODE);
    __shared__ double base[4 * kB2S];
    const int tid = threadIdx.x;
    const bool act = tid < kNb2 * kNb2;
    const int lx = act ? tid / kNb2 : 0, ly = act ? tid % kNb2 : 0;
    const int tile_id = xcd_remap(blockIdx.x, gridDim.x), tx = tile_id / ntx, ty = tile_id % ntx;
    const int gx = tx * kB2 - kH2 + 2 * lx, gy = ty * kB2 - kH2 + 2 * ly;   // the corner (even)
    const int n = N + 1, Nc = N / 2, nc = Nc + 1;
    const int id = (lx + 1) * kB2X + ly + 1;
    Block2 P;
    bool in[4], keep[4];
#pragma unroll
    for (int o = 0; o < 4; o++) {
        const int x = gx + (o >> 1), y = gy + (o & 1);
        in[o] = act && x >= 0 && x <= N && y >= 0 && y <= N;
        keep[o] = act && interior2(N, x, y);
    }
    {
        // rows of the block as 16-byte loads (8-byte aligned); vertices outside
        // the grid: a clamped read, replaced.  At y = N the pair read is
        // (N - 1, N).
        const int yc = min(max(gy, 0), N - 1);
        const int g0 = min(max(gx, 0), N) * n + yc, g1 = min(max(gx + 1, 0), N) * n + yc;
        auto load = [&](const double* p, double* v) {
            const Pair2 r0 = *reinterpret_cast<const Pair2*>(p + g0), r1 = *reinterpret_cast<const Pair2*>(p + g1);
            v[0] = gy == N ? r0.b : r0.a;
            v[1] = r0.b;
            v[2] = gy == N ? r1.b : r1.a;
            v[3] = r1.b;
        };
        double Dv[4], mv[4];
        load(D, Dv);
        load(mu, mv);
        load(q, P.q);
        if (MODE == 1) {
#pragma unroll
            for (int o = 0; o < 4; o++) P.u[o] = 0.0;
        } else {
            load(uin, P.u);
        }
        if (MODE == 2) {
            // the block's four coarse neighbours, from the corner's
            const int X0 = min(max(gx >> 1, 0), Nc), X1 = min(X0 + 1, Nc), Y0 = min(max(gy >> 1, 0), Nc), Y1 = min(Y0 + 1, Nc);
            const double e00 = ec[X0 * nc + Y0], e01 = ec[X0 * nc + Y1], e10 = ec[X1 * nc + Y0], e11 = ec[X1 * nc + Y1];
            const double e[4] = {e00, 0.5 * (e00 + e01), 0.5 * (e00 + e10), 0.25 * ((e00 + e10) + (e01 + e11))};
#pragma unroll
            for (int o = 0; o < 4; o++) P.u[o] += keep[o] ? e[o] : 0.0;
        }
        for (int i = tid; i < 4 * kB2S; i += kB2Threads) base[i] = 1.0;   // any finite D > 0 beyond the box
        __syncthreads();
#pragma unroll
        for (int o = 0; o < 4; o++) {
            if (!in[o]) P.u[o] = P.q[o] = 0.0;
            if (act) base[id + o * kB2S] = Dv[o];
        }
        __syncthreads();
        P.coefs<HARM, kB2S, kB2X>(base, id, Dv, mv, keep, st);
        __syncthreads();
    }
    if (act) {
#pragma unroll
        for (int o = 0; o < 4; o++) base[id + o * kB2S] = P.u[o];
    }
    __syncthreads();
    for (int j = 0; j < 4; j++) {
        if (act) {
            if ((j & 1) ? !first : first) P.half<1, kB2S, kB2X, true>(base, id);
            else P.half<0, kB2S, kB2X, true>(base, id);
        }
        __syncthreads();
    }
    constexpr int H = kH2 / 2, T = kB2 / 2;   // ring and tile in blocks
    const bool tile = lx >= H && lx < H + T && ly >= H && ly < H + T;
#pragma unroll
    for (int o = 0; o < 4; o++)
        if (tile && keep[o]) uout[(gx + (o >> 1)) * n + gy + (o & 1)] = P.u[o];
    if (MODE == 2) return;
    // restriction of the defect: a coarse vertex is the corner of its block
    double r[4] = {};
    if (act) {
        if (first) P.residual<1, kB2S, kB2X>(base, id, r);
        else P.residual<0, kB2S, kB2X>(base, id, r);
    }
    __syncthreads();
    if (act) {
#pragma unroll
        for (int o = 0; o < 4; o++) base[id + o * kB2S] = r[o];
    }
    __syncthreads();
    if (tile && keep[0]) qc[(gx >> 1) * nc + (gy >> 1)] = Block2::restricted<kB2S, kB2X>(base, id);
}

}  // namespace dmgs
