// Fused coarse-level smoothing: one launch runs a whole smoothing phase of a
// coarse level (up to two red/black steps, four half-sweeps) on bricks held
// in LDS, together with the transfer next to it.
#pragma once

#include "kernels.hpp"

#include <type_traits>

namespace ibm {

// ---------------------------------------------------------------- bricks
// A block owns 8 x 8 x 8 cells of the level and works on the 16 x 16 x 16
// region around them.  Every half-sweep spoils one layer of the region, so
// after a phase's dependency depth (four layers) the brick's own cells hold
// what sweeps over the whole level would give: no exchange between blocks,
// and one launch for the level's mean, four half-sweeps and the restriction
// (or the prolongation and four half-sweeps).
//
// Bound: launches and latency.  A launch costs about 4 us on these levels
// whatever it does (a 64^3 half-sweep moves 4 MB), so the eightfold
// recomputation is free while the chip is not full.  FP64, per phase, one
// launch against the launches it replaces: 16^3 10 us against 28 down and 23
// up, 32^3 10 against 26 and 22, 64^3 19 against 29 and 23.  Above
// BRICK_MAX_CELLS recomputing costs more than launching and the one-sweep
// kernels run.  A 128^3 FP64 V-cycle went from 555 to 449 us.
//
// 512 threads; thread (h, j, k mod 4) keeps four planes' cell pairs (one of
// each colour at half-index h): right-hand sides, face coefficients and
// diagonals in registers, only the iterate in LDS (32 KB in FP64).  The sweeps
// have no branches (four cells' loads in flight per thread: 1.1 to 0.6 us).
constexpr int BR_T = 512;
constexpr int BR_U = 4;                 // planes per thread
constexpr int BR_C = 16 * 16 * 8;       // region slots per colour
enum { BR_ZERO = 0, BR_PROLONG = 1, BR_PLAIN = 2 };

struct Brick {
    int gx, gy, gz, nb;  // bricks per axis; launched blocks (multiple of 8)
};
inline Brick make_brick(int nx, int ny, int nz)
{
    Brick g;
    g.gx = (nx + 7) / 8;
    g.gy = (ny + 7) / 8;
    g.gz = (nz + 7) / 8;
    g.nb = (g.gx * g.gy * g.gz + 7) / 8 * 8;
    return g;
}

template <class T, class TB>
struct BrickArgs {
    const TB *b;            // this level's RHS
    const T *xin;           // black iterate the phase starts from (not read from zero)
    T *xr, *xb;             // red (may be null) and black results; xb is not xin
    const T *xc;            // BR_PROLONG: the coarse iterate
    TB *bc;                 // BR_ZERO: coarse RHS to restrict into (null: no restriction)
    const double *part;     // BR_ZERO: partial sums of this level's mean (null: the mean is at *mean)
    int npart;
    double vol;             // active volume of this level
    double *mean;           // this level's mean; written by block 0 when part is given
    double *pout;           // partial sums of the coarse mean, one per block
    int steps;              // red/black steps (1 or 2)
    int renorm;             // the coarse level has inactive cells
};

template <class T, class TB, int MODE>
__global__ void __launch_bounds__(BR_T) k_brick(Lv L, Brick G, Lv C, PMap M, BrickArgs<T, TB> A)
{
    // the iterate, with a plane of padding on either side: neighbours of the
    // region's outer cells are read (and their results dropped), not tested for
    __shared__ T xsm[2][BR_C + 256];
    __shared__ double aux[MODE == BR_PROLONG ? 1000 : 256];    // coarse values; restriction sums
    __shared__ uint8_t ca[MODE == BR_PROLONG ? 1000 : 1];      // coarse activity
    const int blk = (int)(blockIdx.x & 7) * (G.nb >> 3) + (int)(blockIdx.x >> 3);
    const int bx = blk % G.gx, by = (blk / G.gx) % G.gy, bz = blk / (G.gx * G.gy);
    if (bz >= G.gz) {
        if (MODE == BR_ZERO && A.bc && threadIdx.x == 0) A.pout[blockIdx.x] = 0.0;
        return;
    }
    const int t = threadIdx.x;
    T *const xs[2] = {&xsm[0][128], &xsm[1][128]};             // slot t + 512 u: the thread's cell of plane u
    const int hl = t & 7, jl = (t >> 3) & 15;
    const int kq = __builtin_amdgcn_readfirstlane(t >> 7);     // k_local = kq + 4 u: one plane per wave and u
    const int h = 4 * bx - 2 + hl, j = 8 * by - 4 + jl, k0 = 8 * bz - 4;
    const bool hj = h >= 0 && h < L.H && j >= 0 && j < L.ny;
    const int par = (jl + kq) & 1;                             // parity of i of the red cell
    const long long pl = (long long)L.H * L.ny;
    const long long col = h + (long long)L.H * j;
    // every load of the block's set-up goes out before any is used
    double msum = 0.0;
    const bool sum_mean = MODE == BR_ZERO && A.part != nullptr;
    if (sum_mean)
        for (int q = t; q < A.npart; q += BR_T) msum += A.part[q];
    else
        msum = *A.mean;
    double bm[2][BR_U];
    uint32_t fm[2][BR_U];
    T xi[BR_U];
    double czp[BR_U], czm[BR_U];
#pragma unroll
    for (int u = 0; u < BR_U; ++u) {
        const int k = k0 + kq + 4 * u;
        const bool in = hj && k >= 0 && k < L.nz;
        const long long s = in ? col + pl * k : 0;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t f = L.f[c * L.Nh + s];
            bm[c][u] = ld(A.b, c * L.Nh + s);
            fm[c][u] = in ? f : 0u;                            // nothing is active outside the level
        }
        if (MODE != BR_ZERO) xi[u] = A.xin[s];
        czp[u] = L.cp[2][min(max(k, 0), L.nz - 1)];
        czm[u] = L.cm[2][min(max(k, 0), L.nz - 1)];
    }
    double cpx[2], cmx[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int i = 2 * h + (c ? 1 - par : par), ii = hj && i < L.nx ? i : 0;
        cpx[c] = L.cp[0][ii];
        cmx[c] = L.cm[0][ii];
    }
    const double cpy = L.cp[1][hj ? j : 0], cmy = L.cm[1][hj ? j : 0];
    // black cells' places between the coarse nodes: a cell's lower node is its
    // parent or the one before it, so it is among the region's ten per axis
    int qI = 0, qK[BR_U];
    double tx = 0.0, ty = 0.0, tz[BR_U];
    if constexpr (MODE == BR_PROLONG) {
        const int i = 2 * h + 1 - par, ii = hj && i < L.nx ? i : 0, jj = hj ? j : 0;
        qI = (M.pi[0][ii] - (4 * bx - 3)) + 10 * (M.pi[1][jj] - (4 * by - 3));
        tx = M.pt[0][ii];
        ty = M.pt[1][jj];
#pragma unroll
        for (int u = 0; u < BR_U; ++u) {
            const int k = k0 + kq + 4 * u, kk = min(max(k, 0), L.nz - 1);
            qK[u] = 100 * (M.pi[2][kk] - (4 * bz - 3));
            tz[u] = M.pt[2][kk];
        }
        // the coarse region: parents of the region's cells and one layer more
        const int I0 = 4 * bx - 3, J0 = 4 * by - 3, K0 = 4 * bz - 3;
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const int q = t + BR_T * w;
            const int I = I0 + q % 10, J = J0 + (q / 10) % 10, K = K0 + q / 100;
            const bool in = q < 1000 && I >= 0 && I < C.nx && J >= 0 && J < C.ny && K >= 0 && K < C.nz;
            const long long sc = in ? slot(C, (I + J + K) & 1, I >> 1, J, K) : 0;
            const uint8_t a = C.f[sc] & 1;
            const double v = ld(A.xc, sc);
            if (q < 1000) {
                ca[q] = in ? a : 0;
                aux[q] = in && a ? v : 0.0;
            }
        }
    }
    // coefficients of the open faces, the diagonal and its reciprocal (zero
    // for a cell without an open face, which then becomes zero)
    double cf[2][BR_U][6], dg[2][BR_U], rd[2][BR_U];
    bool act[2][BR_U];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int u = 0; u < BR_U; ++u) {
            const uint32_t f = fm[c][u];
            cf[c][u][0] = (f & CM_PX) ? cpx[c] : 0.0;
            cf[c][u][1] = (f & CM_MX) ? cmx[c] : 0.0;
            cf[c][u][2] = (f & CM_PY) ? cpy : 0.0;
            cf[c][u][3] = (f & CM_MY) ? cmy : 0.0;
            cf[c][u][4] = (f & CM_PZ) ? czp[u] : 0.0;
            cf[c][u][5] = (f & CM_MZ) ? czm[u] : 0.0;
            dg[c][u] = cf[c][u][0] + cf[c][u][1] + cf[c][u][2] + cf[c][u][3] + cf[c][u][4] + cf[c][u][5];
            act[c][u] = (f & CM_ACT) != 0;
            rd[c][u] = dg[c][u] > 0.0 ? 1.0 / dg[c][u] : 0.0;
        }
    double mu = msum;
    if (sum_mean) {
        __shared__ double sm[BR_T / 64];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) msum += __shfl_xor(msum, o, 64);
        if ((t & 63) == 0) sm[t >> 6] = msum;
        __syncthreads();
        mu = 0.0;
#pragma unroll
        for (int w = 0; w < BR_T / 64; ++w) mu += sm[w];
        mu = A.vol > 0.0 ? mu / A.vol : 0.0;
        if (blk == 0 && t == 0) *A.mean = mu;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int u = 0; u < BR_U; ++u) bm[c][u] -= mu;

    auto nbs = [&](int c, int u) {
        const T *xo = xs[1 - c] + (t + BR_T * u);
        const int p = c ? 1 - par : par;
        const T v0 = xo[p], v1 = xo[p - 1], v2 = xo[8], v3 = xo[-8], v4 = xo[128], v5 = xo[-128];
        return cf[c][u][0] * (double)v0 + cf[c][u][1] * (double)v1 + cf[c][u][2] * (double)v2 + cf[c][u][3] * (double)v3 +
               cf[c][u][4] * (double)v4 + cf[c][u][5] * (double)v5;
    };
    // one half-sweep over the cells at least `lay` layers inside the region
    const int il[2] = {2 * hl + par, 2 * hl + 1 - par};
    auto sweep = [&](auto cc, int lay) {
        constexpr int c = decltype(cc)::value;
        const bool ij = il[c] >= lay && il[c] < 16 - lay && jl >= lay && jl < 16 - lay;
        double nb[BR_U];
#pragma unroll
        for (int u = 0; u < BR_U; ++u) nb[u] = nbs(c, u);
#pragma unroll
        for (int u = 0; u < BR_U; ++u) {
            const int kl = kq + 4 * u;
            const double v = quot(nb[u] - bm[c][u], dg[c][u], rd[c][u]);
            if (ij && act[c][u] && kl >= lay && kl < 16 - lay) xs[c][t + BR_T * u] = (T)v;
        }
        __syncthreads();
    };
    constexpr std::integral_constant<int, 0> RED{};
    constexpr std::integral_constant<int, 1> BLACK{};

    int lay = 1;
    if constexpr (MODE == BR_ZERO) {
        // first red half-sweep from zero: the diagonal alone; everything else starts at zero
#pragma unroll
        for (int u = 0; u < BR_U; ++u) {
            xs[0][t + BR_T * u] = (T)(act[0][u] ? quot(0.0 - bm[0][u], dg[0][u], rd[0][u]) : 0.0);
            xs[1][t + BR_T * u] = (T)0;
        }
        __syncthreads();
        sweep(BLACK, lay++);
        if (A.steps > 1) {
            sweep(RED, lay++);
            sweep(BLACK, lay++);
        }
    } else {
        if constexpr (MODE == BR_PROLONG) {
            __syncthreads();  // the staged coarse region
            // trilinear correction of the black cells over the active coarse nodes
#pragma unroll
            for (int u = 0; u < BR_U; ++u) {
                const int q = (fm[1][u] & CM_ACT) ? qI + qK[u] : 0;
                auto tri = [&](auto &&v) {
                    auto line = [&](int e) { return (1 - tx) * v(q + e) + tx * v(q + e + 1); };
                    return (1 - tz[u]) * ((1 - ty) * line(0) + ty * line(10)) +
                           tz[u] * ((1 - ty) * line(100) + ty * line(110));
                };
                double num = tri([&](int e) { return aux[e]; });
                if (A.renorm) {
                    const double den = tri([&](int e) { return (double)ca[e]; });
                    num = den > 0.0 ? num / den : 0.0;
                }
                if (fm[1][u] & CM_ACT) xi[u] = (T)((double)xi[u] + num);
            }
        }
#pragma unroll
        for (int u = 0; u < BR_U; ++u) {
            xs[0][t + BR_T * u] = (T)0;
            xs[1][t + BR_T * u] = fm[1][u] ? xi[u] : (T)0;
        }
        __syncthreads();
        for (int it = 0; it < A.steps; ++it) {
            sweep(RED, lay++);
            sweep(BLACK, lay++);
        }
    }
    // results of the brick's own cells (whole half-index pairs)
    const bool own = hl >= 2 && hl < 6 && jl >= 4 && jl < 12 && hj;
#pragma unroll
    for (int u = 0; u < BR_U; ++u) {
        const int kl = kq + 4 * u, k = k0 + kl;
        if (!own || kl < 4 || kl >= 12 || k >= L.nz) continue;
        A.xb[col + pl * k] = xs[1][t + BR_T * u];
        if (A.xr) A.xr[col + pl * k] = xs[0][t + BR_T * u];
    }
    if constexpr (MODE == BR_ZERO) {
        if (!A.bc) return;
        // residual of the own cells, volume-weighted and summed over the pair
        const double wj = hj ? L.w[1][j] : 0.0;
#pragma unroll
        for (int u = 0; u < BR_U; ++u) {
            const int kl = kq + 4 * u, k = k0 + kl;
            if (!own || kl < 4 || kl >= 12) continue;
            double sum = 0.0;
            if (k < L.nz) {
                const double wjk = wj * L.w[2][k];
#pragma unroll
                for (int e = 0; e < 2; ++e) {  // i = 2h + e
                    const bool red = e == par;
                    const double r0 = bm[0][u] - (nbs(0, u) - dg[0][u] * (double)xs[0][t + BR_T * u]);
                    const double r1 = bm[1][u] - (nbs(1, u) - dg[1][u] * (double)xs[1][t + BR_T * u]);
                    if ((red ? fm[0][u] : fm[1][u]) & CM_ACT) sum += L.w[0][2 * h + e] * wjk * (red ? r0 : r1);
                }
            }
            aux[(hl - 2) + 4 * ((jl - 4) + 8 * (kl - 4))] = sum;
        }
        // rows and planes outside the level carry nothing
        if (!hj && hl >= 2 && hl < 6 && jl >= 4 && jl < 12)
#pragma unroll
            for (int u = 0; u < BR_U; ++u) {
                const int kl = kq + 4 * u;
                if (kl >= 4 && kl < 12) aux[(hl - 2) + 4 * ((jl - 4) + 8 * (kl - 4))] = 0.0;
            }
        __syncthreads();
        if (t < 64) {
            const int I = 4 * bx + (t & 3), J = 4 * by + ((t >> 2) & 3), K = 4 * bz + (t >> 4);
            double v = 0.0;
            if (I < C.nx && J < C.ny && K < C.nz) {
                const int q = (t & 3) + 4 * (2 * ((t >> 2) & 3) + 8 * (2 * (t >> 4)));
                const double svr = aux[q] + aux[q + 4] + aux[q + 32] + aux[q + 36];
                const long long sc = slot(C, (I + J + K) & 1, I >> 1, J, K);
                const double VC = C.w[0][I] * C.w[1][J] * C.w[2][K];
                const bool act = C.f[sc] & 1;  // a coarse cell is active when a child is
                st(A.bc, sc, act ? svr / VC : 0.0);
                v = act ? VC * ld(A.bc, sc) : 0.0;
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            if (t == 0) A.pout[blockIdx.x] = v;
        }
    }
}

}  // namespace ibm
