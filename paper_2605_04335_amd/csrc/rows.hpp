// Half-sweeps of level 0 with the sparse rows in the same launch.
//
// The one-sweep sequence takes three or four launches per half-sweep: the
// regular cells, the membrane-adjacent cells of the colour, the ghost rows'
// Jacobi update into a staging array, and its scatter.  On small grids, and on
// the units around bodies of large ones, each costs a launch (4 us) and little
// else.  Here
//   - ghost values live in arrays of their own, one read and one written per
//     half-sweep, so no scatter separates their update from their use;
//   - regular cells with a ghost neighbour ("adjacent" cells) are a list with
//     coded neighbours, so the other cells' sweep never meets a ghost;
//   - a row that needs the new value of a cell being swept in the same launch
//     computes it again from the other colour, which the launch does not write.
// Without membranes a half-sweep is then one launch.  With membranes the
// ghost rows need the membrane cells' new values: a second launch.  Bound:
// launch and dependent-load latency.  FP64 solve at 32^3: 2205 us before,
// 2010 to 2097 after; V-cycle at 128^3 with a membrane: 440 and 406 us.
#pragma once

#include "walk.hpp"

namespace ibm {

constexpr uint8_t F_ADJ = 0x10;  // solver's own level-0 mask: regular cell with a closed ghost neighbour

// Sparse rows with coded columns: v >= 0 the slot of a cell; -1 absent (a
// wall); otherwise ghost row -2 - v (closed ghosts, then membrane unknowns).
struct Rows {
    long long N2, Nh, pin;
    int ng, nrows, nm, na;
    const int32_t *rslot;          // [ng] slots of the closed ghosts
    const int32_t *code, *rix;     // [nrows*8] columns; the membrane cell behind a cell column (>= 0), its
                                   // place in the adjacent list (-2 - a), or -1
    const double *rw, *rsG;
    const int32_t *mslot, *mcode, *mcolor;  // membrane cells: -x,+x,-y,+y,-z,+z
    const int32_t *aslot, *acode;           // adjacent cells: +x,-x,+y,-y,+z,-z
    __device__ __forceinline__ long long unknown(int g) const
    {
        return g < ng ? (long long)rslot[g] : N2 + (g - ng);
    }
};

// what a launch reads: the iterate, the ghost values (null: at their unknowns
// in the iterate), RHS and sink; zero: everything but the RHS counts as zero
template <class T>
struct RowsIn {
    const T *x, *g, *b;
    const double *sink;
    bool zero;
    __device__ __forceinline__ double cell(long long s) const { return zero ? 0.0 : ld(x, s); }
    __device__ __forceinline__ double ghost(const Rows &R, int r) const
    {
        return zero ? 0.0 : (g ? ld(g, r) : ld(x, R.unknown(r)));
    }
    __device__ __forceinline__ double coded(const Rows &R, int32_t v) const
    {
        return v >= 0 ? cell(v) : (v == -1 ? 0.0 : ghost(R, -2 - v));
    }
    __device__ __forceinline__ double rhs(const Rows &R, long long s) const
    {
        const double v = ld(b, s);
        return s == R.pin && sink ? v - sink[0] : v;
    }
};

// new value of the regular cell (h, j, k) of colour c at slot s (of that colour's array)
template <class T>
__device__ __forceinline__ T plain_new(const Lv &L, const Rows &R, const RowsIn<T> &I, const UnitPos &u, int c, long long s)
{
    double dg, nb = 0.0;
    if (I.zero) {
        const int i = min(2 * u.h + ((c + u.j + u.k) & 1), L.nx - 1);
        dg = L.cp[0][i] + L.cm[0][i] + L.cp[1][u.j] + L.cm[1][u.j] + L.cp[2][u.k] + L.cm[2][u.k];
    } else {
        nb = near_nb(L, u, I.x, c, s, dg);
    }
    return (T)((nb - I.rhs(R, c * L.Nh + s)) / dg);
}
// new value of adjacent cell a
template <class T>
__device__ __forceinline__ T adjacent_new(const Lv &L, const Rows &R, const RowsIn<T> &I, int a)
{
    int c, h, j, k, i;
    const long long s = R.aslot[a];
    decode_slot(L, s, c, h, j, k, i);
    const double cf[6] = {L.cp[0][i], L.cm[0][i], L.cp[1][j], L.cm[1][j], L.cp[2][k], L.cm[2][k]};
    double dg = 0.0, nb = 0.0, v[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) v[q] = I.coded(R, R.acode[6 * (long long)a + q]);
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        nb += cf[q] * v[q];
        dg += cf[q];
    }
    return (T)((nb - I.rhs(R, s)) / dg);
}
// value of a ghost row's column after the half-sweep of colour c over the
// regular cells (membrane cells: still the old value, or mnew's)
template <class T>
__device__ __forceinline__ double column_new(const Lv &L, const Rows &R, const RowsIn<T> &I, int32_t v, int32_t ix, int c)
{
    if (v < 0) return v == -1 ? 0.0 : I.ghost(R, -2 - v);
    if ((v >= L.Nh ? 1 : 0) != c || ix >= 0) return I.cell(v);
    if (ix <= -2) return (double)adjacent_new(L, R, I, -2 - ix);
    UnitPos u;
    int cc, i;
    decode_slot(L, v, cc, u.h, u.j, u.k, i);
    return (double)plain_new(L, R, I, u, c, (long long)v - c * L.Nh);
}
// sum over ghost row r's columns, one of eight lanes each (every lane gets it)
__device__ __forceinline__ double sum8(double v)
{
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    return v + __shfl_xor(v, 4, 64);
}
template <class T>
__device__ __forceinline__ double row_sum_new(const Lv &L, const Rows &R, const RowsIn<T> &I, int r, int t, int c)
{
    const long long q = 8 * (long long)r + t;
    const int32_t v = R.code[q], ix = R.rix[q];
    const double w = R.rw[q];
    return sum8(v == -1 ? 0.0 : w * column_new(L, R, I, v, ix, c));
}

// Blocks of one launch: cells (every cell pair, or the listed units), adjacent
// cells, then the rows (ghost rows, or membrane cells)
struct HalfBlocks {
    int cells, adj, rows;
    int total() const { return cells + adj + rows; }
};

// Half-sweep of colour c over the regular cells.  GHOSTS: with the ghost rows'
// Jacobi update into gnew; otherwise with the membrane cells of the colour
// into mtmp.  ZERO sweeps (I.zero) also zero every other slot they cover.
template <class T, bool UNITS, bool GHOSTS>
__global__ void __launch_bounds__(TPB) k_half(Lv L, Rows R, Near U, HalfBlocks B, RowsIn<T> I, T *x, int c,
                                              T *__restrict__ gnew, double *__restrict__ mtmp)
{
    const int blk = (int)blockIdx.x;
    if (blk < B.cells) {
        UnitPos u{0, 0, 0, false, false, false};
        if constexpr (UNITS) {
            u = unit_pos(U, L);
        } else {
            // consecutive blocks of an XCD take consecutive cells
            const int q = (blk & 7) * (B.cells >> 3) + (blk >> 3);
            const uint32_t p = (uint32_t)q * TPB + threadIdx.x;
            if ((long long)p < L.Nh) {
                const uint32_t row = fdiv(p, L.fH), kk = fdiv(row, L.fy);
                u.h = (int)(p - row * (uint32_t)L.H);
                u.j = (int)(row - kk * (uint32_t)L.ny);
                u.k = (int)kk;
                u.in = true;
            }
        }
        if (!u.in) return;
        const long long s = unit_slot(u, L);
        const uint8_t f = L.f[c * L.Nh + s];
        const bool regular = !(f & (F_SOLID | F_MGHOST));
        if (I.zero) {
            x[c * L.Nh + s] = regular ? plain_new(L, R, I, u, c, s) : (T)0;
            x[(1 - c) * L.Nh + s] = (T)0;
        } else {
            // (on a padding slot's place the neighbours of its pair are read: in range, dropped)
            const T v = plain_new(L, R, I, u, c, s);
            if (regular && !(f & F_ADJ)) x[c * L.Nh + s] = v;
        }
        return;
    }
    if (blk < B.cells + B.adj) {
        const int a = (blk - B.cells) * TPB + (int)threadIdx.x;
        if (a < R.na && (R.aslot[a] >= L.Nh ? 1 : 0) == c) x[R.aslot[a]] = adjacent_new(L, R, I, a);
        return;
    }
    // rows: eight lanes each
    const int r = (blk - B.cells - B.adj) * (TPB / 8) + (int)(threadIdx.x >> 3), t = threadIdx.x & 7;
    if constexpr (GHOSTS) {
        if (r >= R.nrows) return;
        const double bv = ld(I.b, R.unknown(r)), sg = R.rsG[r];
        const double sum = row_sum_new(L, R, I, r, t, c);
        if (t == 0) gnew[r] = (T)(sum - bv / sg);
    } else {
        // membrane cell of the colour: across a cut link the far side's ghost
        // unknown is eliminated, i.e. replaced by its row's current value
        if (r >= R.nm || R.mcolor[r] != c) return;
        const long long s = R.mslot[r];
        const int32_t v = t < 6 ? R.mcode[6 * (long long)r + t] : -1;
        int cc, h, j, k, i;
        decode_slot(L, s, cc, h, j, k, i);
        const int d = t >> 1, at = d == 0 ? i : (d == 1 ? j : k);
        const double cf = v == -1 ? 0.0 : (t & 1 ? L.cp[d][at] : L.cm[d][at]);
        const bool cut = v <= -2 - R.ng;
        double val = cut ? 0.0 : I.coded(R, v);  // the other colour, or a closed ghost
        // the group's cut links one after another, its eight lanes on the columns
        uint32_t m = (uint32_t)(__ballot(cut) >> (threadIdx.x & 56)) & 0xff;
        while (m) {
            const int q = __ffs(m) - 1;
            m &= m - 1;
            const int g = -2 - __shfl(v, (threadIdx.x & 56) + q, 64);
            const double far = row_sum_new(L, R, I, g, t, c) - ld(I.b, R.unknown(g)) / R.rsG[g];
            if (t == q) val = far;
        }
        const double off = sum8(cf * val), dg = sum8(cf);
        if (t == 0) mtmp[r] = (off - ld(I.b, s)) / dg;
    }
}

// second launch of a half-sweep with membranes: the membrane cells' new values
// into x, and the ghost rows from them
template <class T>
__global__ void __launch_bounds__(TPB) k_half_ghosts(Lv L, Rows R, RowsIn<T> I, T *x, int c,
                                                     const double *__restrict__ mtmp, T *__restrict__ gnew)
{
    const int r = (int)(blockIdx.x * TPB + threadIdx.x);
    if (r >= R.nrows) {
        const int m = r - R.nrows;
        if (m < R.nm && R.mcolor[m] == c) st(x, R.mslot[m], mtmp[m]);
        return;
    }
    const double bv = ld(I.b, R.unknown(r)), sg = R.rsG[r];
    int32_t v[8], ix[8];
    double w[8], xv[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        v[t] = R.code[8 * (long long)r + t];
        ix[t] = R.rix[8 * (long long)r + t];
        w[t] = R.rw[8 * (long long)r + t];
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        if (v[t] >= 0) xv[t] = ix[t] >= 0 && (v[t] >= L.Nh ? 1 : 0) == c ? round_to<T>(mtmp[ix[t]]) : (double)x[v[t]];
        else xv[t] = v[t] == -1 ? 0.0 : I.ghost(R, -2 - v[t]);
    }
    double acc = 0.0;
#pragma unroll
    for (int t = 0; t < 8; ++t)
        if (v[t] != -1) acc += w[t] * xv[t];
    gnew[r] = (T)(acc - bv / sg);
}

// after a phase: ghost values to their unknowns in x; with RES also the
// residuals of the sparse cells (closed ghosts, membrane cells) into rsp
template <class T, bool RES>
__global__ void __launch_bounds__(TPB) k_rows_out(Lv L, Rows R, RowsIn<T> I, T *x, T *rsp)
{
    const int r = (int)(blockIdx.x * TPB + threadIdx.x);
    if (r < R.nrows) {
        const T gv = I.g[r];
        const long long u = R.unknown(r);
        if constexpr (RES)
            if (r < R.ng) {  // membrane ghost unknowns are not restricted
                double acc = 0.0;
                for (int t = 0; t < 8; ++t) {
                    const int32_t v = R.code[8 * (long long)r + t];
                    if (v != -1) acc += R.rw[8 * (long long)r + t] * I.coded(R, v);
                }
                st(rsp, u, ld(I.b, u) - R.rsG[r] * (acc - (double)gv));
            }
        x[u] = gv;
        return;
    }
    if constexpr (RES) {
        const int m = r - R.nrows;
        if (m >= R.nm) return;
        const long long s = R.mslot[m];
        int cc, h, j, k, i;
        decode_slot(L, s, cc, h, j, k, i);
        const double cf[6] = {L.cm[0][i], L.cp[0][i], L.cm[1][j], L.cp[1][j], L.cm[2][k], L.cp[2][k]};
        const double xp = I.cell(s);
        double acc = 0.0;
        for (int q = 0; q < 6; ++q) {
            const int32_t v = R.mcode[6 * (long long)m + q];
            if (v != -1) acc += cf[q] * (I.coded(R, v) - xp);
        }
        st(rsp, s, ld(I.b, s) - acc);
    }
}

// ---- set-up of the coded rows
// level-0 mask: regular cells with a closed ghost neighbour
__global__ void __launch_bounds__(TPB) k_mark_adjacent(Lv L, Walk W, uint8_t *f)
{
    WALK_BEGIN(W, p)
        int c, h, j, k, i;
        decode_slot(L, p, c, h, j, k, i);
        if (i >= L.nx || (f[p] & (F_SOLID | F_MGHOST))) continue;
        const uint8_t *fo = f + (long long)(1 - c) * L.Nh;
        const long long s = h + (long long)L.H * (j + (long long)L.ny * k), pl = (long long)L.H * L.ny;
        const int e = i & 1;
        uint8_t g = 0;
        if (i + 1 < L.nx) g |= fo[s + e];
        if (i > 0) g |= fo[s + e - 1];
        if (j + 1 < L.ny) g |= fo[s + L.H];
        if (j > 0) g |= fo[s - L.H];
        if (k + 1 < L.nz) g |= fo[s + pl];
        if (k > 0) g |= fo[s - pl];
        // (a padding slot is solid and no ghost; neighbours' own F_ADJ bits may be in flight, the ghost bit is not)
        if (g & F_GHOST) f[p] |= F_ADJ;
    WALK_END
}

struct CodeMap {
    Lv L;
    const int32_t *gcell, *mcell, *aslot;  // sorted: closed ghost cells and membrane cells (natural), adjacent slots
    int ng, nm, na;
};
__device__ __forceinline__ int sorted_index(const int32_t *a, int n, int32_t v)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        const int m = (lo + hi) >> 1;
        if (a[m] < v) lo = m + 1;
        else hi = m;
    }
    return lo < n && a[lo] == v ? lo : -1;
}
// code of the unknown u (a slot, or a membrane unknown), and what stands behind a cell
__device__ __forceinline__ int32_t code_of(const CodeMap &M, int32_t u, int32_t &ix)
{
    ix = -1;
    if (u < 0) return -1;
    const long long N2 = 2 * M.L.Nh;
    if (u >= N2) return -2 - (M.ng + (int)(u - N2));
    const uint8_t f = M.L.f[u];
    int c, h, j, k, i;
    decode_slot(M.L, u, c, h, j, k, i);
    const int32_t cell = (int32_t)(i + (long long)M.L.nx * (j + (long long)M.L.ny * k));
    if ((f & F_SOLID) && (f & F_GHOST)) return -2 - sorted_index(M.gcell, M.ng, cell);
    if (f & F_MGHOST) ix = sorted_index(M.mcell, M.nm, cell);
    else if (f & F_ADJ) ix = -2 - sorted_index(M.aslot, M.na, u);
    return u;
}
__global__ void __launch_bounds__(TPB) k_code_columns(CodeMap M, long long n, const int32_t *__restrict__ cols,
                                                      int32_t *__restrict__ code, int32_t *__restrict__ rix)
{
    for (long long q = blockIdx.x * (long long)TPB + threadIdx.x; q < n; q += (long long)gridDim.x * TPB) {
        int32_t ix;
        code[q] = code_of(M, cols[q], ix);
        if (rix) rix[q] = ix;
    }
}
__global__ void __launch_bounds__(TPB) k_code_adjacent(CodeMap M, int32_t *__restrict__ acode)
{
    for (long long a = blockIdx.x * (long long)TPB + threadIdx.x; a < M.na; a += (long long)gridDim.x * TPB) {
        const Lv &L = M.L;
        int c, h, j, k, i, ix;
        decode_slot(L, M.aslot[a], c, h, j, k, i);
        const long long s = h + (long long)L.H * (j + (long long)L.ny * k) + (1 - c) * L.Nh, pl = (long long)L.H * L.ny;
        const int e = i & 1;
        const long long nb[6] = {i + 1 < L.nx ? s + e : -1, i > 0 ? s + e - 1 : -1,       j + 1 < L.ny ? s + L.H : -1,
                                 j > 0 ? s - L.H : -1,      k + 1 < L.nz ? s + pl : -1, k > 0 ? s - pl : -1};
        for (int q = 0; q < 6; ++q) acode[6 * a + q] = code_of(M, (int32_t)nb[q], ix);
    }
}

}  // namespace ibm
