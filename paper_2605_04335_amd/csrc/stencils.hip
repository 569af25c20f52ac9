// Ghost-cell boundary rows (Sec. 2.5 module 2) on gfx950.
//
// For every closed ghost cell G (solid with a fluid face neighbour) and every
// membrane ghost cell Q (fluid cell next to a cut link, which carries one
// extra unknown: the field of the far side of the sheet extended to Q):
//   BI  = closest point on the triangles of the same body kind (first
//         triangle on ties), Ericson's Voronoi-region walk;
//   IP  = 2 BI - x_G, dl = 2 |BI - x_G| (image point and its distance);
//   the 8 cell centres around IP (clamped to the centre range) give a
//   trilinear fit: value rows for usable nodes, the Neumann derivative row
//   n . grad b at BI for the node G itself, and "degenerate" for nodes on the
//   wrong side; the weights solve V^T beta = b(IP) by LU with partial
//   pivoting (the batched small inversions of Sec. 2.5);
//   the row is sG (sum beta_k x_k - x_G) = sG (dl - beta_BI) g, scaled like
//   a fluid row; a degenerate box falls back to the mean of the face
//   neighbours on the relevant side.
// Ghost lists are compacted in cell order by a block scan (the array
// compaction of Sec. 2.5).  Compiled with -ffp-contract=off so that distance
// ties and side tests round as written.

#include "common.hpp"

#include <algorithm>
#include <climits>
#include <cmath>

namespace ibm {
void classify(const ibm_grid *, const ibm_body *, int, uint8_t *, ibm_class_stats *, hipStream_t);

namespace {

constexpr int CH = 4096;    // cells per compaction block
constexpr int CB = 256;     // its threads, CH / CB consecutive cells each
constexpr int CMAX = 3;     // lists built together

// ---------------------------------------------------------------- compaction
// Ordered lists of the cells whose flag byte has a given bit, up to three of
// them in one pass: counts per block, one scan, fill.  Bound: the flags, read
// twice.  A thread takes 16 consecutive cells in one load (where the array is
// aligned to it).  At 384^3 three lists one after the other took 3 x 180 us
// of kernels; together they take 85.
struct Bits {
    uint8_t m[CMAX];  // single bits
};

__device__ __forceinline__ uint4 cells16(const uint8_t *flags, long long N, long long p)
{
    if (p + 16 <= N && ((uintptr_t)flags & 15) == 0) return *reinterpret_cast<const uint4 *>(flags + p);
    uint32_t w[4] = {0, 0, 0, 0};
    for (int q = 0; q < 16; ++q)
        if (p + q < N) w[q >> 2] |= (uint32_t)flags[p + q] << (8 * (q & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
}
// bit q set: cell q of the sixteen carries the flag bit m
__device__ __forceinline__ uint32_t hits16(const uint4 &v, uint8_t m)
{
    const uint32_t mm = 0x01010101u * m;
    auto four = [&](uint32_t w) {
        w &= mm;
        return (uint32_t)((w & 0xffu) != 0) | (uint32_t)((w & 0xff00u) != 0) << 1 | (uint32_t)((w & 0xff0000u) != 0) << 2 |
               (uint32_t)((w & 0xff000000u) != 0) << 3;
    };
    return four(v.x) | four(v.y) << 4 | four(v.z) << 8 | four(v.w) << 12;
}

// inclusive prefix sum over the block (blockDim a multiple of 64); *total: the sum
__device__ __forceinline__ int block_prefix(int v, int *total)
{
    __shared__ int ws[16];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    __syncthreads();
    if (lane == 63) ws[wid] = v;
    __syncthreads();
    int before = 0, sum = 0;
    for (int w = 0; w < nw; ++w) {
        if (w < wid) before += ws[w];
        sum += ws[w];
    }
    *total = sum;
    return before + v;
}

__global__ void __launch_bounds__(CB) k_count(const uint8_t *flags, long long N, Bits M, int K, int nb, int *cnt)
{
    const uint4 v = cells16(flags, N, (long long)blockIdx.x * CH + 16 * threadIdx.x);
    for (int q = 0; q < K; ++q) {
        int tot;
        (void)block_prefix(__popc(hits16(v, M.m[q])), &tot);
        if (threadIdx.x == 0) cnt[(long long)q * nb + blockIdx.x] = tot;
    }
}

// exclusive scan of one list's n block counts, in place (one block per list)
__global__ void __launch_bounds__(1024) k_scan(int *cnt, int n, int *total)
{
    int *a = cnt + (long long)blockIdx.x * n;
    int carry = 0;
    for (int i0 = 0; i0 < n; i0 += 1024) {
        const int i = i0 + (int)threadIdx.x, v = i < n ? a[i] : 0;
        int tot;
        const int inc = block_prefix(v, &tot);
        if (i < n) a[i] = carry + inc - v;
        carry += tot;
    }
    if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

struct Lists {
    int32_t *out[CMAX];
};
__global__ void __launch_bounds__(CB) k_fill(const uint8_t *flags, long long N, Bits M, int K, int nb, const int *off,
                                             Lists O)
{
    const long long p = (long long)blockIdx.x * CH + 16 * threadIdx.x;
    const uint4 v = cells16(flags, N, p);
    for (int q = 0; q < K; ++q) {
        uint32_t h = hits16(v, M.m[q]);
        const int c = __popc(h);
        int tot;
        int32_t *o = O.out[q] + off[(long long)q * nb + blockIdx.x] + block_prefix(c, &tot) - c;
        while (h) {
            *o++ = (int32_t)(p + __ffs(h) - 1);
            h &= h - 1;
        }
    }
}

// ---------------------------------------------------------------- geometry
struct V3 {
    double x, y, z;
};
__device__ __forceinline__ V3 sub(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ double dot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ V3 axpy(V3 a, double s, V3 d) { return {a.x + s * d.x, a.y + s * d.y, a.z + s * d.z}; }

// Closest point on triangle (a,b,c) to p: Ericson, Real-Time Collision
// Detection (2005) Sec. 5.1.5, vertex / edge / face Voronoi regions.
__device__ V3 closest_on_triangle(V3 p, V3 a, V3 b, V3 c)
{
    V3 ab = sub(b, a), ac = sub(c, a), ap = sub(p, a);
    double d1 = dot(ab, ap), d2 = dot(ac, ap);
    if (d1 <= 0.0 && d2 <= 0.0) return a;
    V3 bp = sub(p, b);
    double d3 = dot(ab, bp), d4 = dot(ac, bp);
    if (d3 >= 0.0 && d4 <= d3) return b;
    double vc = d1 * d4 - d3 * d2;
    if (vc <= 0.0 && d1 >= 0.0 && d3 <= 0.0) return axpy(a, d1 / (d1 - d3), ab);
    V3 cp = sub(p, c);
    double d5 = dot(ab, cp), d6 = dot(ac, cp);
    if (d6 >= 0.0 && d5 <= d6) return c;
    double vb = d5 * d2 - d1 * d6;
    if (vb <= 0.0 && d2 >= 0.0 && d6 <= 0.0) return axpy(a, d2 / (d2 - d6), ac);
    double va = d3 * d6 - d5 * d4;
    if (va <= 0.0 && (d4 - d3) >= 0.0 && (d5 - d6) >= 0.0) {
        double s = (d4 - d3) / ((d4 - d3) + (d5 - d6));
        return axpy(b, s, sub(c, b));
    }
    double den = 1.0 / (va + vb + vc);
    double v = vb * den, w = vc * den;
    V3 q;
    q.x = a.x + ab.x * v + ac.x * w;
    q.y = a.y + ab.y * v + ac.y * w;
    q.z = a.z + ab.z * v + ac.z * w;
    return q;
}

// The triangles of a body are grouped in runs of TGROUP consecutive ones
// (mesh order) with one box per run, and one box per body.  Closed bodies and
// their runs stand before membranes, in (body, triangle) order within a kind.
constexpr int TGROUP = 32;

struct Run {
    int t0, n;  // first triangle, triangles (at most TGROUP); of a body: first run, runs
};
struct Tris {
    const double *v;    // vertex coordinates of all bodies
    const int32_t *tri; // [nt*3] vertices of the triangles
    const Run *run, *body;
    double *box, *bbox; // [6][runs], [6][bodies]: min xyz, max xyz
    int nr, nb, b0[3];  // first body of each kind, end
};
struct Corner3 {
    V3 a, b, c;
};
__device__ __forceinline__ Corner3 corners(const Tris &T, int t)
{
    const double *a = T.v + 3 * (long long)T.tri[3 * (long long)t], *b = T.v + 3 * (long long)T.tri[3 * (long long)t + 1],
                 *c = T.v + 3 * (long long)T.tri[3 * (long long)t + 2];
    return {{a[0], a[1], a[2]}, {b[0], b[1], b[2]}, {c[0], c[1], c[2]}};
}

struct GridD {
    const double *c[3];  // centres
    const double *w[3];  // widths
    const double *cp[3], *cm[3];
    int n[3];
    double hmin;
};

// least and largest squared distance from p to a point of box i of n
__device__ __forceinline__ double box_lb(const double *bx, int n, int i, V3 p)
{
    const double q[3] = {p.x, p.y, p.z};
    double s = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double lo = bx[(long long)d * n + i], hi = bx[(long long)(d + 3) * n + i];
        const double e = q[d] < lo ? lo - q[d] : (q[d] > hi ? q[d] - hi : 0.0);
        s += e * e;
    }
    return s;
}
__device__ __forceinline__ double box_ub(const double *bx, int n, int i, V3 p)
{
    const double q[3] = {p.x, p.y, p.z};
    double s = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double e = fmax(fabs(q[d] - bx[(long long)d * n + i]), fabs(q[d] - bx[(long long)(d + 3) * n + i]));
        s += e * e;
    }
    return s;
}

__device__ __forceinline__ int box_index(const double *c, int n, double x)
{
    // largest i <= n-2 with c[i] <= x (x within [c0, c_{n-1}])
    int lo = 0, hi = n - 2;
    while (lo < hi) {
        int m = (lo + hi + 1) >> 1;
        if (c[m] <= x) lo = m; else hi = m - 1;
    }
    return lo;
}

__device__ __forceinline__ int find_sorted(const int32_t *a, int n, int32_t v)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        int m = (lo + hi) >> 1;
        if (a[m] < v) lo = m + 1; else hi = m;
    }
    return (lo < n && a[lo] == v) ? lo : -1;
}

struct RowOut {
    int32_t *col;
    double *w, *sG, *dlb, *geo;
    uint8_t *rfl;
};

// boxes of the runs, half a wavefront each
__global__ void __launch_bounds__(256) k_run_boxes(Tris T)
{
    const int r = (int)(blockIdx.x * 256 + threadIdx.x) / TGROUP, t = threadIdx.x % TGROUP;
    if (r >= T.nr) return;
    const Run R = T.run[r];
    const Corner3 C = corners(T, R.t0 + min(t, R.n - 1));
    double lo[3] = {fmin(C.a.x, fmin(C.b.x, C.c.x)), fmin(C.a.y, fmin(C.b.y, C.c.y)), fmin(C.a.z, fmin(C.b.z, C.c.z))};
    double hi[3] = {fmax(C.a.x, fmax(C.b.x, C.c.x)), fmax(C.a.y, fmax(C.b.y, C.c.y)), fmax(C.a.z, fmax(C.b.z, C.c.z))};
    for (int d = 0; d < 3; ++d) {
        for (int o = TGROUP / 2; o > 0; o >>= 1) {
            lo[d] = fmin(lo[d], __shfl_xor(lo[d], o, TGROUP));
            hi[d] = fmax(hi[d], __shfl_xor(hi[d], o, TGROUP));
        }
        if (t == 0) {
            T.box[(long long)d * T.nr + r] = lo[d];
            T.box[(long long)(d + 3) * T.nr + r] = hi[d];
        }
    }
}
// boxes of the bodies, a wavefront each
__global__ void __launch_bounds__(64) k_body_boxes(Tris T)
{
    const int b = (int)blockIdx.x, lane = threadIdx.x;
    const Run R = T.body[b];
    for (int d = 0; d < 3; ++d) {
        double lo = INFINITY, hi = -INFINITY;
        for (int q = lane; q < R.n; q += 64) {
            lo = fmin(lo, T.box[(long long)d * T.nr + R.t0 + q]);
            hi = fmax(hi, T.box[(long long)(d + 3) * T.nr + R.t0 + q]);
        }
        for (int o = 32; o > 0; o >>= 1) {
            lo = fmin(lo, __shfl_xor(lo, o, 64));
            hi = fmax(hi, __shfl_xor(hi, o, 64));
        }
        if (lane == 0) {
            T.bbox[(long long)d * T.nb + b] = lo;
            T.bbox[(long long)(d + 3) * T.nb + b] = hi;
        }
    }
}

// Nearest triangle of each ghost's kind, one wavefront per row: the point into
// geo[0..2], its squared distance into geo[11], the triangle into near (-1:
// none).  Bound: the address unit, by the gathers of boxes and vertices.  One
// thread per row walked them one after the other with too few wavefronts to
// hide the latency: 958 us for 93 thousand rows among 20 bodies, with the
// rows' matrices; now 274, and 24 for the matrices.  (Boxes of all runs, six
// doubles together, without the bodies' level: 541.)
//
// A bound on the nearest squared distance comes first: every box holds a
// triangle at most as far as its farthest point, so the smallest such distance
// is one, over the bodies, then over the runs of the bodies within it, then
// over the triangles of the run that gave it; with a relative margin far above
// rounding.  Then every triangle of every run within the bound, a run to half
// a wavefront.  The smallest distance wins and on equal ones the first
// triangle, as in a plain scan.
__global__ void __launch_bounds__(256) k_nearest(Tris T, GridD G, const int32_t *cells, int r0, int ng, int nrows,
                                                 double *geo, int32_t *near)
{
    const int r = r0 + (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= nrows) return;
    const int32_t cell = cells[r];
    const int nx = G.n[0], ny = G.n[1];
    const V3 P = {G.c[0][cell % nx], G.c[1][(cell / nx) % ny], G.c[2][cell / (nx * ny)]};
    const int want = r >= ng ? 1 : 0, b0 = T.b0[want], b1 = T.b0[want + 1];
    const double margin = 1.0 + 1e-9;
    auto wave_min = [](double v) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
        return v;
    };
    double best = INFINITY;  // the lane's nearest triangle
    V3 q = {0, 0, 0};
    int bt = INT_MAX;
    auto triangles = [&](int g) {  // of run g (-1: none)
        if (g < 0) return;
        const Run R = T.run[g];
        if ((lane & 31) >= R.n) return;
        const int t = R.t0 + (lane & 31);
        const Corner3 C = corners(T, t);
        const V3 c = closest_on_triangle(P, C.a, C.b, C.c);
        const double d2 = (c.x - P.x) * (c.x - P.x) + (c.y - P.y) * (c.y - P.y) + (c.z - P.z) * (c.z - P.z);
        if (d2 < best || (d2 == best && t < bt)) {
            best = d2;
            bt = t;
            q = c;
        }
    };
    double bb = INFINITY;
    for (int b = b0 + lane; b < b1; b += 64) bb = fmin(bb, box_ub(T.bbox, T.nb, b, P));
    bb = wave_min(bb) * margin;
    // f(first run, runs) for every body within the distance `within`
    auto bodies = [&](double within, auto &&f) {
        for (int c = b0; c < b1; c += 64) {
            const int b = min(c + lane, b1 - 1);
            const Run R = T.body[b];
            unsigned long long m = __ballot(c + lane < b1 && !(box_lb(T.bbox, T.nb, b, P) > within));
            while (m) {
                const int l = __ffsll(m) - 1;
                m &= m - 1;
                f(__shfl(R.t0, l, 64), __shfl(R.n, l, 64));
            }
        }
    };
    double ub = INFINITY;
    int gb = -1;
    bodies(bb, [&](int g0, int n) {
        for (int g = g0 + lane; g < g0 + n; g += 64) {
            const double v = box_ub(T.box, T.nr, g, P);
            if (v < ub) {
                ub = v;
                gb = g;
            }
        }
    });
    const double ubw = wave_min(ub);
    const unsigned long long at = __ballot(ub == ubw && gb >= 0);
    if (at) triangles(lane < 32 ? __shfl(gb, __ffsll(at) - 1, 64) : -1);
    ub = fmin(ubw, wave_min(best)) * margin;
    bodies(fmin(bb, ub), [&](int g0, int n) {
        for (int c = g0; c < g0 + n; c += 64) {
            const int g = min(c + lane, g0 + n - 1);
            unsigned long long m = __ballot(c + lane < g0 + n && !(box_lb(T.box, T.nr, g, P) > ub));
            while (m) {
                const int q0 = __ffsll(m) - 1;
                m &= m - 1;
                int q1 = -1;
                if (m) {
                    q1 = __ffsll(m) - 1;
                    m &= m - 1;
                }
                triangles(lane < 32 ? c + q0 : (q1 < 0 ? -1 : c + q1));
            }
        }
    });
    double bd = best;
    int bi = bt;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double d = __shfl_xor(bd, o, 64);
        const int t = __shfl_xor(bi, o, 64);
        if (d < bd || (d == bd && t < bi)) {
            bd = d;
            bi = t;
        }
    }
    double *go = geo + 12 * (long long)r;
    if (bi == INT_MAX) {
        if (lane == 0) {
            near[r] = -1;
            go[0] = go[1] = go[2] = 0.0;
            go[11] = INFINITY;
        }
        return;
    }
    const unsigned long long w = __ballot(bt == bi);  // (the run that gave the bound is visited twice)
    if (lane == __ffsll(w) - 1) {
        near[r] = bt;
        go[0] = q.x; go[1] = q.y; go[2] = q.z;
        go[11] = best;
    }
}

// One thread per ghost row: image point, box, 8x8 LU, weights.  The matrix
// stays in registers: every index is known at compile time, row exchanges are
// selections.
__global__ void __launch_bounds__(64) k_stencil(Tris T, GridD G, const uint8_t *flags, const int32_t *cells,
                                                const int32_t *near, int ng, int nrows, const int32_t *mcell, int nm,
                                                long long N, int bc, RowOut O)
{
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrows) return;
    const bool mem = r >= ng;
    const int32_t cell = cells[r];
    const int nx = G.n[0], ny = G.n[1];
    const int ci = cell % nx, cj = (cell / nx) % ny, ck = cell / (nx * ny);
    const V3 P = {G.c[0][ci], G.c[1][cj], G.c[2][ck]};
    const int bt = near[r];
    const double *gi = O.geo + 12 * (long long)r;
    V3 BI = {gi[0], gi[1], gi[2]};
    const double best = gi[11];
    uint8_t fl = 0;
    double dist = sqrt(best);
    V3 nrm, IP;
    double dl;
    if (bt < 0) {  // no body of this kind: cannot happen for a consistent classification
        nrm = {0, 0, 1}; IP = P; dl = 1.0; dist = 0.0; BI = P;
        fl |= 1;
    } else if (dist < 1e-9 * G.hmin) {
        const Corner3 C = corners(T, bt);
        const V3 e1 = sub(C.b, C.a), e2 = sub(C.c, C.a);
        V3 fn = {e1.y * e2.z - e1.z * e2.y, e1.z * e2.x - e1.x * e2.z, e1.x * e2.y - e1.y * e2.x};
        double L = sqrt(fn.x * fn.x + fn.y * fn.y + fn.z * fn.z);
        double hl = fmin(G.w[0][ci], fmin(G.w[1][cj], G.w[2][ck]));
        nrm = {fn.x / L, fn.y / L, fn.z / L};
        BI = P;
        IP = {P.x + hl * nrm.x, P.y + hl * nrm.y, P.z + hl * nrm.z};
        dl = hl;
        fl |= 4;
    } else {
        nrm = {(BI.x - P.x) / dist, (BI.y - P.y) / dist, (BI.z - P.z) / dist};
        IP = {2.0 * BI.x - P.x, 2.0 * BI.y - P.y, 2.0 * BI.z - P.z};
        dl = 2.0 * dist;
    }
    const double ipa[3] = {IP.x, IP.y, IP.z}, bia[3] = {BI.x, BI.y, BI.z}, na[3] = {nrm.x, nrm.y, nrm.z};
    int b0[3];
    double loc[3], del[3], bil[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int n = G.n[d];
        const double *c = G.c[d];
        double x = ipa[d];
        if (x < c[0]) x = c[0];
        if (x > c[n - 1]) x = c[n - 1];
        b0[d] = box_index(c, n, x);
        del[d] = c[b0[d] + 1] - c[b0[d]];
        loc[d] = (x - c[b0[d]]) / del[d];
        bil[d] = (bia[d] - c[b0[d]]) / del[d];
    }
    // rows of V (node m) become columns of M = V^T
    double M[8][8];
    int32_t cl[8];
    int dnode = -1;
    bool degenerate = (fl & 1) != 0;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const int dx = m & 1, dy = (m >> 1) & 1, dz = (m >> 2) & 1;
        const int ii = b0[0] + dx, jj = b0[1] + dy, kk = b0[2] + dz;
        const long long id = (long long)ii + (long long)nx * (jj + (long long)ny * kk);
        const uint8_t f = flags[id];
        cl[m] = -1;
        double row[8];
        if (id == cell && bc == 1) {
            // Dirichlet: value row at BI
            const double x = bil[0], y = bil[1], z = bil[2];
            row[0] = 1.0; row[1] = x; row[2] = y; row[3] = z;
            row[4] = x * y; row[5] = y * z; row[6] = x * z; row[7] = x * y * z;
            dnode = m;
        } else if (id == cell) {
            const double x = bil[0], y = bil[1], z = bil[2];
            const double gx[8] = {0, 1, 0, 0, y, 0, z, y * z};
            const double gy[8] = {0, 0, 1, 0, x, z, 0, x * z};
            const double gz[8] = {0, 0, 0, 1, 0, y, x, x * y};
#pragma unroll
            for (int c = 0; c < 8; ++c) row[c] = na[0] / del[0] * gx[c] + na[1] / del[1] * gy[c] + na[2] / del[2] * gz[c];
            dnode = m;
        } else {
            const double x = dx, y = dy, z = dz;
            row[0] = 1.0; row[1] = x; row[2] = y; row[3] = z;
            row[4] = x * y; row[5] = y * z; row[6] = x * z; row[7] = x * y * z;
            if (!mem) {
                if (!(f & F_SOLID) || (f & F_GHOST)) cl[m] = (int32_t)id;
                else degenerate = true;
            } else {
                double side = na[0] * (G.c[0][ii] - bia[0]) + na[1] * (G.c[1][jj] - bia[1]) + na[2] * (G.c[2][kk] - bia[2]);
                if (side > 0.0) {
                    if (!(f & F_SOLID)) cl[m] = (int32_t)id;
                    else degenerate = true;
                } else {
                    int q = find_sorted(mcell, nm, (int32_t)id);
                    if (q >= 0) cl[m] = (int32_t)(N + q);
                    else degenerate = true;
                }
            }
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) M[c][m] = row[c];
    }
    double beta[8];
    if (!degenerate) {
        const double x = loc[0], y = loc[1], z = loc[2];
        beta[0] = 1.0; beta[1] = x; beta[2] = y; beta[3] = z;
        beta[4] = x * y; beta[5] = y * z; beta[6] = x * z; beta[7] = x * y * z;
        double amax = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) amax = fmax(amax, fabs(M[i][j]));
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            // the first row of the largest entry becomes the pivot
            int p = c;
            double pv = fabs(M[c][c]);
#pragma unroll
            for (int i = c + 1; i < 8; ++i)
                if (fabs(M[i][c]) > pv) {
                    pv = fabs(M[i][c]);
                    p = i;
                }
            if (!(pv >= 1e-12 * amax) || amax == 0.0) degenerate = true;  // (what follows is dropped)
#pragma unroll
            for (int i = c + 1; i < 8; ++i) {
                const bool sw = p == i;
#pragma unroll
                for (int j = c; j < 8; ++j) {
                    const double u = M[c][j], v = M[i][j];
                    M[c][j] = sw ? v : u;
                    M[i][j] = sw ? u : v;
                }
                const double u = beta[c], v = beta[i];
                beta[c] = sw ? v : u;
                beta[i] = sw ? u : v;
            }
#pragma unroll
            for (int i = c + 1; i < 8; ++i) {
                const double l = M[i][c] / M[c][c];
#pragma unroll
                for (int j = c + 1; j < 8; ++j) M[i][j] -= l * M[c][j];
                beta[i] -= l * beta[c];
            }
        }
#pragma unroll
        for (int c = 7; c >= 0; --c) {
            double s = beta[c];
#pragma unroll
            for (int j = c + 1; j < 8; ++j) s -= M[c][j] * beta[j];
            beta[c] = s / M[c][c];
        }
    }
    const double sg = G.cp[0][ci] + G.cm[0][ci] + G.cp[1][cj] + G.cm[1][cj] + G.cp[2][ck] + G.cm[2][ck];
    double bbi = 0.0;
    int32_t *oc = O.col + 8 * (long long)r;
    double *ow = O.w + 8 * (long long)r;
    if (!degenerate) {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            oc[m] = cl[m];
            ow[m] = cl[m] >= 0 ? beta[m] : 0.0;
            if (dnode == m) { bbi = beta[m]; fl |= 2; }
        }
        O.dlb[r] = bc == 1 ? 2.0 - bbi : dl - bbi;
        if (bc == 1 && (fl & 4)) {
            // ghost on the surface: x_G = g
            for (int m = 0; m < 8; ++m) { oc[m] = -1; ow[m] = 0.0; }
            O.dlb[r] = 1.0;
        }
    } else {
        fl |= 1;
        int cnt = 0;
        int32_t nb[6];
        const int cc[3] = {ci, cj, ck};
        const long long st[3] = {1, nx, (long long)nx * ny};
        for (int d = 0; d < 3; ++d)
            for (int sgn = -1; sgn <= 1; sgn += 2) {
                int c2 = cc[d] + sgn;
                if (c2 < 0 || c2 >= G.n[d]) continue;
                long long id = cell + sgn * st[d];
                bool use;
                if (!mem) use = !(flags[id] & F_SOLID);
                else use = (flags[sgn > 0 ? cell : id] & (F_CUTX << d)) != 0;
                if (use) nb[cnt++] = (int32_t)id;
            }
        for (int m = 0; m < 8; ++m) { oc[m] = -1; ow[m] = 0.0; }
        for (int m = 0; m < cnt; ++m) { oc[m] = nb[m]; ow[m] = 1.0 / cnt; }
        O.dlb[r] = bc == 1 ? 2.0 : 0.0;
    }
    O.sG[r] = sg;
    O.rfl[r] = fl;
    double *g = O.geo + 12 * (long long)r;
    g[0] = BI.x; g[1] = BI.y; g[2] = BI.z;
    g[3] = IP.x; g[4] = IP.y; g[5] = IP.z;
    g[6] = nrm.x; g[7] = nrm.y; g[8] = nrm.z;
    g[9] = dl; g[10] = bbi; g[11] = dist;
}

// rows that fell back to the face neighbours, one block
__global__ void __launch_bounds__(1024) k_count_fallback(const uint8_t *rfl, int n, int *cnt)
{
    int c = 0, tot;
    for (int i = threadIdx.x; i < n; i += 1024) c += rfl[i] & 1;
    (void)block_prefix(c, &tot);
    if (threadIdx.x == 0) *cnt = tot;
}

}  // namespace

CellLists::CellLists(const uint8_t *f, long long n, int k, uint8_t m0, uint8_t m1, uint8_t m2)
    : flags(f), N(n), K(k), nb((int)cdiv(n, CH)), m{m0, m1, m2}
{
}
void CellLists::count(int *total_dev, hipStream_t s)
{
    off.alloc((size_t)K * nb);
    k_count<<<nb, CB, 0, s>>>(flags, N, Bits{{m[0], m[1], m[2]}}, K, nb, off.p);
    k_scan<<<K, 1024, 0, s>>>(off.p, nb, total_dev);
    IBM_LAUNCH_CHECK();
}
void CellLists::fill(int32_t *o0, int32_t *o1, int32_t *o2, hipStream_t s)
{
    k_fill<<<nb, CB, 0, s>>>(flags, N, Bits{{m[0], m[1], m[2]}}, K, nb, off.p, Lists{{o0, o1, o2}});
    IBM_LAUNCH_CHECK();
}

void build_stencils(const ibm_grid *grid, const ibm_body *bodies, int n_body, const uint8_t *flags, ibm_stencils **out,
                    hipStream_t s, int bc = 0)
{
    IBM_REQUIRE(bc == IBM_BC_NEUMANN || bc == IBM_BC_DIRICHLET, IBM_EINVAL, "unknown boundary condition");
    HostGrid g = read_grid(grid);
    IBM_REQUIRE(flags && out, IBM_EINVAL, "null argument");
    IBM_REQUIRE(n_body >= 0 && (n_body == 0 || bodies), IBM_EINVAL, "bad body list");
    const long long N = (long long)g.n[0] * g.n[1] * g.n[2];
    auto *S = new ibm_stencils();
    try {
        for (int d = 0; d < 3; ++d) S->n[d] = g.n[d];
        S->N = N;
        S->bc = bc;
        // closed ghosts, membrane ghosts and the pin (kept with the table for the solver)
        CellLists C(flags, N, 3, F_GHOST, F_MGHOST, F_PIN);
        DBuf<int> res(5);  // the pin, fallback rows; counts of the lists
        int tot[3];
        C.count(res.p + 2, s);
        IBM_HIP(hipMemcpyAsync(tot, res.p + 2, sizeof tot, hipMemcpyDeviceToHost, s));
        IBM_HIP(hipStreamSynchronize(s));
        S->ng = tot[0];
        S->nm = tot[1];
        // stencil columns are int32: grid unknowns, then membrane ghost unknowns
        IBM_REQUIRE(N + S->nm < ((int64_t)1 << 31), IBM_EINVAL, "more than 2^31 unknowns with the membrane ghosts");
        const int64_t rows = S->ng + S->nm;
        IBM_REQUIRE(tot[2] == 1, IBM_EGEOM, "flags must hold exactly one pin cell");
        S->cell.alloc(std::max<int64_t>(rows, 1));
        S->col.alloc(std::max<int64_t>(rows, 1) * 8);
        S->w.alloc(std::max<int64_t>(rows, 1) * 8);
        S->sG.alloc(std::max<int64_t>(rows, 1));
        S->dlb.alloc(std::max<int64_t>(rows, 1));
        S->rfl.alloc(std::max<int64_t>(rows, 1));
        S->geo.alloc(std::max<int64_t>(rows, 1) * 12);
        C.fill(S->cell.p, S->cell.p + S->ng, res.p, s);
        Image I;  // (its copy has ended when the results are read)
        DBuf<char> up;
        DBuf<double> box;
        DBuf<int32_t> near;
        if (rows > 0) {
            // grid on device
            std::vector<double> c[3], w[3], cp[3], cm[3];
            double hmin = 1e300;
            for (int d = 0; d < 3; ++d) {
                int n = g.n[d];
                c[d].resize(n); w[d].resize(n); cp[d].resize(n); cm[d].resize(n);
                for (int i = 0; i < n; ++i) {
                    c[d][i] = 0.5 * (g.f[d][i] + g.f[d][i + 1]);
                    w[d][i] = g.f[d][i + 1] - g.f[d][i];
                    hmin = std::min(hmin, w[d][i]);
                }
                for (int i = 0; i < n; ++i) {
                    cp[d][i] = (i + 1 < n) ? 1.0 / (w[d][i] * (c[d][i + 1] - c[d][i])) : 0.0;
                    cm[d][i] = (i > 0) ? 1.0 / (w[d][i] * (c[d][i] - c[d][i - 1])) : 0.0;
                }
            }
            GridD G;
            const std::vector<double> *ga[4] = {c, w, cp, cm};
            size_t go[4][3];
            for (int q = 0; q < 4; ++q)
                for (int d = 0; d < 3; ++d) go[q][d] = I.put(ga[q][d]);
            // vertices and triangles of all bodies, and the runs by kind
            long long nv = 0, nt = 0;
            std::vector<Run> runs, body;
            int nclosed = 0;
            std::vector<long long> first(n_body);  // first triangle
            for (int b = 0; b < n_body; ++b) {
                const ibm_body &B = bodies[b];
                IBM_REQUIRE(B.vert && B.tri && B.n_tri > 0, IBM_EINVAL, "empty body");
                for (int t = 0; t < 3 * B.n_tri; ++t)
                    IBM_REQUIRE(B.tri[t] >= 0 && B.tri[t] < B.n_vert, IBM_EGEOM, "triangle index out of range");
                first[b] = nt;
                nv += B.n_vert;
                nt += B.n_tri;
                IBM_REQUIRE(nv < ((int64_t)1 << 31) && nt < ((int64_t)1 << 31), IBM_EINVAL,
                            "more than 2^31 vertices or triangles");
            }
            for (int kind = 0; kind < 2; ++kind) {
                for (int b = 0; b < n_body; ++b) {
                    if (bodies[b].kind != kind) continue;
                    const int r0 = (int)runs.size(), n = bodies[b].n_tri;
                    for (int t = 0; t < n; t += TGROUP) runs.push_back({(int)first[b] + t, std::min(TGROUP, n - t)});
                    body.push_back({r0, (int)runs.size() - r0});
                }
                if (kind == 0) nclosed = (int)body.size();
            }
            const int nr = (int)runs.size(), nb = (int)body.size();
            const size_t ov = I.take(3 * nv * sizeof(double)), ot = I.take(3 * nt * sizeof(int32_t)),
                         orun = I.put(runs), obody = I.put(body);
            double *hv = I.at<double>(ov);
            int32_t *ht = I.at<int32_t>(ot);
            int v0 = 0;
            for (int b = 0; b < n_body; ++b) {
                const ibm_body &B = bodies[b];
                hv = std::copy(B.vert, B.vert + 3 * (size_t)B.n_vert, hv);
                for (int t = 0; t < 3 * B.n_tri; ++t) *ht++ = v0 + B.tri[t];
                v0 += B.n_vert;
            }
            I.upload(up, s);
            for (int d = 0; d < 3; ++d) {
                G.c[d] = (const double *)(up.p + go[0][d]);
                G.w[d] = (const double *)(up.p + go[1][d]);
                G.cp[d] = (const double *)(up.p + go[2][d]);
                G.cm[d] = (const double *)(up.p + go[3][d]);
                G.n[d] = g.n[d];
            }
            G.hmin = hmin;
            box.alloc(std::max(6 * ((size_t)nr + nb), (size_t)1));
            near.alloc(rows);
            const Tris T{(const double *)(up.p + ov), (const int32_t *)(up.p + ot), (const Run *)(up.p + orun),
                         (const Run *)(up.p + obody), box.p, box.p + 6 * (size_t)nr, nr, nb, {0, nclosed, nb}};
            const RowOut O{S->col.p, S->w.p, S->sG.p, S->dlb.p, S->geo.p, S->rfl.p};
            if (nb) {
                k_run_boxes<<<cdiv((long long)nr * TGROUP, 256), 256, 0, s>>>(T);
                k_body_boxes<<<nb, 64, 0, s>>>(T);
            }
            // (a launch has less than 2^32 threads: 2^24 rows of a wavefront each at a time)
            for (int64_t r0 = 0; r0 < rows; r0 += 1 << 24)
                k_nearest<<<cdiv(std::min<int64_t>(rows - r0, 1 << 24), 4), 256, 0, s>>>(
                    T, G, S->cell.p, (int)r0, (int)S->ng, (int)rows, S->geo.p, near.p);
            k_stencil<<<cdiv(rows, 64), 64, 0, s>>>(T, G, flags, S->cell.p, near.p, (int)S->ng, (int)rows,
                                                   S->cell.p + S->ng, (int)S->nm, N, bc, O);
            IBM_LAUNCH_CHECK();
        }
        k_count_fallback<<<1, 1024, 0, s>>>(S->rfl.p, (int)rows, res.p + 1);
        IBM_LAUNCH_CHECK();
        int h[2];
        IBM_HIP(hipMemcpyAsync(h, res.p, sizeof h, hipMemcpyDeviceToHost, s));
        IBM_HIP(hipStreamSynchronize(s));
        S->pin = h[0];
        S->nfallback = h[1];
    } catch (...) {
        delete S;
        throw;
    }
    *out = S;
}

}  // namespace ibm

extern "C" int32_t ibm_build_ghost_stencils(const ibm_grid *grid, const ibm_body *bodies, int32_t n_body,
                                            const uint8_t *flags_dev, ibm_stencils **out, void *stream)
{
    return ibm::guarded([&] { ibm::build_stencils(grid, bodies, n_body, flags_dev, out, (hipStream_t)stream); });
}

extern "C" int32_t ibm_build_ghost_stencils_bc(const ibm_grid *grid, const ibm_body *bodies, int32_t n_body,
                                               const uint8_t *flags_dev, int32_t bc, ibm_stencils **out, void *stream)
{
    return ibm::guarded(
        [&] { ibm::build_stencils(grid, bodies, n_body, flags_dev, out, (hipStream_t)stream, bc); });
}

extern "C" int32_t ibm_stencils_info(const ibm_stencils *s, int64_t *n_ghost, int64_t *n_mghost, int64_t *n_fallback)
{
    return ibm::guarded([&] {
        IBM_REQUIRE(s, IBM_EINVAL, "null stencils");
        if (n_ghost) *n_ghost = s->ng;
        if (n_mghost) *n_mghost = s->nm;
        if (n_fallback) *n_fallback = s->nfallback;
    });
}

extern "C" int32_t ibm_stencils_export(const ibm_stencils *s, int32_t *cell, int32_t *col, double *w, double *sG,
                                       double *dlb, uint8_t *rflags, double *geo)
{
    return ibm::guarded([&] {
        IBM_REQUIRE(s, IBM_EINVAL, "null stencils");
        size_t rows = (size_t)(s->ng + s->nm);
        if (!rows) return;
        // copies on a private non-blocking stream: nothing here touches the
        // legacy stream, which may not depend on another thread's capture
        hipStream_t st = nullptr;
        IBM_HIP(hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
        struct Del {
            hipStream_t q;
            ~Del() { (void)hipStreamDestroy(q); }
        } del{st};
        if (cell) IBM_HIP(hipMemcpyAsync(cell, s->cell.p, rows * 4, hipMemcpyDeviceToHost, st));
        if (col) IBM_HIP(hipMemcpyAsync(col, s->col.p, rows * 32, hipMemcpyDeviceToHost, st));
        if (w) IBM_HIP(hipMemcpyAsync(w, s->w.p, rows * 64, hipMemcpyDeviceToHost, st));
        if (sG) IBM_HIP(hipMemcpyAsync(sG, s->sG.p, rows * 8, hipMemcpyDeviceToHost, st));
        if (dlb) IBM_HIP(hipMemcpyAsync(dlb, s->dlb.p, rows * 8, hipMemcpyDeviceToHost, st));
        if (rflags) IBM_HIP(hipMemcpyAsync(rflags, s->rfl.p, rows, hipMemcpyDeviceToHost, st));
        if (geo) IBM_HIP(hipMemcpyAsync(geo, s->geo.p, rows * 96, hipMemcpyDeviceToHost, st));
        IBM_HIP(hipStreamSynchronize(st));
    });
}

extern "C" void ibm_stencils_free(ibm_stencils *s) { delete s; }
