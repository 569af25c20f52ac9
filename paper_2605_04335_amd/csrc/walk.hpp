// Fused level-0 smoothing: a whole smoothing phase of the V-cycle (two
// red/black steps and the transfer next to it) in one pass over the level.
//
// Away from the bodies level 0 is a plain 7-point operator.  A block owns a
// tile of 32 half-indices x 20 rows and walks a run of planes; four
// half-sweeps follow each other down the planes as a pipeline, each one plane
// behind the one before, so the right-hand side is read once and the iterate
// is written once where the one-sweep kernels pass over both four times.
// Tiles overlap by the pipeline's dependency depth (2 half-indices, 4 rows, 4
// planes) and recompute the overlap.
//
// Bound: the chain of LDS reads and barriers at one block per CU, and in FP64
// also bytes.  At 512^3, with nothing beside it, the first phase takes 0.79 ms
// and the second 0.80 (2.0 and 1.9 with one launch per half-sweep); per cell 69
// and 79 vector instructions (the vector units issue in 0.39 and 0.45 of the
// busy cycles), 2.05 and 3.53 GB from and to memory (1.18 and 1.25 of what they
// cannot do without), 2.6 and 4.4 TB/s.  FP32 0.68 and 0.77 ms: 91 and 105
// instructions (conversions), 0.61 of the cycles, 1.01 and 1.68 GB.  In a solve
// with bodies the near cells' launches (below) run beside the passes from 2^23
// cells on and take registers and bandwidth: 0.92 and 0.88 ms in FP64; 0.73 and
// 0.75 in FP32.
//
// The pass covers the whole level and treats every cell as a regular one.  Its
// results are wrong near cells with a row of their own (solid, ghost,
// membrane); a list of small units around those runs the one-sweep sequence
// with the sparse rows in a vector of its own, and its results replace the
// pass's there.
#pragma once

#include "fused.hpp"

namespace ibm {

constexpr int WK_H = 36, WK_J = 28;      // columns a block works on
constexpr int WK_OH = 32, WK_OJ = 20;    // columns it owns
constexpr int WK_C = WK_H * WK_J;        // 1008: one per thread
constexpr int WK_T = 1024;
constexpr int WK_KZMAX = 256;            // planes of a block at most (a multiple of 4, as every block's first plane)
constexpr int WK_PAD = 40;
constexpr int WK_PS = WK_C + 2 * WK_PAD; // LDS plane
constexpr int WK_CH = WK_H + 2, WK_CJ = WK_J / 2 + 2;  // coarse tile of the prolongation

// units around irregular cells (below)
constexpr uint8_t UB_IRR = 0x0f;   // irregular cell in quarter (row half) + 2 (plane half)
constexpr uint8_t UB_READ = 0x10;  // a slot read by a sparse row
constexpr uint8_t UB_NEAR = 0x20;
constexpr uint8_t UB_LIST = 0x40;
constexpr uint8_t UB_DEAD = 0x80;  // no active cell
constexpr int NU_T = 256;          // four units per block

struct Near {
    const int32_t *units;   // listed units
    const uint8_t *bits;    // per unit
    int n, nux, nuy, nuz;
    int nb() const { return (n + 3) / 4; }  // blocks
};

// tiles of a level and the planes of a block (even)
struct WalkGeo {
    int ntx, nty, kz, ncz;
    int nb;  // launched blocks (multiple of 8)
};
// run of planes [k0, k1) (k0 a multiple of 4, k1 even) of the tile at (h0, j0)
struct WalkSeg {
    int h0, j0, k0, k1;
};

// wave-uniform load of data that no kernel in flight writes: through the
// constant address space it becomes a scalar load, which needs no vector
// register and does not queue behind the vector loads in flight
template <class T>
__device__ __forceinline__ T uld(const T *p, int i)
{
    typedef const __attribute__((address_space(4))) T *cp;
    return ((cp)(uintptr_t)p)[i];
}

// Constants of a thread's column.  Index q: the red cell of an even (0) or odd
// (1) plane, which is also the black cell of a plane of the other parity: its
// x neighbours are the column's other cell (coefficient cen) and a cell one
// column over (coefficient out, offset off); zero coefficients at the walls.
// Threads beyond the domain repeat its edge column (their values stay finite
// and meet only zero coefficients).
struct WalkCol {
    double cen[2], out[2], dxy[2], cpy, cmy;
    int off;        // of index 0; index 1: -off
    uint32_t col;   // slot within a plane
    int p;          // LDS place
    uint32_t hj;    // hc | jc << 16
    bool own;
    __device__ __forceinline__ int hc() const { return (int)(hj & 0xffff); }
    __device__ __forceinline__ int jc() const { return (int)(hj >> 16); }
};
__device__ __forceinline__ WalkCol walk_col(const Lv &F, const WalkSeg &S)
{
    WalkCol w;
    const int tid = threadIdx.x;
    w.p = tid < WK_C ? tid : 0;
    const int jl = w.p / WK_H, hl = w.p - jl * WK_H;
    const int h = S.h0 - 2 + hl, j = S.j0 - 4 + jl;
    const int hc = min(max(h, 0), F.H - 1), jc = min(max(j, 0), F.ny - 1);
    w.hj = (uint32_t)hc | ((uint32_t)jc << 16);
    w.own = tid < WK_C && hl >= 2 && hl < 2 + WK_OH && jl >= 4 && jl < 4 + WK_OJ && h < F.H && j < F.ny;
    w.col = (uint32_t)(hc + F.H * jc);
    w.cpy = F.cp[1][jc];  // zero at the walls, as every coefficient
    w.cmy = F.cm[1][jc];
    w.off = (jc & 1) ? 1 : -1;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int e = (jc + q) & 1, i = 2 * hc + e;
        const double cpx = F.cp[0][i], cmx = F.cm[0][i];
        w.cen[q] = e ? cmx : cpx;
        w.out[q] = e ? cpx : cmx;
        w.dxy[q] = cpx + cmx + w.cpy + w.cmy;
    }
    return w;
}

// the pin's plane, column and colour (wave-uniform; plane -1 without a sink)
struct WalkPin {
    int k, c;
    uint32_t col;
    double sink;
};
__device__ __forceinline__ WalkPin walk_pin(const Lv &F, const WalkSeg &S, long long pin, const double *sink)
{
    WalkPin q{-1, 0, 0, 0.0};
    if (!sink) return q;
    q.c = pin >= F.Nh;
    const uint32_t r = (uint32_t)(pin - (q.c ? F.Nh : 0)), pl = (uint32_t)(F.H * F.ny);
    const int k = (int)(r / pl);
    q.col = r - (uint32_t)k * pl;
    // only where the block's planes hold it
    if (k >= S.k0 - 4 && k < S.k1 + 4) q.k = k;
    q.sink = uld(sink, 0);
    return q;
}

// segment of this block (consecutive blocks of an XCD take neighbouring tiles
// of one run of planes, which share their overlap in its L2); false for
// padding blocks
__device__ __forceinline__ bool walk_seg(const WalkGeo &G, int nz, WalkSeg &S)
{
    const int q = (int)(blockIdx.x & 7) * (G.nb >> 3) + (int)(blockIdx.x >> 3);
    const int tx = q % G.ntx, r = q / G.ntx, ty = r % G.nty, tz = r / G.nty;
    if (tz >= G.ncz) return false;
    S.h0 = tx * WK_OH;
    S.j0 = ty * WK_OJ;
    S.k0 = tz * G.kz;
    S.k1 = min(nz, S.k0 + G.kz);
    return true;
}

// store at a block-uniform base plus a 32-bit element offset
template <class T>
__device__ __forceinline__ void stu_nt(T *base, uint32_t i, T v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<T *>(reinterpret_cast<char *>(base) + i * (uint32_t)sizeof(T)));
}

// barrier that orders LDS only: global loads stay in flight across it
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// neighbour sum of a cell with index q: centre, outer x and y neighbours from
// the LDS plane at l, z neighbours zp and zm
#define WALK_NB(q, l, xc, zp, zm, cp_, cm_)                                                                       \
    (w.cen[q] * (xc) + w.out[q] * (double)(l)[(q) ? -w.off : w.off] + w.cpy * (double)(l)[WK_H] + w.cmy * (double)(l)[-WK_H] + \
     (cp_) * (zp) + (cm_) * (zm))

// First phase of a V-cycle: red, black, red, black from zero, the residual and
// its restriction.  Plane k: first red; k-1: first black; k-2: second red;
// k-3: second black, written to xk; k-4: residual of the red cells (the black
// ones were relaxed last: theirs is zero to rounding).  Of the iterate only the
// black cells leave the kernel: the second phase starts from them.
template <class T, class TBc>
__global__ void __launch_bounds__(WK_T) k_walk_down(Lv F, Lv C, WalkGeo G, Near U, long long pin,
                                                    const double *__restrict__ sink, const T *__restrict__ b,
                                                    T *__restrict__ xk, TBc *__restrict__ bc, double *part)
{
    __shared__ T lds[2 * 4 * WK_PS];
    // right-hand sides kept for their second use two planes on (in FP64 whatever T:
    // the pin's less the sink is not a T)
    __shared__ double lagb[4][WK_T];
    __shared__ double lagr[2][WK_T];  // b + dg x of the red cells, for the residual two planes on
    __shared__ double e0[WK_T], ex[WK_T + WK_H];  // per column: the residual of a coarse cell's lower plane; of both
    __shared__ double ms[WK_T];         // per column: its share of the coarse mean
    __shared__ double red[WK_T / 64];
    __shared__ double wxl[2 * WK_H], wyl[WK_J], cxl[WK_H], cyl[WK_J];
    __shared__ uint8_t ub[WK_OH / 4 * (WK_OJ / 4) * (WK_KZMAX / 4)];
    WalkSeg S;
    if (!walk_seg(G, F.nz, S)) {
        if (threadIdx.x == 0) part[blockIdx.x] = 0.0;
        return;
    }
    const WalkCol w = walk_col(F, S);
    const int tid = threadIdx.x;
    for (int q = tid; q < 2 * 4 * WK_PS; q += WK_T) lds[q] = (T)0;
    const long long pl = (long long)F.H * F.ny;
    const T *const bp[2] = {b, b + F.Nh};
    auto cz = [&](int k) { return min(max(k, 0), F.nz - 1); };
    const WalkPin pn = walk_pin(F, S, pin, sink);  // the pin's RHS carries the sink
    // widths: of the cells of index 0 and 1 and of the rows, and of the coarse columns and rows
    if (tid < WK_H)
#pragma unroll
        for (int e = 0; e < 2; ++e) wxl[2 * tid + e] = F.w[0][2 * min(max(S.h0 - 2 + tid, 0), F.H - 1) + e];
    else if (tid < WK_H + WK_J) wyl[tid - WK_H] = F.w[1][min(max(S.j0 - 4 + tid - WK_H, 0), F.ny - 1)];
    else if (tid < 2 * WK_H + WK_J) cxl[tid - WK_H - WK_J] = C.w[0][min(max(S.h0 - 2 + tid - WK_H - WK_J, 0), C.nx - 1)];
    else if (tid < 2 * WK_H + 2 * WK_J)
        cyl[tid - 2 * WK_H - WK_J] = C.w[1][min(max((S.j0 - 4 + tid - 2 * WK_H - WK_J) >> 1, 0), C.ny - 1)];
    // bits of the tile's own units
    for (int q = tid; q < WK_OH / 4 * (WK_OJ / 4) * ((S.k1 - S.k0 + 3) / 4); q += WK_T) {
        const int ux = (S.h0 >> 2) + q % (WK_OH / 4), r = q / (WK_OH / 4), uy = (S.j0 >> 2) + r % (WK_OJ / 4),
                  uz = (S.k0 >> 2) + r / (WK_OJ / 4);
        ub[q] = U.n && ux < U.nux && uy < U.nuy && uz < U.nuz ? U.bits[ux + (long long)U.nux * (uy + (long long)U.nuy * uz)]
                                                              : (uint8_t)0;
    }
    const bool odd_row = w.jc() & 1;
    const bool lead = w.own && !odd_row;  // the even row of a pair writes the coarse cell
    __syncthreads();
    T bR[3], bB[3];
    double czp[6], czm[6], R1[3] = {}, B1[3] = {}, R2[3] = {}, B2[3] = {}, rdR[3] = {}, rdB[3] = {};
#pragma unroll
    for (int q = 0; q < 6; ++q) czp[q] = czm[q] = 1.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) lagb[q][tid] = 0.0;
    lagr[0][tid] = lagr[1][tid] = ms[tid] = 0.0;
    bB[2] = (T)0;
    const int ks = S.k0 - 4, ke = S.k1 + 4;  // steps load-plane ks .. ke-1
    bR[0] = ldu(bp[0] + pl * cz(ks), w.col);
    bR[1] = ldu(bp[0] + pl * cz(ks + 1), w.col);
    bB[0] = ldu(bp[1] + pl * cz(ks), w.col);
    czp[0] = uld(F.cp[2], cz(ks));
    czm[0] = uld(F.cm[2], cz(ks));
    const double *const wxr = wxl + 2 * (w.p % WK_H);
    // coarse cell of rows (2J, 2J+1), fine planes (2K, 2K+1)
    auto coarse = [&](int K) {
        const double svr = ex[w.p] + ex[w.p + WK_H];
        const int I = w.hc(), J = w.jc() >> 1;
        const int jl = w.p / WK_H;
        const double VC = cxl[w.p - jl * WK_H] * cyl[jl] * uld(C.w[2], K);
        // (a near unit's cells are restricted by the near sequence)
        if (ub[(((K << 1) - S.k0) >> 2) * (WK_OH / 4 * (WK_OJ / 4)) + ((jl - 4) >> 2) * (WK_OH / 4) +
               ((w.p - jl * WK_H - 2) >> 2)] & UB_NEAR) return;
        st(bc, slot(C, (I + J + K) & 1, I >> 1, J, K), svr / VC);
        ms[tid] += VC * round_to<TBc>(svr / VC);
    };
    for (int kk = ks; kk < ke; kk += 6) {
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            const int k = kk + s;
            if (k >= ke) break;
            const int q = s & 1;  // parity of k (ks is even)
            T *const lw = lds + q * 4 * WK_PS + WK_PAD + w.p;
            const T *const lr = lds + (1 - q) * 4 * WK_PS + WK_PAD + w.p;
            // loads of later steps
            double b0 = bR[s % 3], b1 = bB[(s + 2) % 3];  // red of plane k, black of plane k-1
            bR[(s + 2) % 3] = ldu(bp[0] + pl * cz(k + 2), w.col);
            bB[(s + 1) % 3] = ldu(bp[1] + pl * cz(k + 1), w.col);
            czp[(s + 1) % 6] = uld(F.cp[2], cz(k + 1));
            czm[(s + 1) % 6] = uld(F.cm[2], cz(k + 1));
            if (pn.k >= 0) {
                if (pn.c == 0 && cz(k) == pn.k && w.col == pn.col) b0 -= pn.sink;
                if (pn.c == 1 && cz(k - 1) == pn.k && w.col == pn.col) b1 -= pn.sink;
            }
            // the other side of the row pair's sum, one step after it was made
            if (q == 0 && lead && k - 6 >= S.k0) coarse((k - 6) >> 1);
            {   // plane k: first red
                const double dg = w.dxy[q] + czp[s] + czm[s];
                rdR[s % 3] = recip(dg);
                R1[s % 3] = (double)(T)quot(-b0, dg, rdR[s % 3]);
            }
            {   // plane k-1: first black
                const int m = (s + 5) % 6;
                const double dg = w.dxy[q] + czp[m] + czm[m];
                rdB[(s + 2) % 3] = recip(dg);
                const double nb = WALK_NB(q, lr, R1[(s + 2) % 3], R1[s % 3], R1[(s + 1) % 3], czp[m], czm[m]);
                B1[(s + 2) % 3] = (double)(T)quot(nb - b1, dg, rdB[(s + 2) % 3]);
            }
            double rk;
            {   // plane k-2: second red
                const int m = (s + 4) % 6;
                const double dg = w.dxy[q] + czp[m] + czm[m];
                const double nb = WALK_NB(q, lr + WK_PS, B1[(s + 1) % 3], B1[(s + 2) % 3], B1[s % 3], czp[m], czm[m]);
                const double b2 = lagb[q][tid];
                lagb[q][tid] = b0;
                const double v = (double)(T)quot(nb - b2, dg, rdR[(s + 1) % 3]);
                R2[(s + 1) % 3] = v;
                rk = b2 + dg * v;
            }
            {   // plane k-3: second black
                const int m = (s + 3) % 6;
                const double dg = w.dxy[q] + czp[m] + czm[m];
                const double nb = WALK_NB(q, lr + 2 * WK_PS, R2[s % 3], R2[(s + 1) % 3], R2[(s + 2) % 3], czp[m], czm[m]);
                const double b3 = lagb[2 + q][tid];
                lagb[2 + q][tid] = b1;
                const T v = (T)quot(nb - b3, dg, rdB[s % 3]);
                B2[s % 3] = (double)v;
                lw[3 * WK_PS] = v;
                if (w.own && k - 3 >= S.k0 && k - 3 < S.k1) stu_nt(xk + pl * (k - 3), w.col, v);
            }
            {   // plane k-4: residual of the red cells, volume-weighted
                const int m = (s + 2) % 6;
                const double nb =
                    WALK_NB(q, lr + 3 * WK_PS, B2[(s + 2) % 3], B2[s % 3], B2[(s + 1) % 3], czp[m], czm[m]);
                const double r4 = lagr[q][tid];
                lagr[q][tid] = rk;
                const double v = uld(F.w[2], cz(k - 4)) * (wxr[q ^ (odd_row ? 1 : 0)] * (r4 - nb));
                if (q == 0) e0[tid] = v;
                else ex[tid] = (e0[tid] + v) * wyl[w.p / WK_H];
            }
            lw[0] = (T)R1[s % 3];
            lw[WK_PS] = (T)B1[(s + 2) % 3];
            lw[2 * WK_PS] = (T)R2[(s + 1) % 3];
            lds_barrier();
        }
    }
    if (lead) coarse((S.k1 - 2) >> 1);
    double msum = ms[tid];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) msum += __shfl_xor(msum, o, 64);
    if ((tid & 63) == 0) red[tid >> 6] = msum;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int q = 0; q < WK_T / 64; ++q) t += red[q];
        part[blockIdx.x] = t;
    }
}

// Second phase: prolongation onto the black cells and red, black, red, black.
// Plane k: corrected black; k-1: first red; k-2: first black; k-3: second red
// (written); k-4: second black (written).  Coarse values are loaded by coarse
// plane, interpolated in y and x as they arrive (two values per thread: the
// black cells of even and of odd planes) and kept for the z interpolation.
template <class T>
__global__ void __launch_bounds__(WK_T) k_walk_up(Lv F, Lv C, PMap M, WalkGeo G, long long pin,
                                                  const double *__restrict__ sink,
                                                  const T *__restrict__ b, const T *__restrict__ xk,
                                                  const T *__restrict__ xc, T *__restrict__ x)
{
    __shared__ T lds[2 * 4 * WK_PS];
    __shared__ double lagb[4][WK_T];         // right-hand sides kept for their second use two planes on
    __shared__ T cl[3][WK_CH * WK_CJ];       // coarse planes by their number modulo 3
    __shared__ double txl[2 * WK_H], tyl[WK_J];
    WalkSeg S;
    if (!walk_seg(G, F.nz, S)) return;
    const WalkCol w = walk_col(F, S);
    const int tid = threadIdx.x;
    for (int q = tid; q < 2 * 4 * WK_PS; q += WK_T) lds[q] = (T)0;
    const long long pl = (long long)F.H * F.ny;
    const T *const bp[2] = {b, b + F.Nh};
    auto cz = [&](int k) { return min(max(k, 0), F.nz - 1); };
    const WalkPin pn = walk_pin(F, S, pin, sink);
    // the coarse tile: parents of the columns and one more on either side;
    // threads below WK_CH WK_CJ load one value each per coarse plane
    const long long cpl = (long long)C.H * C.ny;
    const int Ia = S.h0 - 3, Ja = (S.j0 >> 1) - 3;
    const bool cth = tid < WK_CH * WK_CJ;
    uint32_t ccol;
    bool cpar;
    {
        const int r = tid / WK_CH, I = min(max(Ia + tid - r * WK_CH, 0), C.nx - 1), J = min(max(Ja + r, 0), C.ny - 1);
        ccol = (uint32_t)((I >> 1) + C.H * J);
        cpar = (I + J) & 1;
    }
    auto cload = [&](int K) {
        K = min(max(K, 0), C.nz - 1);
        return cth ? ldu(xc + cpl * K, ccol + (cpar != (bool)(K & 1) ? (uint32_t)C.Nh : 0u)) : (T)0;
    };
    // lower coarse node and weights of the thread's cells: the black cell of an
    // even plane has i parity 1 - (j & 1), of an odd plane (j & 1)
    int cn[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
        cn[q] = M.pi[0][2 * w.hc() + ((w.jc() + 1 + q) & 1)] - Ia + WK_CH * (M.pi[1][w.jc()] - Ja);
    if (tid < 2 * WK_H) txl[tid] = M.pt[0][min(max(2 * (S.h0 - 2) + tid, 0), F.nx - 1)];
    else if (tid < 2 * WK_H + WK_J) tyl[tid - 2 * WK_H] = M.pt[1][min(max(S.j0 - 4 + tid - 2 * WK_H, 0), F.ny - 1)];
    const double *const txr = txl + 2 * (w.p % WK_H), *const tyr = tyl + w.p / WK_H;
    const bool odd_row = w.jc() & 1;
    // weight of the upper of the two coarse planes of fine plane k: the map's,
    // except at the walls, where the clamped interpolation takes one node alone
    auto upper = [&](int k) {
        const int kc = min(max(k, 0), F.nz - 1), low = (k >> 1) - 1 + (k & 1), node = uld(M.pi[2], kc);
        const double t = uld(M.pt[2], kc);
        return node == low ? t : (node > low ? 1.0 : 0.0);
    };
    const int ks = S.k0 - 4, ke = S.k1 + 4;
    const int K0 = ks >> 1;  // ks is even and may be negative: -4 -> -2
    if (cth) {
        cl[2][tid] = cload(K0 - 1);
        cl[0][tid] = cload(K0);
        cl[1][tid] = cload(K0 + 1);
    }
    T cnext = cload(K0 + 2);
    double tz = upper(ks);
    T KB[3], bR[3], bB[3];
    double czp[6], czm[6], B0[3] = {}, R1[3] = {}, B1[3] = {}, R2[3] = {}, rdR[3] = {}, rdB[3] = {};
#pragma unroll
    for (int q = 0; q < 6; ++q) czp[q] = czm[q] = 1.0;
#pragma unroll
    for (int q = 0; q < 3; ++q) bR[q] = bB[q] = (T)0;
#pragma unroll
    for (int q = 0; q < 4; ++q) lagb[q][tid] = 0.0;
    KB[0] = ldu(xk + pl * cz(ks), w.col);
    KB[1] = ldu(xk + pl * cz(ks + 1), w.col);
    KB[2] = (T)0;
    bR[0] = ldu(bp[0] + pl * cz(ks), w.col);
    czp[0] = uld(F.cp[2], cz(ks));
    czm[0] = uld(F.cm[2], cz(ks));
    __syncthreads();
    for (int kk = ks; kk < ke; kk += 6) {
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            const int k = kk + s;
            if (k >= ke) break;
            const int q = s & 1;
            T *const lw = lds + q * 4 * WK_PS + WK_PAD + w.p;
            const T *const lr = lds + (1 - q) * 4 * WK_PS + WK_PAD + w.p;
            KB[(s + 2) % 3] = ldu(xk + pl * cz(k + 2), w.col);
            double b1 = bR[(s + 2) % 3], b2 = bB[(s + 1) % 3];  // red of plane k-1, black of plane k-2
            bR[(s + 1) % 3] = ldu(bp[0] + pl * cz(k + 1), w.col);
            bB[s % 3] = ldu(bp[1] + pl * cz(k), w.col);
            czp[(s + 1) % 6] = uld(F.cp[2], cz(k + 1));
            czm[(s + 1) % 6] = uld(F.cm[2], cz(k + 1));
            if (pn.k >= 0) {
                if (pn.c == 0 && cz(k - 1) == pn.k && w.col == pn.col) b1 -= pn.sink;
                if (pn.c == 1 && cz(k - 2) == pn.k && w.col == pn.col) b2 -= pn.sink;
            }
            {   // plane k: prolongation onto the black cell, from coarse planes
                // K-1, K when k is even and K, K+1 when it is odd; plane K+1 is
                // loaded at the even plane and used at the odd one
                const int a = (s >> 1) % 3, lo = q ? a : (a + 2) % 3, up = q ? (a + 1) % 3 : a;
                // (plane K+2 was loaded two steps ago; K-1's place is free after the even plane)
                const double tx = txr[q ^ (odd_row ? 0 : 1)], ty = *tyr;
                auto lerp = [](double t, double u, double v) { return (1 - t) * u + t * v; };
                auto face = [&](const T *v) {
                    return lerp(ty, lerp(tx, v[0], v[1]), lerp(tx, v[WK_CH], v[WK_CH + 1]));
                };
                const double c = lerp(tz, face(cl[lo] + cn[q]), face(cl[up] + cn[q]));
                B0[s % 3] = (double)(T)((double)KB[s % 3] + c);
                tz = upper(k + 1);
                if (q == 1) {
                    if (cth) cl[(a + 2) % 3][tid] = cnext;
                    cnext = cload((k >> 1) + 3);
                }
            }
            {   // plane k-1: first red
                const int m = (s + 5) % 6;
                const double dg = w.dxy[1 - q] + czp[m] + czm[m];
                rdR[(s + 2) % 3] = recip(dg);
                const double nb = WALK_NB(1 - q, lr, B0[(s + 2) % 3], B0[s % 3], B0[(s + 1) % 3], czp[m], czm[m]);
                R1[(s + 2) % 3] = (double)(T)quot(nb - b1, dg, rdR[(s + 2) % 3]);
            }
            {   // plane k-2: first black
                const int m = (s + 4) % 6;
                const double dg = w.dxy[1 - q] + czp[m] + czm[m];
                rdB[(s + 1) % 3] = recip(dg);
                const double nb =
                    WALK_NB(1 - q, lr + WK_PS, R1[(s + 1) % 3], R1[(s + 2) % 3], R1[s % 3], czp[m], czm[m]);
                B1[(s + 1) % 3] = (double)(T)quot(nb - b2, dg, rdB[(s + 1) % 3]);
            }
            {   // plane k-3: second red
                const int m = (s + 3) % 6;
                const double dg = w.dxy[1 - q] + czp[m] + czm[m];
                const double nb =
                    WALK_NB(1 - q, lr + 2 * WK_PS, B1[s % 3], B1[(s + 1) % 3], B1[(s + 2) % 3], czp[m], czm[m]);
                const double b3 = lagb[q][tid];
                lagb[q][tid] = b1;
                const T v = (T)quot(nb - b3, dg, rdR[s % 3]);
                R2[s % 3] = (double)v;
                lw[3 * WK_PS] = v;
                if (w.own && k - 3 >= S.k0 && k - 3 < S.k1) stu_nt(x + pl * (k - 3), w.col, v);
            }
            {   // plane k-4: second black
                const int m = (s + 2) % 6;
                const double dg = w.dxy[1 - q] + czp[m] + czm[m];
                const double nb =
                    WALK_NB(1 - q, lr + 3 * WK_PS, R2[(s + 2) % 3], R2[s % 3], R2[(s + 1) % 3], czp[m], czm[m]);
                const double b4 = lagb[2 + q][tid];
                lagb[2 + q][tid] = b2;
                const T v = (T)quot(nb - b4, dg, rdB[(s + 2) % 3]);
                if (w.own && k - 4 >= S.k0 && k - 4 < S.k1) stu_nt(x + F.Nh + pl * (k - 4), w.col, v);
            }
            lw[0] = (T)B0[s % 3];
            lw[WK_PS] = (T)R1[(s + 2) % 3];
            lw[2 * WK_PS] = (T)B1[(s + 1) % 3];
            lds_barrier();
        }
    }
}

// ---------------------------------------------------------------- near cells
// Units of 4 half-indices x 4 rows x 4 planes (8 x 4 x 4 cells), one per wave.
// Near units: every cell within six of a solid or membrane-adjacent cell (four
// layers spoiled by a phase, and a coarse cell of the prolongation beyond
// them), and every slot that a ghost or membrane row reads.  The listed units
// are the near ones and their neighbours, a margin of at least the four layers
// that the sequence spoils from outside: it is exact on the near units.  Units
// inside bodies (no active cell) are near, but not listed: nothing reads them,
// and their results are zero.
struct UnitPos {
    int h, j, k;   // this lane's pair of cells
    bool in, near, dead;
};
__device__ __forceinline__ UnitPos unit_pos(const Near &U, const Lv &L)
{
    const int q = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    UnitPos p{0, 0, 0, false, false, false};
    if (q >= U.n) return p;
    const int u = U.units[q], ux = u % U.nux, r = u / U.nux, uy = r % U.nuy, uz = r / U.nuy;
    const int l = threadIdx.x & 63;
    p.h = 4 * ux + (l & 3);
    p.j = 4 * uy + ((l >> 2) & 3);
    p.k = 4 * uz + (l >> 4);
    p.in = p.h < L.H && p.j < L.ny && p.k < L.nz;
    p.near = (U.bits[u] & UB_NEAR) != 0;
    p.dead = (U.bits[u] & UB_DEAD) != 0;
    return p;
}
__device__ __forceinline__ long long unit_slot(const UnitPos &p, const Lv &L)
{
    return p.h + (long long)L.H * (p.j + (long long)L.ny * p.k);
}

// first red half-sweep from zero, everything else zero; blocks past the units
// zero the membrane unknowns
template <class T>
__global__ void __launch_bounds__(NU_T) k_near_zero(Lv L, Near U, int nbu, long long nm, long long pin,
                                                    const double *__restrict__ sink, const T *__restrict__ b,
                                                    T *__restrict__ W)
{
    if ((int)blockIdx.x >= nbu) {
        const long long m = (long long)(blockIdx.x - nbu) * NU_T + threadIdx.x;
        if (m < nm) W[2 * L.Nh + m] = (T)0;
        return;
    }
    const UnitPos u = unit_pos(U, L);
    if (!u.in) return;
    const long long s = unit_slot(u, L);
    const int i = 2 * u.h + ((u.j + u.k) & 1);
    double v = 0.0;
    if (!(L.f[s] & (F_SOLID | F_MGHOST))) {
        const double dg = L.cp[0][i] + L.cm[0][i] + L.cp[1][u.j] + L.cm[1][u.j] + L.cp[2][u.k] + L.cm[2][u.k];
        double bv = ld(b, s);
        if (s == pin && sink) bv -= sink[0];
        v = -bv / dg;
    }
    st(W, s, v);
    st(W, L.Nh + s, 0.0);
}

// neighbour sum and diagonal of the lane's cell of colour c (a wall's
// neighbour is the cell's own place, with a zero coefficient)
template <class T>
__device__ __forceinline__ double near_nb(const Lv &L, const UnitPos &u, const T *W, int c, long long s, double &dg)
{
    const T *xo = W + (long long)(1 - c) * L.Nh;
    const long long pl = (long long)L.H * L.ny;
    const int p = (c + u.j + u.k) & 1, i = min(2 * u.h + p, L.nx - 1);  // (a padding slot: as its neighbour, dropped)
    const double cpx = L.cp[0][i], cmx = L.cm[0][i], cpy = L.cp[1][u.j], cmy = L.cm[1][u.j], cpz = L.cp[2][u.k],
                 cmz = L.cm[2][u.k];
    const double vxp = ld(xo, s + (i + 1 < L.nx ? p : 0)), vxm = ld(xo, s + (i > 0 ? p - 1 : 0));
    const double vyp = ld(xo, s + (u.j + 1 < L.ny ? L.H : 0)), vym = ld(xo, s - (u.j > 0 ? L.H : 0));
    const double vzp = ld(xo, s + (u.k + 1 < L.nz ? pl : 0)), vzm = ld(xo, s - (u.k > 0 ? pl : 0));
    dg = cpx + cmx + cpy + cmy + cpz + cmz;
    return cpx * vxp + cmx * vxm + cpy * vyp + cmy * vym + cpz * vzp + cmz * vzm;
}

// half-sweep of colour c over the units' regular cells
template <class T>
__global__ void __launch_bounds__(NU_T) k_near_sweep(Lv L, Near U, long long pin, const double *__restrict__ sink,
                                                     const T *__restrict__ b, T *__restrict__ W, int c)
{
    const UnitPos u = unit_pos(U, L);
    if (!u.in) return;
    const long long s = unit_slot(u, L), sc = c * L.Nh + s;
    const uint8_t f = L.f[sc];
    double bv = ld(b, sc), dg;
    const double nb = near_nb(L, u, W, c, s, dg);
    if (f & (F_SOLID | F_MGHOST)) return;
    if (sc == pin && sink) bv -= sink[0];
    st(W, sc, (nb - bv) / dg);
}

// residual and restriction of the near units' coarse cells, and their share of
// the coarse mean; irregular cells' residuals come from rsp
template <class T, class TBc>
__global__ void __launch_bounds__(NU_T) k_near_restrict(Lv F, Lv C, Near U, long long pin,
                                                        const double *__restrict__ sink, const T *__restrict__ b,
                                                        const T *__restrict__ W, const T *__restrict__ rsp,
                                                        TBc *__restrict__ bc, double *part)
{
    Acc<1> a;
    a.v[0] = 0.0;
    const UnitPos u = unit_pos(U, F);
    if (u.near) {  // per wave
        double sv = 0.0, svr = 0.0;
        if (u.in) {
            const long long s = unit_slot(u, F);
            const double wjk = F.w[1][u.j] * F.w[2][u.k];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const long long sc = c * F.Nh + s;
                const uint8_t f = F.f[sc];
                double bv = ld(b, sc), dg;
                const double nb = near_nb(F, u, W, c, s, dg), rs = ld(rsp, sc), xv = ld(W, sc);
                if (!active0(f)) continue;
                if (sc == pin && sink) bv -= sink[0];
                const double r = (f & (F_GHOST | F_MGHOST)) ? rs : bv - (nb - dg * xv);
                const double V = F.w[0][2 * u.h + ((c + u.j + u.k) & 1)] * wjk;
                sv += V;
                svr += V * r;
            }
        }
        sv += __shfl_xor(sv, 4, 64);
        svr += __shfl_xor(svr, 4, 64);
        sv += __shfl_xor(sv, 16, 64);
        svr += __shfl_xor(svr, 16, 64);
        if (u.in && !(u.j & 1) && !(u.k & 1)) {
            const int I = u.h, J = u.j >> 1, K = u.k >> 1;
            const long long sc = slot(C, (I + J + K) & 1, I >> 1, J, K);
            const double VC = C.w[0][I] * C.w[1][J] * C.w[2][K];
            st(bc, sc, sv > 0.0 ? svr / VC : 0.0);
            a.v[0] = (C.f[sc] & CM_ACT) ? VC * ld(bc, sc) : 0.0;
        }
    }
    block_reduce<1>(a, part, 0, blockIdx.x);
}

// black cells between the phases: near ones into xk, margin ones out of it
template <class T>
__global__ void __launch_bounds__(NU_T) k_near_merge(Lv L, Near U, T *__restrict__ W, T *__restrict__ xk)
{
    const UnitPos u = unit_pos(U, L);
    if (!u.in) return;
    const long long s = unit_slot(u, L);
    if (u.near) xk[s] = W[L.Nh + s];
    else W[L.Nh + s] = xk[s];
}

// prolongation onto the units' black cells and irregular red ones
template <class T>
__global__ void __launch_bounds__(NU_T) k_near_prolong(Lv L, Lv C, PMap M, Near U, const T *__restrict__ xc,
                                                       T *__restrict__ W)
{
    const UnitPos u = unit_pos(U, L);
    if (!u.in) return;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const long long s = c * L.Nh + unit_slot(u, L);
        const uint8_t f = L.f[s];
        if (!active0(f) || (c == 0 && !(f & (F_GHOST | F_MGHOST)))) continue;
        st(W, s, ld(W, s) + interp(C, M, xc, 2 * u.h + ((c + u.j + u.k) & 1), u.j, u.k));
    }
}

// the near units' results, and the membrane unknowns (blocks past the units)
template <class T>
__global__ void __launch_bounds__(NU_T) k_near_final(Lv L, Near U, int nbu, long long nm, const T *__restrict__ W,
                                                     T *__restrict__ x)
{
    if ((int)blockIdx.x >= nbu) {
        const long long m = (long long)(blockIdx.x - nbu) * NU_T + threadIdx.x;
        if (m < nm) x[2 * L.Nh + m] = W[2 * L.Nh + m];
        return;
    }
    // (U lists the near units; a unit without an active cell is not in W)
    const UnitPos u = unit_pos(U, L);
    if (!u.in) return;
    const long long s = unit_slot(u, L);
    x[s] = u.dead ? (T)0 : W[s];
    x[L.Nh + s] = u.dead ? (T)0 : W[L.Nh + s];
}

// ---- set-up of the lists: irregular and read cells per unit, the near units
// around them, the listed units
// (sixteen lanes per unit, four cell pairs each: a word per colour where rows
// and the mask's halves are aligned to it)
__global__ void __launch_bounds__(NU_T) k_unit_cells(Lv L, int nux, int nuy, long long nu, uint8_t *__restrict__ bits)
{
    const int l = threadIdx.x & 15, sh = threadIdx.x & 48;
    const long long u = ((long long)blockIdx.x * NU_T + threadIdx.x) >> 4;
    const int h = 4 * (int)(u % nux), j = 4 * (int)((u / nux) % nuy) + (l & 3),
              k = 4 * (int)(u / ((long long)nux * nuy)) + (l >> 2);
    uint32_t f = 0;
    bool act = false;
    if (u < nu && j < L.ny && k < L.nz) {
        const long long s = h + (long long)L.H * (j + (long long)L.ny * k);
        if (L.H % 4 == 0) {
            const uint32_t a = *reinterpret_cast<const uint32_t *>(L.f + s),
                           b = *reinterpret_cast<const uint32_t *>(L.f + L.Nh + s), one = 0x01010101u;
            f = a | b;
            act = ((~a | a >> 1 | ~b | b >> 1) & one) != 0;
        } else {
            for (int q = 0; q < 4 && h + q < L.H; ++q) {
                f |= L.f[s + q] | L.f[L.Nh + s + q];
                act = act || active0(L.f[s + q]) || active0(L.f[L.Nh + s + q]);
            }
        }
        f |= f >> 16;
        f |= f >> 8;
    }
    // lane bits: 0-1 row, 2-3 plane
    auto group = [&](bool v) { return (uint32_t)(__ballot(v) >> sh) & 0xffffu; };
    const uint32_t live = group(act), irr = group((f & (F_SOLID | F_MGHOST)) != 0), rd = group((f & F_RD) != 0);
    if (l == 0 && u < nu) {
        const uint32_t lowj = 0x3333u, lowk = 0x00ffu;
        uint8_t o = 0;
        if (irr & lowj & lowk) o |= 1;
        if (irr & ~lowj & lowk) o |= 2;
        if (irr & lowj & ~lowk) o |= 4;
        if (irr & ~lowj & ~lowk) o |= 8;
        if (rd) o |= UB_READ;
        if (!live) o |= UB_DEAD;
        bits[u] = o;
    }
}
__global__ void __launch_bounds__(256) k_unit_near(int nux, int nuy, int nuz, const uint8_t *__restrict__ cells,
                                                   uint8_t *__restrict__ bits)
{
    const long long nu = (long long)nux * nuy * nuz, u = (long long)blockIdx.x * 256 + threadIdx.x;
    if (u >= nu) return;
    const int x = (int)(u % nux), y = (int)((u / nux) % nuy), z = (int)(u / ((long long)nux * nuy));
    bool near = (cells[u] & UB_READ) != 0;
    // within eight cells in x, six (two rows or planes of the unit after the next) in y and z
    for (int dz = -2; dz <= 2; ++dz)
        for (int dy = -2; dy <= 2; ++dy) {
            const int yy = y + dy, zz = z + dz;
            if (yy < 0 || yy >= nuy || zz < 0 || zz >= nuz) continue;
            uint8_t want = UB_IRR;
            if (dy == -2) want &= 2 | 8;
            if (dy == 2) want &= 1 | 4;
            if (dz == -2) want &= 4 | 8;
            if (dz == 2) want &= 1 | 2;
            for (int dx = -1; dx <= 1; ++dx) {
                const int xx = x + dx;
                if (xx >= 0 && xx < nux) near |= (cells[xx + (long long)nux * (yy + (long long)nuy * zz)] & want) != 0;
            }
        }
    bits[u] = (near ? UB_NEAR : 0) | (cells[u] & UB_DEAD);
}
__global__ void __launch_bounds__(256) k_unit_list(int nux, int nuy, int nuz, const uint8_t *__restrict__ near,
                                                   uint8_t *__restrict__ bits)
{
    const long long nu = (long long)nux * nuy * nuz, u = (long long)blockIdx.x * 256 + threadIdx.x;
    if (u >= nu) return;
    const int x = (int)(u % nux), y = (int)((u / nux) % nuy), z = (int)(u / ((long long)nux * nuy));
    uint8_t any = 0;
    for (int q = 0; q < 27; ++q) {
        const int xx = x + q % 3 - 1, yy = y + (q / 3) % 3 - 1, zz = z + q / 9 - 1;
        if (xx >= 0 && xx < nux && yy >= 0 && yy < nuy && zz >= 0 && zz < nuz)
            any |= near[xx + (long long)nux * (yy + (long long)nuy * zz)];
    }
    bits[u] = (near[u] & (UB_NEAR | UB_DEAD)) | ((any & UB_NEAR) && !(near[u] & UB_DEAD) ? UB_LIST : 0);
}

}  // namespace ibm
