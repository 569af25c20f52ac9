// Cell classification ("iblanking", Sec. 2.5 module 1) on gfx950.
//
// Closed bodies: a cell is solid iff the ray along +x through its centre has
// crossed the body an odd number of times before reaching the centre.
// Membranes: the link between two face neighbours is cut iff an odd number of
// membrane triangles cross it (rays along x, y and z).  All predicates are
// exact int64 arithmetic on lattice coordinates q(v) = floor((v-lo)*S + 0.5),
// S = 2^16 / longest domain edge; a point exactly on a projected edge belongs
// to the triangle for which that edge is "top-left" (d_w < 0, or d_w == 0 and
// d_u > 0), the same as perturbing the ray by (+e, +e^2).
//
// GPU form: up to sixteen lanes per triangle walk the rays its projected bounding
// box covers, find the first cell beyond the crossing by binary search and flip
// one bit of a toggle bitset with an integer atomic XOR; one wavefront per ray
// then turns toggles into parity.  A closed body's toggles cover its own box of
// cells, so that many bodies share one launch of each kind and one bitset.
// Twenty bodies at 384^3, body after body with a bitset of the whole grid and
// one thread per triangle and per ray: 2.2 ms of kernels and 46 copies; now
// 34 us and one copy.  This file is compiled with -ffp-contract=off so that
// the quantisation, on the host and on the device, rounds exactly as written.

#include "common.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace ibm {

HostGrid read_grid(const ibm_grid *g)
{
    IBM_REQUIRE(g != nullptr, IBM_EINVAL, "null grid");
    HostGrid h;
    h.n[0] = g->nx; h.n[1] = g->ny; h.n[2] = g->nz;
    const double *f[3] = {g->xf, g->yf, g->zf};
    for (int d = 0; d < 3; ++d) {
        IBM_REQUIRE(h.n[d] >= 4, IBM_EINVAL, "grid dimension below 4");
        IBM_REQUIRE(f[d] != nullptr, IBM_EINVAL, "null face array");
        h.f[d].assign(f[d], f[d] + h.n[d] + 1);
        for (int i = 0; i < h.n[d]; ++i)
            IBM_REQUIRE(h.f[d][i + 1] > h.f[d][i], IBM_EINVAL, "face coordinates not strictly increasing");
    }
    IBM_REQUIRE((int64_t)h.n[0] * h.n[1] * h.n[2] < ((int64_t)1 << 31), IBM_EINVAL, "more than 2^31 cells");
    return h;
}

namespace {

struct Lat {
    double lo[3];
    double S;
};

__host__ __device__ __forceinline__ long long qnt(double v, double lo, double S)
{
    double t = (v - lo) * S;
    t = t + 0.5;
    return (long long)floor(t);
}

__global__ void k_fill_u32(uint32_t *a, long long n, uint32_t v)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n; i += (long long)gridDim.x * blockDim.x) a[i] = v;
}

__global__ void k_fill_u8(uint8_t *a, long long n, uint8_t v)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n; i += (long long)gridDim.x * blockDim.x) a[i] = v;
}

__device__ __forceinline__ long long o2(const long long *U, const long long *V, const long long *P, int u, int w)
{
    return (V[u] - U[u]) * (P[w] - U[w]) - (V[w] - U[w]) * (P[u] - U[u]);
}

__device__ __forceinline__ bool owns(const long long *U, const long long *V, const long long *P, int u, int w)
{
    long long e = o2(U, V, P, u, w);
    if (e != 0) return e > 0;
    long long du = V[u] - U[u], dw = V[w] - U[w];
    return dw < 0 || (dw == 0 && du > 0);
}

__device__ __forceinline__ int lower_bound_ll(const long long *a, int n, long long v)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        int m = (lo + hi) >> 1;
        if (a[m] < v) lo = m + 1; else hi = m;
    }
    return lo;
}

// One body of a launch.  Closed: its toggles are one bit per cell of its box
// [at, at + ext), x fastest, from word w0 of the bitset; every cell that a
// crossing of the body can toggle lies in the box.  Its blocks of the two
// launches are [rays, rays + nray) per axis and [par, par + npar).
struct RayBody {
    const double *v;     // vertices
    const int32_t *tri;
    int nt, closed;
    int at[3], ext[3];
    long long w0;
    int lanes;           // per triangle: log2
    int rays, nray, par, npar;
};
constexpr int RAY_BODIES = 40;  // per launch: the descriptions travel as a kernel argument (3.3 of 4 KiB)
struct RayBatch {
    Lat lat;
    const long long *qc[3];  // lattice centres per axis
    int n[3], nb;
    uint32_t *tog, *cut[3];
    RayBody body[RAY_BODIES];
};
// Lanes per triangle: as many as a triangle has rays on average (its box holds
// about four times its share of the body's projection), at most sixteen.  A
// call at 256^3 with a body of 200 thousand triangles: 714 us with sixteen for
// every triangle, 638 with this; with 2 million 5.7 and 5.0 ms.
constexpr int RAY_LANES = 4;         // log2
constexpr int PAR_BLOCKS = 1 << 16;  // of one body: its wavefronts take several rays each beyond

// body of the launch that block i belongs to: the last whose first block (m) is not behind it
__device__ __forceinline__ int body_of(const RayBatch &A, int RayBody::*m, int i)
{
    int lo = 0, hi = A.nb - 1;
    while (lo < hi) {
        const int q = (lo + hi + 1) >> 1;
        if (A.body[q].*m <= i) lo = q; else hi = q - 1;
    }
    return lo;
}

// Triangles of a body along one axis (closed bodies: x only): every covered ray
// flips the bit of the first cell whose centre lies strictly beyond the crossing
// (closed), or the link just before it (membrane).  Each body has the blocks
// that its triangles need, whatever mesh stands beside it in the launch.
__global__ void __launch_bounds__(256) k_rays(RayBatch A)
{
    const RayBody &B = A.body[body_of(A, &RayBody::rays, (int)blockIdx.x)];
    const int q0 = (int)blockIdx.x - B.rays, d = q0 / B.nray, lanes = 1 << B.lanes;
    const uint32_t th = (uint32_t)(q0 - d * B.nray) * 256u + threadIdx.x;
    const int t = (int)(th >> B.lanes), lane = (int)th & (lanes - 1);
    if (t >= B.nt) return;
    const int u = (d + 1) % 3, w = (d + 2) % 3;
    long long P[3][3];
    for (int m = 0; m < 3; ++m) {
        const double *v = B.v + 3 * (long long)B.tri[3 * (long long)t + m];
        for (int c = 0; c < 3; ++c) P[m][c] = qnt(v[c], A.lat.lo[c], A.lat.S);
    }
    const long long *P0 = P[0], *P1 = P[1], *P2 = P[2];
    long long e1[3], e2[3], Nn[3];
    for (int c = 0; c < 3; ++c) { e1[c] = P1[c] - P0[c]; e2[c] = P2[c] - P0[c]; }
    Nn[0] = e1[1] * e2[2] - e1[2] * e2[1];
    Nn[1] = e1[2] * e2[0] - e1[0] * e2[2];
    Nn[2] = e1[0] * e2[1] - e1[1] * e2[0];
    const long long a = Nn[d];
    if (a == 0) return;
    // counter-clockwise order in (u, w)
    long long Bv[3], Cv[3];
    for (int c = 0; c < 3; ++c) {
        Bv[c] = a < 0 ? P2[c] : P1[c];
        Cv[c] = a < 0 ? P1[c] : P2[c];
    }
    long long umin = min(P0[u], min(P1[u], P2[u])), umax = max(P0[u], max(P1[u], P2[u]));
    long long wmin = min(P0[w], min(P1[w], P2[w])), wmax = max(P0[w], max(P1[w], P2[w]));
    const int nu = A.n[u], nw = A.n[w], nr = A.n[d];
    const long long *qu = A.qc[u], *qw = A.qc[w], *qr = A.qc[d];
    const long long sa = a > 0 ? 1 : -1, aa = a > 0 ? a : -a;
    const int ia0 = lower_bound_ll(qu, nu, umin), ib0 = lower_bound_ll(qw, nw, wmin);
    const int na = lower_bound_ll(qu, nu, umax + 1) - ia0, nb = lower_bound_ll(qw, nw, wmax + 1) - ib0;
    const long long rays = (long long)na * nb;
    const long long st[3] = {1, A.n[0], (long long)A.n[0] * A.n[1]};
    for (long long r = lane; r < rays; r += lanes) {
        const int ia = ia0 + (int)(r / nb), ib = ib0 + (int)(r % nb);
        long long X[3];
        X[d] = 0;
        X[u] = qu[ia];
        X[w] = qw[ib];
        if (!owns(P0, Bv, X, u, w) || !owns(Bv, Cv, X, u, w) || !owns(Cv, P0, X, u, w)) continue;
        // first i with (qr[i]-A_d)|a| + sign(a) K > 0 (centre strictly beyond the crossing)
        long long K = (X[u] - P0[u]) * Nn[u] + (X[w] - P0[w]) * Nn[w];
        long long sk = sa * K;
        int lo = 0, hi = nr;
        while (lo < hi) {
            int m = (lo + hi) >> 1;
            if ((qr[m] - P0[d]) * aa + sk > 0) hi = m; else lo = m + 1;
        }
        if (B.closed) {  // d == 0, so u is y and w is z
            const int x = lo - B.at[0], y = ia - B.at[1], z = ib - B.at[2];
            if (lo < nr && x >= 0 && x < B.ext[0] && y >= 0 && y < B.ext[1] && z >= 0 && z < B.ext[2]) {
                const long long q = x + (long long)B.ext[0] * (y + (long long)B.ext[1] * z);
                atomicXor(&A.tog[B.w0 + (q >> 5)], 1u << (q & 31));
            }
        } else if (lo >= 1 && lo <= nr - 1) {
            const long long cell = (long long)ia * st[u] + (long long)ib * st[w] + (long long)(lo - 1) * st[d];
            atomicXor(&A.cut[d][cell >> 5], 1u << (cell & 31));
        }
    }
}

// One wavefront per x-ray of a closed body's box: prefix parity of the
// toggles; odd cells become solid, past the box too if the mesh is open.
// (Bodies of one launch that overlap store the same byte.)
__global__ void __launch_bounds__(256) k_ray_parity(RayBatch A, uint8_t *flags)
{
    const RayBody &B = A.body[body_of(A, &RayBody::par, (int)blockIdx.x)];
    const int lane = threadIdx.x & 63, nx = A.n[0];
    const long long rays = (long long)B.ext[1] * B.ext[2];
    for (long long r = 4LL * ((int)blockIdx.x - B.par) + (threadIdx.x >> 6); r < rays; r += 4LL * B.npar) {
        const int y = B.at[1] + (int)(r % B.ext[1]), z = B.at[2] + (int)(r / B.ext[1]);
        uint8_t *row = flags + (long long)nx * (y + (long long)A.n[1] * z);
        int carry = 0;
        for (int x0 = 0; x0 < B.ext[0]; x0 += 64) {
            const int x = x0 + lane;
            const long long q = r * B.ext[0] + x;
            const bool on = x < B.ext[0] && ((A.tog[B.w0 + (q >> 5)] >> (q & 31)) & 1u);
            const unsigned long long m = __ballot(on);
            const unsigned long long upto = lane == 63 ? ~0ull : (1ull << (lane + 1)) - 1ull;
            if (x < B.ext[0] && ((carry + __popcll(m & upto)) & 1)) row[B.at[0] + x] = F_SOLID;
            carry += __popcll(m);
        }
        if (carry & 1)
            for (int x = B.at[0] + B.ext[0] + lane; x < nx; x += 64) row[x] = F_SOLID;
    }
}

__device__ __forceinline__ bool bit(const uint32_t *b, long long c) { return (b[c >> 5] >> (c & 31)) & 1u; }

// Ghost, membrane-ghost and cut bits from the solid bits and the raw cut
// toggles, with the counts (solid, ghost, membrane ghost, cut links) and the
// first cell for the pin.  Bound: the flags, read and written once.  W4: four
// cells of a row to a thread as the bytes of a word (rows of a multiple of
// four cells, flags aligned to four bytes); one byte per thread, the counts
// and the pin in passes of their own took 315 us at 384^3, this 83.
struct FlagArgs {
    uint8_t *flags;
    const uint32_t *cut[3];
    int n[3], has_membrane;
    long long N;
    unsigned long long *pin, *cnt;
};
template <bool W4>
__global__ void __launch_bounds__(256) k_flags(FlagArgs A)
{
    const int nx = A.n[0], ny = A.n[1], nz = A.n[2];
    const uint32_t one = 0x01010101u;
    unsigned long long c[4] = {0, 0, 0, 0}, pin = ~0ull;
    const long long items = W4 ? A.N / 4 : A.N;
    for (long long q = (long long)blockIdx.x * 256 + threadIdx.x; q < items; q += (long long)gridDim.x * 256) {
        const uint32_t p = (uint32_t)(W4 ? 4 * q : q);
        const uint32_t row = p / (uint32_t)nx, i = p - row * (uint32_t)nx, k = row / (uint32_t)ny,
                       j = row - k * (uint32_t)ny;
        const uint32_t st[3] = {1, (uint32_t)nx, (uint32_t)nx * (uint32_t)ny};
        const bool lo[3] = {i > 0, j > 0, k > 0}, hi[3] = {(int)i + (W4 ? 4 : 1) < nx, (int)j + 1 < ny, (int)k + 1 < nz};
        if constexpr (W4) {
            auto solid = [&](uint32_t at) { return *reinterpret_cast<const uint32_t *>(A.flags + at) & one; };
            auto spread = [&](uint32_t b) { return ((b & 0xfu) * 0x00204081u) & one; };
            auto four = [&](const uint32_t *b, uint32_t at) { return b[at >> 5] >> (at & 31); };
            const uint32_t S = solid(p);
            // the neighbours' solid bits (outside the domain: as if solid)
            uint32_t sp[3], sm[3];
            sp[0] = (S >> 8) | ((hi[0] ? solid(p + 4) & 1u : 1u) << 24);
            sm[0] = (S << 8) | (lo[0] ? solid(p - 4) >> 24 : 1u);
            for (int d = 1; d < 3; ++d) {
                sp[d] = hi[d] ? solid(p + st[d]) : one;
                sm[d] = lo[d] ? solid(p - st[d]) : one;
            }
            uint32_t f = S | (S & ~(sp[0] & sm[0] & sp[1] & sm[1] & sp[2] & sm[2])) << 1, mg = 0;
            if (A.has_membrane && S != one) {
                for (int d = 0; d < 3; ++d) {
                    const uint32_t own = four(A.cut[d], p);
                    uint32_t prev;
                    if (d == 0) prev = (own << 1) | (lo[0] ? (A.cut[0][(p - 1) >> 5] >> ((p - 1) & 31)) & 1u : 0u);
                    else prev = lo[d] ? four(A.cut[d], p - st[d]) : 0u;
                    const uint32_t link = spread(own) & ~S & ~sp[d];
                    f |= link << (4 + d);
                    mg |= link | (spread(prev) & ~S & ~sm[d]);
                }
                f |= mg << 2;
                c[2] += __popc(mg);
                c[3] += __popc(f & 0x70707070u);
            }
            c[0] += __popc(S);
            c[1] += __popc(f & (one << 1));
            const uint32_t ok = one & ~(S | mg);
            if (ok && pin == ~0ull) pin = p + (uint32_t)((__ffs(ok) - 1) >> 3);
            *reinterpret_cast<uint32_t *>(A.flags + p) = f;
        } else {
            uint8_t f = A.flags[p] & F_SOLID;
            if (f) {
                bool g = false;
                for (int d = 0; d < 3; ++d) {
                    if (lo[d] && !(A.flags[p - st[d]] & F_SOLID)) g = true;
                    if (hi[d] && !(A.flags[p + st[d]] & F_SOLID)) g = true;
                }
                if (g) f |= F_GHOST;
            } else if (A.has_membrane) {
                for (int d = 0; d < 3; ++d) {
                    if (hi[d] && bit(A.cut[d], p) && !(A.flags[p + st[d]] & F_SOLID)) f |= (uint8_t)(F_CUTX << d);
                    if (lo[d] && bit(A.cut[d], p - st[d]) && !(A.flags[p - st[d]] & F_SOLID)) f |= F_MGHOST;
                }
                if (f & 0x70) f |= F_MGHOST;
            }
            c[0] += f & F_SOLID;
            c[1] += (f >> 1) & 1;
            c[2] += (f >> 2) & 1;
            c[3] += __popc(f & 0x70u);
            if (!(f & (F_SOLID | F_MGHOST)) && pin == ~0ull) pin = p;
            A.flags[p] = f;
        }
    }
    __shared__ unsigned long long s[4][5];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int o = 32; o > 0; o >>= 1) {
        for (int q = 0; q < 4; ++q) c[q] += __shfl_xor(c[q], o, 64);
        pin = min(pin, (unsigned long long)__shfl_xor(pin, o, 64));
    }
    if (lane == 0) {
        for (int q = 0; q < 4; ++q) s[wid][q] = c[q];
        s[wid][4] = pin;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const unsigned long long v = s[0][threadIdx.x] + s[1][threadIdx.x] + s[2][threadIdx.x] + s[3][threadIdx.x];
        if (v) atomicAdd(&A.cnt[threadIdx.x], v);
    } else if (threadIdx.x == 4) {
        const unsigned long long v = min(min(s[0][4], s[1][4]), min(s[2][4], s[3][4]));
        if (v != ~0ull) atomicMin(A.pin, v);
    }
}

__global__ void k_set_pin(uint8_t *flags, const unsigned long long *pin, long long N)
{
    if (threadIdx.x == 0 && blockIdx.x == 0 && *pin < (unsigned long long)N) flags[*pin] |= F_PIN;
}

// counters of one classification: pin (minimum), then the four counts
__global__ void k_init_counters(unsigned long long *dev)
{
    if (threadIdx.x < 5) dev[threadIdx.x] = threadIdx.x == 0 ? ~0ull : 0ull;
}

// Device scratch of one classification, carved from one region in 256-byte
// aligned pieces.  A carve with a null base only measures.
struct Carve {
    char *base = nullptr;
    size_t off = 0;
    template <class T>
    T *take(size_t n)
    {
        off = (off + 255) / 256 * 256;
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off += n * sizeof(T);
        return p;
    }
};

// The scratch a call is charged with: per axis the faces and the quantised
// centres; the toggle bitset and a byte per ray (closed bodies); three
// cut-link bitsets (membranes); per body its vertices, triangles and quantised
// vertices; five counters.  Callers see this size and are refused by it; what
// is carved from it (below) is no larger: the same pieces without the faces,
// the bytes per ray and the quantised vertices, the bodies' without padding.
size_t classify_bytes(const HostGrid &g, const ibm_body *bodies, int n_body, bool any_closed, bool any_mem)
{
    Carve C;
    const long long N = (long long)g.n[0] * g.n[1] * g.n[2];
    const size_t words = (size_t)((N + 31) / 32 + 1);
    for (int d = 0; d < 3; ++d) {
        (void)C.take<double>(g.n[d] + 1);
        (void)C.take<long long>(g.n[d]);
    }
    if (any_closed) {
        (void)C.take<uint32_t>(words);
        (void)C.take<uint8_t>((size_t)g.n[1] * g.n[2]);
    }
    if (any_mem)
        for (int d = 0; d < 3; ++d) (void)C.take<uint32_t>(words);
    for (int b = 0; b < n_body; ++b) {
        (void)C.take<double>((size_t)3 * bodies[b].n_vert);
        (void)C.take<int32_t>((size_t)3 * bodies[b].n_tri);
        (void)C.take<long long>((size_t)3 * bodies[b].n_vert);
    }
    (void)C.take<unsigned long long>(5);
    return C.off;
}

// What a classification uses: centres and the small bodies' vertices and
// triangles (one copy from the host), the large bodies' (a copy each from where
// the caller holds them), then the bitsets and the counters.
// Largest body of the common copy.  Twenty bodies of 368 KB at 256^3: 1.09 ms a
// call staged, 1.22 with two copies each; of 750 KB 2.19 and 1.92; one of 48 MB
// 15.6 and 5.0.
constexpr size_t STAGE_BYTES = 512 << 10;
size_t body_bytes(const ibm_body &B) { return 24 * (size_t)B.n_vert + 12 * (size_t)B.n_tri; }
struct ClassifyScratch {
    long long *qc[3];
    double *vert[2];  // small, large
    int32_t *tri[2];
    size_t input;  // bytes up to here come in the one copy
    uint32_t *tog = nullptr, *cut[3] = {nullptr, nullptr, nullptr};
    unsigned long long *dev;
};
ClassifyScratch carve_classify(Carve &C, const HostGrid &g, const size_t nv[2], const size_t nt[2], bool any_closed,
                               bool any_mem)
{
    ClassifyScratch S;
    const size_t words = (size_t)(((long long)g.n[0] * g.n[1] * g.n[2] + 31) / 32 + 1);
    for (int d = 0; d < 3; ++d) S.qc[d] = C.take<long long>(g.n[d]);
    S.vert[0] = C.take<double>(3 * nv[0]);
    S.tri[0] = C.take<int32_t>(3 * nt[0]);
    S.input = C.off;
    S.vert[1] = C.take<double>(3 * nv[1]);
    S.tri[1] = C.take<int32_t>(3 * nt[1]);
    if (any_closed) S.tog = C.take<uint32_t>(words);
    if (any_mem)
        for (int d = 0; d < 3; ++d) S.cut[d] = C.take<uint32_t>(words);
    S.dev = C.take<unsigned long long>(5);
    return S;
}

struct ClassifyPlan {
    HostGrid g;
    bool any_closed = false, any_mem = false;
    size_t bytes = 0;  // device scratch the classification is charged with
    struct Box {
        double lo[3], hi[3];
    };
    std::vector<Box> box;  // of each body's vertices
};

// Argument checks and the scratch size; nothing touches the device.
ClassifyPlan plan_classify(const ibm_grid *grid, const ibm_body *bodies, int n_body, const uint8_t *flags)
{
    ClassifyPlan P;
    P.g = read_grid(grid);
    const HostGrid &g = P.g;
    IBM_REQUIRE(flags != nullptr, IBM_EINVAL, "null flags");
    IBM_REQUIRE(n_body >= 0 && (n_body == 0 || bodies != nullptr), IBM_EINVAL, "bad body list");
    double least[3], most[3];
    for (int d = 0; d < 3; ++d) {
        const double Ld = g.f[d][g.n[d]] - g.f[d][0];
        least[d] = g.f[d][0] - Ld;
        most[d] = g.f[d][g.n[d]] + Ld;
    }
    for (int b = 0; b < n_body; ++b) {
        const ibm_body &B = bodies[b];
        IBM_REQUIRE(B.kind == IBM_KIND_CLOSED || B.kind == IBM_KIND_MEMBRANE, IBM_EINVAL, "bad body kind");
        (B.kind == IBM_KIND_CLOSED ? P.any_closed : P.any_mem) = true;
        IBM_REQUIRE(B.n_vert >= 3 && B.n_tri >= 1 && B.vert && B.tri, IBM_EINVAL, "empty body");
        ClassifyPlan::Box X;
        for (int d = 0; d < 3; ++d) X.lo[d] = X.hi[d] = B.vert[d];
        bool inside = true;
        for (int v = 0; v < B.n_vert; ++v)
            for (int d = 0; d < 3; ++d) {
                const double x = B.vert[3 * (size_t)v + d];
                inside = inside && std::isfinite(x) && x >= least[d] && x <= most[d];
                X.lo[d] = std::min(X.lo[d], x);
                X.hi[d] = std::max(X.hi[d], x);
            }
        IBM_REQUIRE(inside, IBM_EINVAL, "body vertex more than one domain length outside the domain");
        P.box.push_back(X);
        for (int t = 0; t < 3 * B.n_tri; ++t)
            IBM_REQUIRE(B.tri[t] >= 0 && B.tri[t] < B.n_vert, IBM_EGEOM, "triangle index out of range");
    }
    P.bytes = classify_bytes(g, bodies, n_body, P.any_closed, P.any_mem);
    return P;
}

// Host orchestration of the classification; every device buffer of the call
// comes from `scratch` (at least plan.bytes, 256-byte aligned).
void classify_with(const ClassifyPlan &plan, const ibm_body *bodies, int n_body, uint8_t *flags, ibm_class_stats *st,
              char *scratch, hipStream_t s)
{
    const HostGrid &g = plan.g;
    const long long N = (long long)g.n[0] * g.n[1] * g.n[2];
    double L = 0.0;
    for (int d = 0; d < 3; ++d) L = std::max(L, g.f[d][g.n[d]] - g.f[d][0]);
    Lat lat;
    lat.S = 65536.0 / L;
    for (int d = 0; d < 3; ++d) lat.lo[d] = g.f[d][0];
    size_t nv[2] = {0, 0}, nt[2] = {0, 0};
    for (int b = 0; b < n_body; ++b) {
        const int big = body_bytes(bodies[b]) > STAGE_BYTES;
        nv[big] += bodies[b].n_vert;
        nt[big] += bodies[b].n_tri;
    }
    Carve C;
    C.base = scratch;
    const ClassifyScratch S = carve_classify(C, g, nv, nt, plan.any_closed, plan.any_mem);
    IBM_REQUIRE(C.off <= plan.bytes, IBM_EINVAL, "classification scratch above its plan");

    std::vector<char> image(S.input);
    std::vector<long long> qc[3];
    for (int d = 0; d < 3; ++d) {
        qc[d].resize(g.n[d]);
        for (int i = 0; i < g.n[d]; ++i) qc[d][i] = qnt(0.5 * (g.f[d][i] + g.f[d][i + 1]), lat.lo[d], lat.S);
        std::memcpy(image.data() + ((char *)S.qc[d] - scratch), qc[d].data(), g.n[d] * sizeof(long long));
    }
    const double *dv[2] = {S.vert[0], S.vert[1]};
    const int32_t *dt[2] = {S.tri[0], S.tri[1]};
    std::vector<RayBody> body(n_body);
    for (int b = 0; b < n_body; ++b) {
        const ibm_body &B = bodies[b];
        const int big = body_bytes(B) > STAGE_BYTES;
        RayBody &R = body[b];
        R = RayBody{dv[big], dt[big], B.n_tri, B.kind == IBM_KIND_CLOSED, {0, 0, 0}, {0, 0, 0}, 0, 0, 0, 0, 0, 0};
        dv[big] += 3 * (size_t)B.n_vert;
        dt[big] += 3 * (size_t)B.n_tri;
        const size_t bv = (size_t)3 * B.n_vert * sizeof(double), bt = (size_t)3 * B.n_tri * sizeof(int32_t);
        if (big) {
            IBM_HIP(hipMemcpyAsync((void *)R.v, B.vert, bv, hipMemcpyHostToDevice, s));
            IBM_HIP(hipMemcpyAsync((void *)R.tri, B.tri, bt, hipMemcpyHostToDevice, s));
        } else {
            std::memcpy(image.data() + ((const char *)R.v - scratch), B.vert, bv);
            std::memcpy(image.data() + ((const char *)R.tri - scratch), B.tri, bt);
        }
    }
    IBM_HIP(hipMemcpyAsync(scratch, image.data(), S.input, hipMemcpyHostToDevice, s));
    k_fill_u8<<<2048, 256, 0, s>>>(flags, N, 0);
    const long long words = (N + 31) / 32 + 1;
    for (int d = 0; d < 3; ++d)
        if (S.cut[d]) k_fill_u32<<<2048, 256, 0, s>>>(S.cut[d], words, 0u);
    IBM_LAUNCH_CHECK();

    // bodies in order, as many to a launch as descriptions and toggles fit
    RayBatch A;
    A.lat = lat;
    A.tog = S.tog;
    for (int d = 0; d < 3; ++d) {
        A.qc[d] = S.qc[d];
        A.n[d] = g.n[d];
        A.cut[d] = S.cut[d];
    }
    A.nb = 0;
    int rays = 0, par = 0;  // blocks of the two launches
    long long used = 0;     // toggle words
    auto flush = [&] {
        if (!A.nb) return;
        if (used) k_fill_u32<<<(unsigned)std::min<long long>(2048, (used + 255) / 256), 256, 0, s>>>(S.tog, used, 0u);
        k_rays<<<rays, 256, 0, s>>>(A);
        if (par) k_ray_parity<<<par, 256, 0, s>>>(A, flags);
        IBM_LAUNCH_CHECK();
        A.nb = rays = par = 0;
        used = 0;
    };
    for (int b = 0; b < n_body; ++b) {
        RayBody &R = body[b];
        // a crossing lies within the body's lattice box, the first centre
        // beyond it at most one past the last centre inside
        for (int d = 0; d < 3; ++d) {
            const auto &q = qc[d];
            const int a = (int)(std::lower_bound(q.begin(), q.end(), qnt(plan.box[b].lo[d], lat.lo[d], lat.S)) - q.begin());
            const int e = (int)(std::upper_bound(q.begin(), q.end(), qnt(plan.box[b].hi[d], lat.lo[d], lat.S)) - q.begin());
            R.at[d] = a;
            R.ext[d] = std::max(0, std::min(g.n[d], R.closed && d == 0 ? e + 1 : e) - a);
        }
        const long long x = R.ext[0], y = R.ext[1], z = R.ext[2], box = x * y * z;
        if (R.closed && !box) continue;  // no ray meets it within the domain
        const long long need = R.closed ? (box + 31) / 32 : 0, proj = R.closed ? y * z : std::max(y * z, std::max(z * x, x * y));
        while (R.lanes < RAY_LANES && ((long long)R.nt << R.lanes) < std::min(4 * proj, 1LL << 28)) ++R.lanes;
        R.nray = (int)cdiv((long long)R.nt << R.lanes, 256);
        R.npar = R.closed ? (int)std::min<long long>((y * z + 3) / 4, PAR_BLOCKS) : 0;
        // (2^23 blocks: a launch of fewer than 2^32 threads, which is the limit)
        if (A.nb == RAY_BODIES || used + need > words || (A.nb && rays + 3LL * R.nray > 1 << 23)) flush();
        R.w0 = used;
        R.rays = rays;
        R.par = par;
        used += need;
        rays += R.closed ? R.nray : 3 * R.nray;
        par += R.npar;
        A.body[A.nb++] = R;
    }
    flush();
    k_init_counters<<<1, 64, 0, s>>>(S.dev);
    const FlagArgs F{flags, {S.cut[0], S.cut[1], S.cut[2]}, {g.n[0], g.n[1], g.n[2]}, plan.any_mem ? 1 : 0, N, S.dev, S.dev + 1};
    if (g.n[0] % 4 == 0 && ((uintptr_t)flags & 3) == 0) k_flags<true><<<std::min(2048u, cdiv(N / 4, 256)), 256, 0, s>>>(F);
    else k_flags<false><<<std::min(2048u, cdiv(N, 256)), 256, 0, s>>>(F);
    k_set_pin<<<1, 64, 0, s>>>(flags, S.dev, N);
    IBM_LAUNCH_CHECK();
    unsigned long long h[5];
    IBM_HIP(hipMemcpyAsync(h, S.dev, 5 * 8, hipMemcpyDeviceToHost, s));
    // the counts are needed on the host; this also ends every use of the scratch
    IBM_HIP(hipStreamSynchronize(s));
    IBM_REQUIRE(h[0] < (unsigned long long)N, IBM_EGEOM, "no fluid cell outside the membrane ghosts");
    if (st) {
        st->pin = (int64_t)h[0];
        st->n_solid = (int64_t)h[1];
        st->n_ghost = (int64_t)h[2];
        st->n_mghost = (int64_t)h[3];
        st->n_cut_links = (int64_t)h[4];
    }
}

// Scratch of ibm_classify_noalloc: one array per device, for the life of the
// process.  Its host-side name is not a device address; the address comes
// from hipGetSymbolAddress, once per device.
constexpr size_t NOALLOC_BYTES = (size_t)IBM_CLASSIFY_NOALLOC_MAX_BYTES;
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

std::mutex g_scratch_mu;
std::vector<char *> g_scratch_ptr;  // per device ordinal, null until looked up

char *device_scratch()
{
    int dev = 0;
    IBM_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if ((int)g_scratch_ptr.size() <= dev) g_scratch_ptr.resize(dev + 1, nullptr);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        IBM_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        IBM_REQUIRE(ptr != nullptr, IBM_EHIP, "no device address for the classification scratch");
        g_scratch_ptr[dev] = (char *)ptr;
    }
    return g_scratch_ptr[dev];
}

}  // namespace

void classify(const ibm_grid *grid, const ibm_body *bodies, int n_body, uint8_t *flags, ibm_class_stats *st,
              hipStream_t s)
{
    const ClassifyPlan plan = plan_classify(grid, bodies, n_body, flags);
    DBuf<char> ws(plan.bytes);
    classify_with(plan, bodies, n_body, flags, st, ws.p, s);
}

}  // namespace ibm

extern "C" int32_t ibm_classify(const ibm_grid *grid, const ibm_body *bodies, int32_t n_body, uint8_t *flags_dev,
                                ibm_class_stats *st, void *stream)
{
    return ibm::guarded([&] { ibm::classify(grid, bodies, n_body, flags_dev, st, (hipStream_t)stream); });
}

extern "C" int32_t ibm_classify_noalloc(const ibm_grid *grid, const ibm_body *bodies, int32_t n_body,
                                        uint8_t *flags_dev, ibm_class_stats *st, size_t *scratch_bytes, void *stream)
{
    return ibm::guarded([&] {
        const ibm::ClassifyPlan plan = ibm::plan_classify(grid, bodies, n_body, flags_dev);
        if (scratch_bytes) *scratch_bytes = plan.bytes;
        IBM_REQUIRE(plan.bytes <= ibm::NOALLOC_BYTES, IBM_ENOMEM,
                    "ibm_classify_noalloc: this grid and these bodies need " + std::to_string(plan.bytes) +
                        " bytes of scratch, above its fixed " + std::to_string(ibm::NOALLOC_BYTES) +
                        " (use ibm_classify)");
        ibm::classify_with(plan, bodies, n_body, flags_dev, st, ibm::device_scratch(), (hipStream_t)stream);
    });
}
