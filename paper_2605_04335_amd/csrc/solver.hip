// PPE solver (Sec. 2.1: BiCGStab on the pressure Poisson equation; Sec. 2.5
// module 3: matrix-free bulk plus ELLPACK rows for the irregular part) with a
// geometric-multigrid V-cycle as right preconditioner, FP64 or mixed
// precision (FP32 inner BiCGSTAB and V-cycle, BF16 coarse right-hand sides,
// FP64 iterative refinement).
//
// Pinned system: the singular Neumann operator has its first fluid
// non-membrane-ghost cell's row replaced by -s x = 0.  The preconditioner is
// V-cycle(b') with b' = b minus the volume-weighted net of b placed at the
// pin as a sink, run on the unpinned operator, followed by a shift of its
// output to a zero pin value; the shift is folded into the consumers (the
// operator writes 0 on the pin row, the x update subtracts the pin values).
//
// All vectors are held in the red/black split layout (kernels.hpp); the C
// ABI takes and returns natural x-fastest arrays, converted at the boundary.

#include "kernels.hpp"
#include "rows.hpp"
#include "setup.hpp"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <type_traits>

namespace ibm {
namespace {

// The Krylov vector updates run one block per 256 groups of four unknowns up
// to W4MAXB blocks (a 512^3 vector: 131072 blocks, one group per thread):
// against a 4096-block walk this measured 3% (x/r update) to 11% (p update)
// faster in FP64 and 11-14% in FP32.  Their block partials set the stride.
constexpr int W4MAXB = 131072;
constexpr int PSTRIDE = W4MAXB + 2048;  // partial slots per reduction: stencil or walk blocks, then sparse blocks
constexpr int XB = 1024;               // cap on blocks of the sparse row kernels

// Coarse levels up to this size smooth on bricks (fused.hpp).  At 64^3 a phase
// takes 19 us against 23 to 29 us of one-sweep launches; at 128^3 the bricks'
// eightfold recomputation alone is eight times that work, against 34 to 37 us.
constexpr long long BRICK_MAX_CELLS = 300000;
// A level that is thin in y or z fills its bricks in part: by their count, except
// where the level is narrow in x, which leaves the one-sweep tiles of 64 pairs
// emptier still.  FP64 V-cycle, bricks against one-sweep launches on level 1: 625
// bricks 330 and 336 us, 729 (65^3, odd) 447 and 523, 784 (220 x 220 x 5) 519 and
// 482, 1444 (300 x 300 x 3) 670 and 481; 3 x 300 x 300 903 and 2036.  The mixed
// form's solves cross at 700.
constexpr long long BRICK_MAX = 750;
constexpr int BRICK_NARROW = 16;

// Whether level 0 may smooth with the fused passes: the two-step V-cycle of a
// hierarchy with coarse levels (every dimension even), and enough cells.  At
// 128^3 with a membrane the two forms are equal (447 and 449 us per FP64
// V-cycle); below, a pass leaves part of the chip idle.
constexpr long long WALK_MIN_CELLS = 1 << 21;
// Largest share of the units in the near list: where the pass (a of the one-sweep
// launches' time when both fill their tiles, over the share of its own tiles that
// is filled) and the listed units (b times their share of it) take as long as
// the launches (over the share of theirs).  FP64 a = 0.64, b = 1.2; mixed 0.8 and
// 1.1: the FP32 pass moves half the bytes in nearly the same time.  Iterations
// of whole solves by listed share, the pass over one-sweep launches: 256^3 FP64
// 0.87 (0.17), 0.97 (0.28), 1.07 (0.50), mixed 0.99 (0.13), 1.03 (0.21), 1.10
// (0.28); 208^3 FP64 0.97 (0.23), 1.04 (0.35), mixed 0.85 (0.03), 1.04 (0.23); 160^3,
// which fills 0.63 of the launches' tiles, FP64 0.87 (0.45), mixed 0.95 (0.51); 128^3
// FP64 0.96 (0.22), 1.02 (0.50), mixed 0.98 (0.06), 1.05 (0.21).
double walk_max_near(int H, int ny, bool mixed)
{
    auto fill = [&](int h, int j) { return (double)H * ny / ((double)cdiv(H, h) * h * cdiv(ny, j) * j); };
    const double a = mixed ? 0.8 : 0.64, b = mixed ? 1.1 : 1.2;
    return std::max(0.05, (1.0 / fill(64, 4) - a / fill(WK_OH, WK_OJ)) / b);  // (64 x 4: make_geo's tiles)
}
// From here on the near sequence runs beside the pass on a stream of its own;
// the fork and join cost 10 us.  160^3 mixed: one after the other 22.3 ms per
// step, beside 25.9; 256^3 FP64 42.0 and 40.5 ms per solve, 512^3 mixed 288 and 264.
constexpr long long BESIDE_MIN_CELLS = 1 << 23;
// Up to this many rows the near units take the half-sweeps of rows.hpp (one
// or two launches each instead of four); beyond, their recomputed cells cost
// more than the launches.  FP64 V-cycle at 128^3 with a membrane: 440 us
// without, 406 us with; 256^3 with 63 thousand rows: 41.2 and 42.2 ms per
// solve; 512^3 with 150 thousand: 11.1 and 11.4 ms per iteration.
constexpr long long FEW_ROWS = 1 << 15;
// The same on all of level 0 below WALK_MIN_CELLS: up to this many rows, or with
// closed ghosts and membranes together (five launches otherwise).  Per
// iteration, rows.hpp against the one-sweep kernels, FP64 and mixed: 10 thousand
// rows at 64^3 0.97 and 0.97, 28 at 80^3 0.96 and 1.01, 35 at 96^3 0.99 and
// 1.00, 44 at 112^3 0.99 and 1.01, 52 there 1.00 and 1.03, 59 at 124^3 1.03 and
// 1.10; membranes alone: 29 at 96^3 0.98 and 0.93, 61 at 124^3 1.02 and 1.02;
// both kinds, 79 at 124^3, 0.94 and 0.99.
constexpr long long FLAT_ROWS = 45000;

inline int sparse_blocks(long long n) { return (int)std::max<long long>(1, std::min<long long>(XB, (n + TPB - 1) / TPB)); }

struct Level {
    int n[3] = {0, 0, 0};
    int H = 0;
    long long N = 0, Nh = 0;
    size_t cp[3], cm[3], w[3];       // places of the coefficients in the context's image
    DBuf<uint8_t> m;                 // split layout: coarse mask (CM_* bits); level 0 flags
    size_t pi[3] = {0, 0, 0}, pt[3] = {0, 0, 0};  // prolongation map from the coarse parent
    double volA = 0.0;               // volume of the active cells
    long long n_inactive = 0;        // coarse levels: inactive cells (inside bodies)
    Geo geo;                         // tiles over (h, j, k) of one colour
    Geo geo2;                        // level 0: 64 x 8 tiles of the FP64 half-sweep (two rows per thread)
    Geo geon;                        // tiles over (i, j, k): restriction into this level
    Walk walk;                       // over 2 Nh slots
    DBuf<double> x64, b64;
    DBuf<float> x32;
    DBuf<bf16> b16;
    bool brick = false;              // smoothing phases on bricks (one launch each)
    Brick br;
    DBuf<double> k64;                // brick levels: black iterate between the phases
    DBuf<float> k32;
    Lv lv;
    PMap pm{};
    std::vector<double> hc[3], hw[3];
};

void level_geometry(Level &L, const std::vector<double> *f, Image &I)
{
    for (int d = 0; d < 3; ++d) {
        int n = L.n[d];
        L.hc[d].resize(n);
        L.hw[d].resize(n);
        std::vector<double> cp(n), cm(n);
        for (int i = 0; i < n; ++i) {
            L.hc[d][i] = 0.5 * (f[d][i] + f[d][i + 1]);
            L.hw[d][i] = f[d][i + 1] - f[d][i];
        }
        for (int i = 0; i < n; ++i) {
            cp[i] = (i + 1 < n) ? 1.0 / (L.hw[d][i] * (L.hc[d][i + 1] - L.hc[d][i])) : 0.0;
            cm[i] = (i > 0) ? 1.0 / (L.hw[d][i] * (L.hc[d][i] - L.hc[d][i - 1])) : 0.0;
        }
        L.cp[d] = I.put(cp);
        L.cm[d] = I.put(cm);
        L.w[d] = I.put(L.hw[d]);
    }
    L.N = (long long)L.n[0] * L.n[1] * L.n[2];
    L.H = (L.n[0] + 1) / 2;
    L.Nh = (long long)L.H * L.n[1] * L.n[2];
    // levels below 2^26 cells take half the blocks (twice the planes per
    // thread): their per-thread set-up is then spread over more planes
    const int maxb = L.N < (1LL << 26) ? 4096 : 8192;
    L.geo = make_geo(L.H, L.n[1], L.n[2], maxb);
    L.geon = make_geo_nat(L.n[0], L.n[1], L.n[2], maxb);
    L.walk = make_walk(2 * L.Nh);
}

// LDS layout of one tail level (mask, iterate with its pads, RHS), 16-byte
// aligned pieces; in the RHS's place of the first level stand the residual
// sums (one double per pair of cells)
inline void tail_layout(const Level &L, size_t tsz, bool first, int &off, int &moff, int &xoff, int &boff)
{
    auto al = [](long long v) { return (int)((v + 15) / 16 * 16); };
    moff = off;
    off = al(off + 2 * L.Nh);
    xoff = off;
    off = al(off + 2LL * tail_stride(L.H, L.n[1], L.n[2]) * (long long)tsz);
    boff = off;
    off = al(off + (first ? std::max<long long>(2 * L.Nh * (long long)tsz, 8 * L.Nh) : 2 * L.Nh * (long long)tsz));
}

// slot of natural cell (i,j,k) in a level with half-width H
inline long long host_slot(int H, int ny, long long Nh, int i, int j, int k)
{
    return (long long)((i + j + k) & 1) * Nh + (i >> 1) + (long long)H * (j + (long long)ny * k);
}

}  // namespace
}  // namespace ibm

using namespace ibm;

namespace ibm {
namespace {
// Pinned host slots for the per-context scalar read-back, cut from chunks
// that live until the process ends: freeing pinned memory synchronises the
// device, which a graph capture running in another thread does not allow.
std::mutex g_pin_mu;
std::vector<double *> g_pin_free;
double *pinned_slot()
{
    std::lock_guard<std::mutex> lk(g_pin_mu);
    if (g_pin_free.empty()) {
        constexpr int per = 64;
        double *chunk = nullptr;
        std::shared_lock<std::shared_mutex> cl(capture_mutex());
        IBM_HIP(hipHostMalloc((void **)&chunk, per * S_COUNT * sizeof(double), hipHostMallocDefault));
        for (int q = per - 1; q >= 0; --q) g_pin_free.push_back(chunk + q * S_COUNT);
    }
    double *p = g_pin_free.back();
    g_pin_free.pop_back();
    return p;
}
void pinned_release(double *p)
{
    std::lock_guard<std::mutex> lk(g_pin_mu);
    g_pin_free.push_back(p);
}
}  // namespace
}  // namespace ibm

// what a set-up sums and counts on the device
struct SetupSums {
    double volume[16], inactive[16];  // fluid volume (level 0), active volumes; inactive cells
    int units[2], adjacent, err;
};

struct poisson_ctx {
    poisson_opts opts;
    HostGrid g;
    long long N = 0, nm = 0, ng = 0, nrows = 0, n_fallback = 0, pin = 0;
    long long N2 = 0, Nt = 0;  // 2 Nh cell slots, + membrane unknowns
    double vol_fluid = 0.0, vol_pin = 0.0;
    int tail0 = 1;             // first level of the single-workgroup tail (FP32 levels in the mixed form)
    int tail0d = 1;            // the same for FP64 levels
    std::vector<double> srj_w; // SRJ relaxation factors in application order
    DBuf<int32_t> rslot, rcol, mslot, mcol, mcolor;
    DBuf<int32_t> rmrow;  // membrane cell behind each ghost-row column
    DBuf<double> rw, rsG, rdlb;
    std::vector<Level> lv;
    Sp sp;
    Walk W0;   // over Nt unknowns
    Walk W4;   // over ceil(Nt / 4) groups of 4 unknowns
    Walk Wc;   // over 2 Nh cell slots
    Walk Wp;   // over Nh pairs of cells, then the membrane unknowns
    DBuf<double> x, r, rh, p, v, ph, sh, t, rsp, b;
    DBuf<float> fr, frh, fp, fv, fph, fsh, ft, frsp;
    // mixed: the inner solution accumulates in FP64 (a smooth correction
    // rounded to FP32 loses its small Laplacian: the operator multiplies the
    // rounding by up to |A| ~ 12/h^2)
    DBuf<double> d64;
    DBuf<double> r2;           // mixed: right-hand side of the FP64 fallback solve
    DBuf<double> gtmp, mtmp, sc, part;  // ghost and membrane staging; scalars; partials
    DBuf<SetupSums> ssum;       // set-up sums, read back once
    DBuf<uint8_t> hact[2];      // set-up: natural-order coarse active/cut bits of two consecutive levels
    // fused level-0 smoothing (walk.hpp) and the units around irregular cells
    bool walk = false, beside = false;
    DBuf<char> coef;            // coefficients and prolongation maps of all levels
    // level-0 half-sweeps with the sparse rows in the same launch (rows.hpp):
    // on all of level 0 (flat), or on the near units of the fused passes (few)
    bool flat = false, few = false;
    Rows rows{};
    DBuf<int32_t> code, rix, mcode, aslot, acode;
    DBuf<double> gtmp2;
    WalkGeo wg{};
    DBuf<int32_t> units, nunits;
    DBuf<uint8_t> ubits[2];
    Near near{}, nearres{};     // the sequence's units; the units whose results replace the pass's
    hipStream_t ns = nullptr;   // the near cells' launches, beside the pass over the rest
    hipEvent_t ef = nullptr, en = nullptr;
    double *hsc = nullptr;
    hipStream_t cs = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr, ej = nullptr;
    hipGraphExec_t g64 = nullptr, g32 = nullptr;
    hipGraphExec_t g64w = nullptr;  // FP64 iteration on the correction (solves from a guess)
    size_t bytes = 0;
    bool mixed = false;
    // per-launch timing of one kernel (HIP events on the solve stream)
    int prof_kernel = -1;
    bool capturing = false;
    std::vector<hipEvent_t> prof_ev;
    int prof_used = 0;
    double prof_ms = 0.0;
    long long prof_count = 0;

    const Lv &L0() const { return lv[0].lv; }

    // (making and destroying an executable graph allocates and frees: like
    // every such call, not while another thread captures)
    void drop_graphs()
    {
        for (hipGraphExec_t *g : {&g64, &g32, &g64w}) {
            if (!*g) continue;
            std::shared_lock<std::shared_mutex> cl(capture_mutex());
            (void)hipGraphExecDestroy(*g);
            *g = nullptr;
        }
    }
    ~poisson_ctx()
    {
        drop_graphs();
        if (hsc) pinned_release(hsc);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        if (ej) (void)hipEventDestroy(ej);
        if (ef) (void)hipEventDestroy(ef);
        if (en) (void)hipEventDestroy(en);
        if (ns) (void)hipStreamDestroy(ns);
        if (cs) (void)hipStreamDestroy(cs);
        for (auto e : prof_ev) (void)hipEventDestroy(e);
    }
};

namespace ibm {
namespace {

// IBM_LOG=1 logs each solve's refinement steps to stderr, IBM_LOG=2 every iteration
int log_level()
{
    static const int lvl = [] {
        const char *e = getenv("IBM_LOG");
        return (e && *e) ? atoi(e) : 0;
    }();
    return lvl;
}
inline bool log_enabled() { return log_level() > 0; }

// kernel ids of the timing hook
enum { PK_SWEEP0 = 0, PK_APPLY0 = 1, PK_XR = 2, PK_WALK_UP = 3 };

inline void prof_begin(poisson_ctx &c, int kid, hipStream_t s)
{
    if (c.prof_kernel != kid || c.capturing) return;
    if ((int)c.prof_ev.size() < 2 * (c.prof_used + 1)) {
        hipEvent_t a, b;
        IBM_HIP(hipEventCreate(&a));
        IBM_HIP(hipEventCreate(&b));
        c.prof_ev.push_back(a);
        c.prof_ev.push_back(b);
    }
    IBM_HIP(hipEventRecord(c.prof_ev[2 * c.prof_used], s));
}

inline void prof_end(poisson_ctx &c, int kid, hipStream_t s)
{
    if (c.prof_kernel != kid || c.capturing) return;
    IBM_HIP(hipEventRecord(c.prof_ev[2 * c.prof_used + 1], s));
    ++c.prof_used;
}

inline void prof_harvest(poisson_ctx &c)
{
    for (int i = 0; i < c.prof_used; ++i) {
        float ms = 0.f;
        IBM_HIP(hipEventElapsedTime(&ms, c.prof_ev[2 * i], c.prof_ev[2 * i + 1]));
        c.prof_ms += ms;
        ++c.prof_count;
    }
    c.prof_used = 0;
}

inline void fin(poisson_ctx &c, int n, int op, int dst, double aux, hipStream_t s)
{
    k_fin<<<1, 1024, 0, s>>>(c.part.p, PSTRIDE, n, op, dst, aux, c.sc.p);
    IBM_LAUNCH_CHECK();
}

// partial sums of level l's RHS mean: alternate levels use alternate places,
// since a brick launch reads its level's while writing the next one's
inline double *mean_part(poisson_ctx &c, int l) { return c.part.p + (size_t)PSTRIDE * (2 + (l & 1)); }

// y = A x (or y = b - A x) on level 0, with dots; returns the partial count
template <class T>
int launch_apply(poisson_ctx &c, int mode, bool res, int nd, const T *x, T *y, const T *b, const double *sink,
                 const T *u1, const T *u2, hipStream_t s)
{
    const Level &L = c.lv[0];
    double *P = c.part.p;
    const int nsp = (int)(c.nrows + c.nm);
    const int sb = sparse_blocks(nsp);
    const int gb = L.geo.nb;
#define AP(MODE, RES, ND)                                                                                        \
    k0_apply2<T, MODE, RES, ND><<<gb, TPB, 0, s>>>(L.lv, L.geo, c.pin, x, y, b, sink, u1, u2, P, PSTRIDE);     \
    if (nsp) k0_sparse<T, RES, ND><<<sb, TPB, 0, s>>>(L.lv, c.sp, x, y, b, u1, u2, P, PSTRIDE, gb);
    if (res) {
        if (mode == M_PINNED && nd == 2) { AP(M_PINNED, true, 2) }
        else if (mode == M_UNPINNED && nd == 0) { AP(M_UNPINNED, true, 0) }
        else throw Error(IBM_EINVAL, "apply variant");
    } else {
        if (mode == M_PINZERO && nd == 1) { AP(M_PINZERO, false, 1) }
        else if (mode == M_PINZERO && nd == 2) { AP(M_PINZERO, false, 2) }
        else if (mode == M_PINNED && nd == 0) { AP(M_PINNED, false, 0) }
        else throw Error(IBM_EINVAL, "apply variant");
    }
#undef AP
    IBM_LAUNCH_CHECK();
    return gb + (nsp ? sb : 0);
}

template <class T>
struct Store;
template <>
struct Store<double> {
    typedef double Tc;
    typedef double TB;
    static Tc *x(Level &L) { return L.x64.p; }
    static Tc *k(Level &L) { return L.k64.p; }
    static TB *b(Level &L) { return L.b64.p; }
};
template <>
struct Store<float> {
    typedef float Tc;
    typedef bf16 TB;
    static Tc *x(Level &L) { return L.x32.p; }
    static Tc *k(Level &L) { return L.k32.p; }
    static TB *b(Level &L) { return L.b16.p; }
};

// prolongation of coarse level C onto F; the renormalised form only where C
// has inactive cells
template <bool FINE, class Tc, class Tf>
void launch_prolong(const Level &F, const Level &C, bool skip_red, const Tc *xc, Tf *xf, hipStream_t s)
{
    const bool rn = C.n_inactive > 0;
    if (skip_red && rn)
        k_prolong_z<FINE, Tc, Tf, true, true><<<C.geon.nb, TPB, 0, s>>>(F.lv, C.lv, F.pm, C.geon, xc, xf);
    else if (skip_red)
        k_prolong_z<FINE, Tc, Tf, true, false><<<C.geon.nb, TPB, 0, s>>>(F.lv, C.lv, F.pm, C.geon, xc, xf);
    else if (rn)
        k_prolong_z<FINE, Tc, Tf, false, true><<<C.geon.nb, TPB, 0, s>>>(F.lv, C.lv, F.pm, C.geon, xc, xf);
    else
        k_prolong_z<FINE, Tc, Tf, false, false><<<C.geon.nb, TPB, 0, s>>>(F.lv, C.lv, F.pm, C.geon, xc, xf);
}

// after a half-sweep of colour `color`: the membrane-adjacent cells of that
// colour, then a Jacobi update of every ghost unknown
template <class T>
void irregular_rows(poisson_ctx &c, T *x, const T *b, int color, hipStream_t s)
{
    const int mb = sparse_blocks(c.nm), gb = sparse_blocks(c.nrows + c.nm);
    if (c.nm) k0_msweep<T><<<mb, TPB, 0, s>>>(c.lv[0].lv, c.sp, x, b, color, c.mtmp.p);
    if (c.nrows) {
        k0_mscat_gjac<T><<<gb, TPB, 0, s>>>(c.sp, x, b, color, c.mtmp.p, c.gtmp.p);
        k0_gscat<T><<<gb, TPB, 0, s>>>(c.sp, x, c.gtmp.p);
    }
}

// level-0 smoothing step: for red then black, the dense half-sweep, the
// membrane-adjacent cells of that colour, then Jacobi on all ghost unknowns
template <class T>
void fine_smooth(poisson_ctx &c, T *x, const T *b, const double *sink, bool from_zero, hipStream_t s)
{
    const Level &L = c.lv[0];
    for (int color = 0; color < 2; ++color) {
        if (from_zero && color == 0) {
            // the other colour is zeroed too: ghost rows and membrane rows read it before its sweep
            const long long pin_s = (sink && c.pin < L.Nh) ? c.pin : -1;
            k0_sweep_zero<T><<<L.geo.nb, TPB, 0, s>>>(L.lv, L.geo, pin_s, x, x + L.Nh, b, L.lv.f, sink, 0);
            if (c.nm) {
                Walk Wt = make_walk(c.nm);
                k_fill<T><<<Wt.nb, TPB, 0, s>>>(Wt, x + c.N2, 0.0);
            }
        } else {
            // (from zero, the black slots were zeroed by the red sweep; ghost
            // values set since then must survive, so this is an ordinary sweep)
            const long long co = (long long)color * L.Nh;
            const long long pin_s = (sink && c.pin >= co && c.pin < co + L.Nh) ? c.pin - co : -1;
            if (!from_zero) prof_begin(c, PK_SWEEP0, s);
            const Geo &G = std::is_same<T, double>::value ? L.geo2 : L.geo;  // FP64: two rows per thread
            k0_sweep<T><<<G.nb, TPB, 0, s>>>(L.lv, G, pin_s, x + co, x + (L.Nh - co), b + co, L.lv.f + co, sink,
                                             color);
            if (!from_zero) prof_end(c, PK_SWEEP0, s);
        }
        irregular_rows<T>(c, x, b, color, s);
    }
    IBM_LAUNCH_CHECK();
}

template <class Tc, class TB>
void coarse_smooth(Level &L, int steps, bool from_zero, const double *mean, hipStream_t s)
{
    Tc *x = Store<Tc>::x(L);
    const TB *b = Store<Tc>::b(L);
    for (int it = 0; it < steps; ++it) {
        if (it == 0 && from_zero) {
            k_csweep<Tc, TB, 1><<<L.geo.nb, TPB, 0, s>>>(L.lv, L.geo, x, b, mean, 0);
            k_csweep<Tc, TB, 2><<<L.geo.nb, TPB, 0, s>>>(L.lv, L.geo, x, b, mean, 1);
        } else {
            k_csweep<Tc, TB, 0><<<L.geo.nb, TPB, 0, s>>>(L.lv, L.geo, x, b, mean, 0);
            k_csweep<Tc, TB, 0><<<L.geo.nb, TPB, 0, s>>>(L.lv, L.geo, x, b, mean, 1);
        }
    }
    IBM_LAUNCH_CHECK();
}

template <class Tc, class TB>
BrickArgs<Tc, TB> brick_args(poisson_ctx &c, int l, int steps)
{
    Level &L = c.lv[l];
    BrickArgs<Tc, TB> a{};
    a.b = Store<Tc>::b(L);
    a.vol = L.volA;
    a.mean = c.sc.p + S_MEAN0 + l;
    a.steps = steps;
    return a;
}

// first phase of brick level l: nu1 steps from zero (the level's mean from
// the partial sums of the launch before) and the restriction into level l+1;
// returns the count of partial sums of that level's mean
template <class Tc, class TB>
int brick_down(poisson_ctx &c, int l, int npart, hipStream_t s)
{
    Level &L = c.lv[l], &C = c.lv[l + 1];
    auto a = brick_args<Tc, TB>(c, l, c.opts.nu1);
    a.part = mean_part(c, l);
    a.npart = npart;
    a.xb = Store<Tc>::k(L);
    a.bc = Store<Tc>::b(C);
    a.pout = mean_part(c, l + 1);
    k_brick<Tc, TB, BR_ZERO><<<L.br.nb, BR_T, 0, s>>>(L.lv, L.br, C.lv, L.pm, a);
    IBM_LAUNCH_CHECK();
    return L.br.nb;
}

// second phase: prolongation from level l+1 and nu2 steps
template <class Tc, class TB>
void brick_up(poisson_ctx &c, int l, hipStream_t s)
{
    Level &L = c.lv[l], &C = c.lv[l + 1];
    auto a = brick_args<Tc, TB>(c, l, c.opts.nu2);
    a.xin = Store<Tc>::k(L);
    a.xr = Store<Tc>::x(L);
    a.xb = a.xr + L.Nh;
    a.xc = Store<Tc>::x(C);
    a.renorm = C.n_inactive > 0;
    k_brick<Tc, TB, BR_PROLONG><<<L.br.nb, BR_T, 0, s>>>(L.lv, L.br, C.lv, L.pm, a);
    IBM_LAUNCH_CHECK();
}

// coarsest level on bricks: all its sweeps, two per launch, the black iterate
// alternating between two buffers so that the last launch writes the level's own
template <class Tc, class TB>
void brick_coarsest(poisson_ctx &c, int l, int npart, hipStream_t s)
{
    Level &L = c.lv[l];
    Tc *x = Store<Tc>::x(L), *buf[2] = {x + L.Nh, Store<Tc>::k(L)};
    const int n = (c.opts.coarse_sweeps + 1) / 2;
    for (int q = 0; q < n; ++q) {
        const int left = n - 1 - q;
        auto a = brick_args<Tc, TB>(c, l, q == n - 1 ? c.opts.coarse_sweeps - 2 * q : 2);
        a.xb = buf[left & 1];
        a.xr = left ? nullptr : x;
        if (q == 0) {
            a.part = mean_part(c, l);
            a.npart = npart;
            k_brick<Tc, TB, BR_ZERO><<<L.br.nb, BR_T, 0, s>>>(L.lv, L.br, L.lv, L.pm, a);
        } else {
            a.xin = buf[(left + 1) & 1];
            k_brick<Tc, TB, BR_PLAIN><<<L.br.nb, BR_T, 0, s>>>(L.lv, L.br, L.lv, L.pm, a);
        }
    }
    IBM_LAUNCH_CHECK();
}

// n half-sweeps (red first) with the sparse rows, over every cell of level 0
// or (UNITS) the near units; zero: from a zero iterate.  Ghost values start
// at their unknowns in x and then alternate between two arrays: the array that
// holds them at the end is returned (null without ghost rows).
template <class T, bool UNITS>
T *half_sweeps(poisson_ctx &c, T *x, const T *b, const double *sink, int n, bool zero, hipStream_t s)
{
    const Level &L = c.lv[0];
    const Rows &R = c.rows;
    T *G[2] = {(T *)c.gtmp.p, (T *)c.gtmp2.p}, *g = nullptr;
    HalfBlocks B;
    B.cells = UNITS ? c.near.nb() : (int)((L.Nh + 8 * TPB - 1) / (8 * TPB) * 8);
    for (int q = 0; q < n; ++q) {
        const int color = q & 1;
        const RowsIn<T> I{x, g, b, sink, zero && q == 0};
        T *gn = g == G[0] ? G[1] : G[0];
        B.adj = I.zero ? 0 : (int)cdiv(R.na, TPB);
        B.rows = (int)cdiv(8LL * (R.nm ? R.nm : R.nrows), TPB);
        if (!UNITS && !I.zero) prof_begin(c, PK_SWEEP0, s);
        if (R.nm) {
            k_half<T, UNITS, false><<<B.total(), TPB, 0, s>>>(L.lv, R, c.near, B, I, x, color, gn, c.mtmp.p);
            k_half_ghosts<T><<<cdiv(R.nrows + R.nm, TPB), TPB, 0, s>>>(L.lv, R, I, x, color, c.mtmp.p, gn);
        } else {
            k_half<T, UNITS, true><<<B.total(), TPB, 0, s>>>(L.lv, R, c.near, B, I, x, color, gn, nullptr);
        }
        if (!UNITS && !I.zero) prof_end(c, PK_SWEEP0, s);
        if (R.nrows) g = gn;
    }
    IBM_LAUNCH_CHECK();
    return g;
}

// ghost values to their unknowns in x; rs: also the sparse cells' residuals
template <class T>
void rows_out(poisson_ctx &c, T *x, const T *b, const T *g, T *rs, hipStream_t s)
{
    const Rows &R = c.rows;
    if (!R.nrows || !g) return;
    const RowsIn<T> I{x, g, b, nullptr, false};
    if (rs) k_rows_out<T, true><<<cdiv(R.nrows + R.nm, TPB), TPB, 0, s>>>(c.lv[0].lv, R, I, x, rs);
    else k_rows_out<T, false><<<cdiv(R.nrows, TPB), TPB, 0, s>>>(c.lv[0].lv, R, I, x, rs);
    IBM_LAUNCH_CHECK();
}

// the near cells' launches run on c.ns between fork() and join()
void fork(poisson_ctx &c, hipStream_t s)
{
    IBM_HIP(hipEventRecord(c.ef, s));
    IBM_HIP(hipStreamWaitEvent(c.ns, c.ef, 0));
}
void join(poisson_ctx &c, hipStream_t s)
{
    IBM_HIP(hipEventRecord(c.en, c.ns));
    IBM_HIP(hipStreamWaitEvent(s, c.en, 0));
}

// level 0, first phase (two steps from zero, residual, restriction) with the
// fused pass; w: scratch vector of the near cells, xk: black iterate between
// the phases, rs: scratch for the irregular cells' residuals.  Returns the
// count of partial sums of level 1's mean.
template <class T>
int walk_down(poisson_ctx &c, const T *b, T *w, T *xk, T *rs, const double *sink, hipStream_t s)
{
    typedef typename Store<T>::TB TB;
    Level &L = c.lv[0], &C = c.lv[1];
    double *part = mean_part(c, 1);
    TB *bc = Store<T>::b(C);
    const int nu = c.near.nb();
    if (nu) {
        hipStream_t n = c.beside ? c.ns : s;
        if (c.beside) fork(c, s);
        if (c.few) {
            rows_out<T>(c, w, b, half_sweeps<T, true>(c, w, b, sink, 4, true, n), rs, n);
        } else {
            k_near_zero<T><<<nu + (int)cdiv(c.nm, NU_T), NU_T, 0, n>>>(L.lv, c.near, nu, c.nm, c.pin, sink, b, w);
            irregular_rows<T>(c, w, b, 0, n);
            for (int q = 0; q < 3; ++q) {
                const int color = q == 1 ? 0 : 1;
                k_near_sweep<T><<<nu, NU_T, 0, n>>>(L.lv, c.near, c.pin, sink, b, w, color);
                irregular_rows<T>(c, w, b, color, n);
            }
            const int nsp = (int)(c.nrows + c.nm);
            if (nsp) k0_sparse_res<T><<<sparse_blocks(nsp), TPB, 0, n>>>(L.lv, c.sp, w, b, rs);
        }
        k_near_restrict<T, TB><<<nu, NU_T, 0, n>>>(L.lv, C.lv, c.near, c.pin, sink, b, w, rs, bc, part + c.wg.nb);
    }
    k_walk_down<T, TB><<<c.wg.nb, WK_T, 0, s>>>(L.lv, C.lv, c.wg, c.near, c.pin, sink, b, xk, bc, part);
    IBM_LAUNCH_CHECK();
    if (nu && c.beside) join(c, s);
    return c.wg.nb + nu;
}

// second phase: prolongation and two steps; x receives every unknown
template <class T>
void walk_up(poisson_ctx &c, const T *b, T *x, T *w, T *xk, const double *sink, hipStream_t s)
{
    Level &L = c.lv[0], &C = c.lv[1];
    const T *xc = (const T *)Store<T>::x(C);
    const int nu = c.near.nb();
    if (nu) {
        hipStream_t n = c.beside ? c.ns : s;
        k_near_merge<T><<<nu, NU_T, 0, s>>>(L.lv, c.near, w, xk);
        if (c.beside) fork(c, s);
        k_near_prolong<T><<<nu, NU_T, 0, n>>>(L.lv, C.lv, L.pm, c.near, xc, w);
        if (c.few) {
            rows_out<T>(c, w, b, half_sweeps<T, true>(c, w, b, sink, 4, false, n), (T *)nullptr, n);
        } else {
            for (int q = 0; q < 4; ++q) {
                k_near_sweep<T><<<nu, NU_T, 0, n>>>(L.lv, c.near, c.pin, sink, b, w, q & 1);
                irregular_rows<T>(c, w, b, q & 1, n);
            }
        }
    }
    prof_begin(c, PK_WALK_UP, s);
    k_walk_up<T><<<c.wg.nb, WK_T, 0, s>>>(L.lv, C.lv, L.pm, c.wg, c.pin, sink, b, xk, xc, x);
    prof_end(c, PK_WALK_UP, s);
    if (nu) {
        if (c.beside) join(c, s);
        const int nr = c.nearres.nb();
        k_near_final<T><<<nr + (int)cdiv(c.nm, NU_T), NU_T, 0, s>>>(L.lv, c.nearres, nr, c.nm, w, x);
    }
    IBM_LAUNCH_CHECK();
}

// x = V-cycle(b) on the unpinned operator with the sink at the pin; x
// unshifted; w: a scratch vector over the unknowns (neither b nor x)
template <class T>
void vcycle(poisson_ctx &c, const T *b, T *x, T *w, const double *sink, hipStream_t s)
{
    typedef typename Store<T>::Tc Tc;
    typedef typename Store<T>::TB TB;
    const int nl = (int)c.lv.size();
    const poisson_opts &o = c.opts;
    const bool walk = c.walk && c.prof_kernel != PK_SWEEP0;  // timing the half-sweeps needs their launches
    T *r0 = std::is_same<T, double>::value ? (T *)c.rsp.p : (T *)c.frsp.p;
    if (c.flat)
        rows_out<T>(c, x, b, half_sweeps<T, false>(c, x, b, sink, 2 * o.nu1, true, s), nl > 1 ? r0 : (T *)nullptr, s);
    else if (!walk)
        for (int it = 0; it < o.nu1; ++it) fine_smooth<T>(c, x, b, sink, it == 0, s);
    if (nl > 1) {
        Level &L1 = c.lv[1];
        int npart;  // partial sums of the next level's mean
        if (walk) {
            npart = walk_down<T>(c, b, w, r0, x, sink, s);  // x is free until the second phase
        } else {
            // level-0 residual: the sparse rows into r0, then the regular rows
            // computed and restricted in one pass
            const int nsp = (int)(c.nrows + c.nm);
            if (nsp && !c.flat) k0_sparse_res<T><<<sparse_blocks(nsp), TPB, 0, s>>>(c.lv[0].lv, c.sp, x, b, r0);
            k0_restrict_res<T, TB><<<L1.geon.nb, TPB, 0, s>>>(c.lv[0].lv, L1.lv, L1.geon, c.pin, x, b, sink, r0,
                                                             Store<T>::b(L1), mean_part(c, 1));
            IBM_LAUNCH_CHECK();
            npart = L1.geon.nb;
        }
        const int lt = std::is_same<T, double>::value ? c.tail0d : c.tail0;
        for (int l = 1; l < lt; ++l) {
            Level &L = c.lv[l];
            if (L.brick) {
                if (l == nl - 1) brick_coarsest<Tc, TB>(c, l, npart, s);
                else npart = brick_down<Tc, TB>(c, l, npart, s);
                continue;
            }
            const double *mean = c.sc.p + S_MEAN0 + l;
            k_fin<<<1, 1024, 0, s>>>(mean_part(c, l), PSTRIDE, npart, FIN_MEAN, S_MEAN0 + l, L.volA, c.sc.p);
            if (l == nl - 1) {
                coarse_smooth<Tc, TB>(L, o.coarse_sweeps, true, mean, s);
                break;
            }
            coarse_smooth<Tc, TB>(L, o.nu1, true, mean, s);
            Level &C = c.lv[l + 1];
            k_restrict<Tc, TB, TB><<<C.geon.nb, TPB, 0, s>>>(L.lv, C.lv, C.geon, Store<T>::x(L), Store<T>::b(L), mean,
                                                            Store<T>::b(C), mean_part(c, l + 1));
            IBM_LAUNCH_CHECK();
            npart = C.geon.nb;
        }
        if (lt < nl) {
            Tail tl;
            tl.n = nl - lt;
            tl.nu1 = o.nu1;
            tl.nu2 = o.nu2;
            tl.ncs = o.coarse_sweeps;
            int off = 0;
            for (int q = 0; q < tl.n; ++q) {
                Level &L = c.lv[lt + q];
                tl.t[q].L = L.lv;
                tl.t[q].M = L.pm;
                tl.t[q].volA = L.volA;
                tl.t[q].xg = Store<T>::x(L);
                tl.t[q].bg = Store<T>::b(L);
                tail_layout(L, sizeof(Tc), q == 0, off, tl.t[q].moff, tl.t[q].xoff, tl.t[q].boff);
            }
            tl.coff = off;
            for (int q = 0; q < tl.n; ++q) {
                const Level &L = c.lv[lt + q];
                off += tail_coef_bytes(L.n[0], L.n[1], L.n[2]);
            }
            k_tail<Tc, TB><<<1, TAIL_T, off, s>>>(tl, mean_part(c, lt), npart);
            IBM_LAUNCH_CHECK();
        }
        for (int l = std::min(lt, nl - 1) - 1; l >= 1; --l) {
            Level &L = c.lv[l];
            Level &C = c.lv[l + 1];
            if (L.brick) {
                brick_up<Tc, TB>(c, l, s);
                continue;
            }
            launch_prolong<false>(L, C, o.nu2 > 0, Store<T>::x(C), Store<T>::x(L), s);
            coarse_smooth<Tc, TB>(L, o.nu2, false, c.sc.p + S_MEAN0 + l, s);
        }
        if (walk) {
            walk_up<T>(c, b, x, w, r0, sink, s);
            return;
        }
        Level &L0v = c.lv[0];
        launch_prolong<true>(L0v, L1, o.nu2 > 0, Store<T>::x(L1), x, s);
        IBM_LAUNCH_CHECK();
    }
    if (c.flat) rows_out<T>(c, x, b, half_sweeps<T, false>(c, x, b, sink, 2 * o.nu2, false, s), (T *)nullptr, s);
    else
        for (int it = 0; it < o.nu2; ++it) fine_smooth<T>(c, x, b, sink, false, s);
}

// SRJ schedule: the reciprocals of the roots of the degree-m Chebyshev
// polynomial on [kmin, 2], kmin = 16/m^2 (the minimax factors for the
// amplification prod (1 - w k) over the spectrum of D^-1 A), in the order
// smallest, largest, second smallest, ...
std::vector<double> srj_schedule(int m)
{
    const double kmin = 16.0 / ((double)m * m), pi = 3.14159265358979323846;
    std::vector<double> w(m), out;
    for (int j = 1; j <= m; ++j)
        w[j - 1] = 1.0 / (0.5 * (2.0 + kmin) - 0.5 * (2.0 - kmin) * std::cos(pi * (2 * j - 1) / (2.0 * m)));
    std::sort(w.begin(), w.end());
    for (int lo = 0, hi = m - 1; lo <= hi; ++lo, --hi) {
        out.push_back(w[lo]);
        if (hi != lo) out.push_back(w[hi]);
    }
    return out;
}

// x = SRJ(b): the scheduled sweeps from zero, alternating between x and the
// residual scratch (the starting buffer is chosen so the last sweep lands in x)
template <class T>
void srj_apply(poisson_ctx &c, const T *b, T *x, hipStream_t s)
{
    T *tmp = std::is_same<T, double>::value ? (T *)c.rsp.p : (T *)c.frsp.p;
    const Level &L = c.lv[0];
    const int m = (int)c.srj_w.size(), nsp = (int)(c.nrows + c.nm);
    T *xo = (m % 2) ? tmp : x, *xn = (m % 2) ? x : tmp;
    k_fill<T><<<c.W0.nb, TPB, 0, s>>>(c.W0, xo, 0.0);
    for (int q = 0; q < m; ++q) {
        k0_jacobi<T><<<L.geo.nb, TPB, 0, s>>>(L.lv, L.geo, c.pin, xo, xn, b, c.srj_w[q]);
        if (nsp) k0_jacobi_sparse<T><<<sparse_blocks(nsp), TPB, 0, s>>>(L.lv, c.sp, xo, xn, b, c.srj_w[q]);
        std::swap(xo, xn);
    }
    IBM_LAUNCH_CHECK();
}

// x = M^-1 b: the V-cycle (with the pin sink) or SRJ; the output is not yet
// shifted to a zero pin value (its consumers do that)
template <class T>
void precond(poisson_ctx &c, const T *b, T *x, T *w, const double *sink, hipStream_t s)
{
    if (c.opts.precond == IBM_PRECOND_SRJ) srj_apply<T>(c, b, x, s);
    else vcycle<T>(c, b, x, w, sink, s);
}

// One BiCGSTAB iteration (van der Vorst 1992, right preconditioning): all
// scalars stay on the device.
template <class T, class TX>
void bicg_iteration(poisson_ctx &c, TX *y, T *r, T *rh, T *p, T *v, T *ph, T *sh, T *t, hipStream_t s)
{
    const Walk &W = c.W4;
    const Lv &L = c.L0();
    k_p_update4<T><<<W.nb, TPB, 0, s>>>(L, W, c.Nt, r, p, v, c.sc.p, c.part.p);
    fin(c, W.nb, FIN_SINK, S_SINKP, 0.0, s);
    precond<T>(c, p, ph, t, c.sc.p + S_SINKP, s);  // t is free until the second operator apply
    prof_begin(c, PK_APPLY0, s);
    int np = launch_apply<T>(c, M_PINZERO, false, 1, ph, v, nullptr, nullptr, rh, nullptr, s);
    prof_end(c, PK_APPLY0, s);
    fin(c, np, FIN_ALPHA, 0, 0.0, s);
    k_s_update4<T><<<W.nb, TPB, 0, s>>>(L, W, c.Nt, r, v, c.sc.p, c.part.p);
    fin(c, W.nb, FIN_SINK, S_SINKS, 0.0, s);
    precond<T>(c, r, sh, t, c.sc.p + S_SINKS, s);
    np = launch_apply<T>(c, M_PINZERO, false, 2, sh, t, nullptr, nullptr, r, nullptr, s);
    fin(c, np, FIN_OMEGA, 0, 0.0, s);
    prof_begin(c, PK_XR, s);
    k_xr_update4<T, TX><<<W.nb, TPB, 0, s>>>(L, W, c.Nt, c.pin, y, ph, sh, r, t, rh, c.sc.p, c.part.p,
                                              PSTRIDE);
    prof_end(c, PK_XR, s);
    IBM_LAUNCH_CHECK();
    fin(c, W.nb, FIN_RHO, 0, 0.0, s);
}

void read_scalars(poisson_ctx &c, hipStream_t s)
{
    IBM_HIP(hipMemcpyAsync(c.hsc, c.sc.p, S_COUNT * sizeof(double), hipMemcpyDeviceToHost, s));
    IBM_HIP(hipStreamSynchronize(s));
    prof_harvest(c);
}

// Right-preconditioned BiCGSTAB on A y = rhs; y starts at zero.  rhs may be
// in a wider type than the vectors (the FP64 residual of a refinement step
// feeding an FP32 inner solve: it is rounded on the way in).  Returns the
// iteration count; *rc gets the status.
constexpr int INNER_STALL = 12;

template <class T, class TX, class TR>
int bicgstab(poisson_ctx &c, const TR *rhs, TX *y, T *r, T *rh, T *p, T *v, T *ph, T *sh, T *t, double tol, int maxit,
             bool true_check, hipGraphExec_t *graph, hipStream_t s, int *rc, double *relout)
{
    const Walk &W = c.W0;
    k_fill<TX><<<W.nb, TPB, 0, s>>>(W, y, 0.0);
    k_fill<T><<<W.nb, TPB, 0, s>>>(W, p, 0.0);
    k_fill<T><<<W.nb, TPB, 0, s>>>(W, v, 0.0);
    k_copy_norm4<TR, T><<<c.W4.nb, TPB, 0, s>>>(c.W4, c.Nt, rhs, r, rh, c.part.p);
    IBM_LAUNCH_CHECK();
    fin(c, c.W4.nb, FIN_INIT, 0, 0.0, s);
    read_scalars(c, s);
    *rc = IBM_ENOCONV;
    if (c.hsc[S_BN2] == 0.0) {
        *rc = IBM_OK;
        *relout = 0.0;
        return 0;
    }
    // Only an iteration on one stream becomes a graph: with the near sequence
    // beside the pass (from 2^23 cells) its launches are enqueued one by one.
    // They take 20 us and more each there, longer than the host needs for one.
    const bool forked = c.walk && c.beside && c.near.nb() > 0;
    const bool use_graph = c.opts.use_graph && c.prof_kernel < 0 && !forked;
    if (use_graph && !*graph) {
        std::unique_lock<std::shared_mutex> lk(capture_mutex());
        // a failure inside the capture still ends it, so the stream never
        // stays in capture mode (the user's stream joins it afterwards)
        struct Capture {
            poisson_ctx &c;
            hipStream_t s;
            hipGraph_t gr = nullptr;
            bool open = false;
            ~Capture()
            {
                if (open) {
                    hipGraph_t g2 = nullptr;
                    if (hipStreamEndCapture(s, &g2) == hipSuccess && g2) (void)hipGraphDestroy(g2);
                    (void)hipGetLastError();
                }
                if (gr) (void)hipGraphDestroy(gr);
                c.capturing = false;
            }
        } cap{c, s};
        c.capturing = true;
        IBM_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
        cap.open = true;
        bicg_iteration<T, TX>(c, y, r, rh, p, v, ph, sh, t, s);
        cap.open = false;
        IBM_HIP(hipStreamEndCapture(s, &cap.gr));
        IBM_HIP(hipGraphInstantiate(graph, cap.gr, nullptr, nullptr, 0));
    }
    int it = 0;
    double rel = 1.0;
    // inner solves stop once they no longer halve their residual within
    // INNER_STALL iterations: FP32 vectors cannot resolve corrections below
    // about kappa * u32, and refinement then continues in FP64
    double mark = 1.0;
    int mark_it = 0;
    while (it < maxit) {
        ++it;
        if (use_graph) IBM_HIP(hipGraphLaunch(*graph, s));
        else bicg_iteration<T, TX>(c, y, r, rh, p, v, ph, sh, t, s);
        read_scalars(c, s);
        const double st = c.hsc[S_STATUS];
        rel = c.hsc[S_REL];
        if (log_level() >= 2)
            fprintf(stderr, "[ibm]   it %d rel %.3e status %g alpha %.3e omega %.3e sinks %.3e %.3e\n", it, rel, st,
                    c.hsc[S_ALPHA], c.hsc[S_OMEGA], c.hsc[S_SINKP], c.hsc[S_SINKS]);
        if (st >= 2.0 || !std::isfinite(rel)) { *rc = IBM_EBREAKDOWN; break; }
        if (rel <= tol) {
            if constexpr (!std::is_same<T, TX>::value || !std::is_same<TR, T>::value) {
                *rc = IBM_OK;  // inner solves: no true check
                break;
            } else {
                if (!true_check) { *rc = IBM_OK; break; }
                int np = launch_apply<T>(c, M_PINNED, true, 2, (const T *)y, t, rhs, nullptr, rh, nullptr, s);
                k_fin<<<1, 1024, 0, s>>>(c.part.p + PSTRIDE, PSTRIDE, np, FIN_SUM, S_TMP, 0.0, c.sc.p);
                read_scalars(c, s);
                double trel = std::sqrt(c.hsc[S_TMP] / c.hsc[S_BN2]);
                rel = trel;
                if (trel <= tol) { *rc = IBM_OK; break; }
                // residual replacement
                k_copy<T, T><<<W.nb, TPB, 0, s>>>(W, t, r);
                k_dot2<T><<<W.nb, TPB, 0, s>>>(W, rh, r, c.part.p, PSTRIDE);
                fin(c, W.nb, FIN_REPLACE, 0, 0.0, s);
                continue;
            }
        }
        if constexpr (!std::is_same<T, TX>::value) {
            if (rel < 0.5 * mark) {
                mark = rel;
                mark_it = it;
            } else if (it - mark_it >= INNER_STALL) {
                if (log_enabled()) fprintf(stderr, "[ibm]   inner stagnation at %.3e after %d iterations\n", rel, it);
                break;  // *rc stays IBM_ENOCONV
            }
        }
        if (st == 1.0) {  // rho breakdown: restart with rh = r
            k_fill<T><<<W.nb, TPB, 0, s>>>(W, p, 0.0);
            k_fill<T><<<W.nb, TPB, 0, s>>>(W, v, 0.0);
            k_copy_norm<T, T><<<W.nb, TPB, 0, s>>>(W, r, rh, (T *)nullptr, c.part.p);
            fin(c, W.nb, FIN_RESTART, 0, 0.0, s);
        }
    }
    *relout = rel;
    return it;
}

// ------------------------------------------------------------------ RHS, gauge (split layout)
// ghost rows of the RHS, in split or (NAT) natural order
template <bool NAT>
__global__ void __launch_bounds__(TPB) k_rhs_ghost(Lv L, Sp S, const double *dlb, const double *g, double *b)
{
    for (int r = blockIdx.x * TPB + threadIdx.x; r < S.nrows; r += gridDim.x * TPB) {
        const long long u = ghost_unknown(S, r);
        b[NAT ? natural_of(L, u) : u] = g ? S.rsG[r] * dlb[r] * g[r] : 0.0;
    }
}

template <class T>
__global__ void __launch_bounds__(TPB) k_shift(Lv L, Walk W, long long pin, T *x)
{
    const double c = ld(x, pin);
    WALK_BEGIN(W, p)
        if (p != pin && (p >= 2 * L.Nh || active0(L.f[p]))) st(x, p, ld(x, p) - c);
    WALK_END
}

__global__ void k_shift_pin(long long pin, double *x) { x[pin] = 0.0; }

// unpinned residual at the pin (the inconsistency the pin absorbs)
__global__ void k_pinres(Lv L, long long pin, const double *x, double *sc)
{
    if (threadIdx.x || blockIdx.x) return;
    int c, h, j, k, i;
    decode_slot(L, pin, c, h, j, k, i);
    double dg;
    const double off = nbsum(L, x + (long long)(1 - c) * L.Nh, h, j, k, i, dg);
    sc[S_TMP] = off - dg * x[pin];
}

}  // namespace

// ------------------------------------------------------------------ setup
size_t estimate_bytes(int nx, int ny, int nz, long long nrows, int precision)
{
    long long Nh = (long long)((nx + 1) / 2) * ny * nz;
    long long Nt = 2 * Nh + nrows;
    size_t b = (size_t)2 * Nh;  // flags
    if (2 * Nh >= WALK_MIN_CELLS) b += (size_t)(2 * Nh) / 128 * 2 + (size_t)nrows * 8;  // near units' bits and lists
    b += (size_t)nrows * (8 * 4 + 8 * 8 + 16 + 8 + 4 + 6 * 4 + 4 + 8 * 4 + 8);
    b += (size_t)nrows * (16 * 4 + 6 * 4 + 2 * (4 + 6 * 4) + 8);  // coded rows, adjacent cells
    b += (size_t)Nt * 8 * (precision == IBM_PREC_MIXED ? 4 : 10);
    if (precision == IBM_PREC_MIXED) b += (size_t)Nt * (4 * 8 + 8);
    long long Nc = 2 * Nh;
    size_t coarse = 0;
    while (true) {
        Nc /= 8;
        if (Nc < 8) break;
        coarse += (size_t)Nc * (precision == IBM_PREC_MIXED ? (4 + 2 + 1) : (8 * 2 + 1));
        if (Nc <= BRICK_MAX_CELLS) coarse += (size_t)Nc / 2 * (precision == IBM_PREC_MIXED ? 4 : 8);
    }
    b += coarse;
    b += (size_t)PSTRIDE * 4 * 8;
    return b;
}

// grow-only device buffer: reallocated (contents dropped) when too small
template <class T>
void reserve(DBuf<T> &b, size_t n)
{
    if (!b.p || b.n < n) b.alloc(n);
}

// (the passes keep a column's half-index and row in 16 bits each; longer boxes
// take the one-sweep kernels)
bool walk_wanted(const poisson_ctx &c)
{
    return c.opts.precond == IBM_PRECOND_MG && c.opts.nu1 == 2 && c.opts.nu2 == 2 && c.lv.size() > 1 &&
           c.N >= WALK_MIN_CELLS && c.lv[0].H <= 0xffff && c.lv[0].n[1] <= 0xffff;
}

// Lists of the fused level-0 pass for the current classification, in two
// halves: bits of the near and listed units and their counts; then, with the
// counts read, the lists and the blocks' plane runs.
void count_units(poisson_ctx &c, CellLists &U, hipStream_t s)
{
    const Level &Z = c.lv[0];
    const int nux = (Z.H + 3) / 4, nuy = (Z.n[1] + 3) / 4, nuz = (Z.n[2] + 3) / 4;
    const long long nu = (long long)nux * nuy * nuz;
    k_unit_cells<<<cdiv(16 * nu, NU_T), NU_T, 0, s>>>(Z.lv, nux, nuy, nu, c.ubits[0].p);
    k_unit_near<<<cdiv(nu, 256), 256, 0, s>>>(nux, nuy, nuz, c.ubits[0].p, c.ubits[1].p);
    k_unit_list<<<cdiv(nu, 256), 256, 0, s>>>(nux, nuy, nuz, c.ubits[1].p, c.ubits[0].p);
    U.count(c.ssum.p->units, s);
}
void plan_walk(poisson_ctx &c, CellLists *U, const int n[2], hipStream_t s)
{
    c.walk = walk_wanted(c);
    if (!c.walk) return;
    const Level &Z = c.lv[0];
    c.near = Near{};
    if (U) {
        const int nux = (Z.H + 3) / 4, nuy = (Z.n[1] + 3) / 4, nuz = (Z.n[2] + 3) / 4;
        reserve(c.units, std::max(n[0], 1));
        reserve(c.nunits, std::max(n[1], 1));
        U->fill(c.units.p, c.nunits.p, nullptr, s);
        c.near = Near{c.units.p, c.ubits[0].p, n[0], nux, nuy, nuz};
        c.nearres = Near{c.nunits.p, c.ubits[0].p, n[1], nux, nuy, nuz};
        c.walk = n[0] <= walk_max_near(Z.H, Z.n[1], c.mixed) * U->N;
    }
    // planes per block: a block fills a CU and computes eight planes more than
    // it owns; the length that takes the fewest plane steps over the rounds
    WalkGeo &g = c.wg;
    g.ntx = (Z.H + WK_OH - 1) / WK_OH;
    g.nty = (Z.n[1] + WK_OJ - 1) / WK_OJ;
    long long best = -1;
    for (int kz = 4; kz <= WK_KZMAX; kz += 4) {
        const int ncz = (Z.n[2] + kz - 1) / kz;
        const long long cost = ((long long)g.ntx * g.nty * ncz + 255) / 256 * (kz + 8 + 2);
        if (best < 0 || cost < best) {
            best = cost;
            g.kz = kz;
            g.ncz = ncz;
        }
    }
    g.nb = (g.ntx * g.nty * g.ncz + 7) / 8 * 8;
    if ((long long)g.nb + c.near.nb() > PSTRIDE) c.walk = false;
    c.beside = c.N >= BESIDE_MIN_CELLS;
    if (c.walk && c.beside && !c.ns) {
        IBM_HIP(hipStreamCreateWithFlags(&c.ns, hipStreamNonBlocking));
        IBM_HIP(hipEventCreateWithFlags(&c.ef, hipEventDisableTiming));
        IBM_HIP(hipEventCreateWithFlags(&c.en, hipEventDisableTiming));
    }
}

// Coded sparse rows of the fused half-sweeps, from the rows in slot numbering;
// A: the adjacent cells, na of them (null without closed ghosts).
void code_rows(poisson_ctx &c, const ibm_stencils *st, CellLists *A, int na, hipStream_t s)
{
    const Level &Z = c.lv[0];
    Rows &R = c.rows;
    R = Rows{};
    R.N2 = c.N2;
    R.Nh = Z.Nh;
    R.pin = c.pin;
    R.ng = (int)c.ng;
    R.nrows = (int)c.nrows;
    R.nm = (int)c.nm;
    if (!c.nrows) return;
    if (A) {
        R.na = na;
        reserve(c.aslot, std::max(na, 1));
        A->fill(c.aslot.p, nullptr, nullptr, s);
    }
    const CodeMap M{Z.lv, st->cell.p, st->cell.p + c.ng, c.aslot.p, R.ng, R.nm, R.na};
    auto blocks = [](long long n) { return (int)std::min<long long>(std::max<long long>((n + TPB - 1) / TPB, 1), 4096); };
    reserve(c.code, 8 * c.nrows);
    reserve(c.rix, 8 * c.nrows);
    reserve(c.mcode, std::max<long long>(6 * c.nm, 1));
    reserve(c.acode, std::max(6 * R.na, 1));
    k_code_columns<<<blocks(8 * c.nrows), TPB, 0, s>>>(M, 8 * c.nrows, c.rcol.p, c.code.p, c.rix.p);
    if (c.nm) k_code_columns<<<blocks(6 * c.nm), TPB, 0, s>>>(M, 6 * c.nm, c.mcol.p, c.mcode.p, nullptr);
    if (R.na) k_code_adjacent<<<blocks(R.na), TPB, 0, s>>>(M, c.acode.p);
    IBM_LAUNCH_CHECK();
    R.rslot = c.rslot.p;
    R.code = c.code.p;
    R.rix = c.rix.p;
    R.rw = c.rw.p;
    R.rsG = c.rsG.p;
    R.mslot = c.mslot.p;
    R.mcode = c.mcode.p;
    R.mcolor = c.mcolor.p;
    R.aslot = c.aslot.p;
    R.acode = c.acode.p;
}

// Flag-dependent parts of a context -- level-0 flags, ghost and membrane rows
// in slot numbering, fluid and pin volumes, coarse masks, vectors sized by
// the unknown count -- built on the device from the classification and the
// ghost-row table.  Runs at set-up and again when bodies move.
void setup_geometry(poisson_ctx &c, const uint8_t *flags, const ibm_stencils *st)
{
    const HostGrid &g = c.g;
    for (int d = 0; d < 3; ++d) IBM_REQUIRE(g.n[d] == st->n[d], IBM_EINVAL, "stencil table of another grid");
    IBM_REQUIRE(st->pin >= 0 && st->pin < c.N, IBM_EGEOM, "no fluid cell to pin");
    // row columns are int32 slots: the cell slots (with row padding), then the membrane ghost unknowns
    IBM_REQUIRE(c.N2 + st->nm < (1LL << 31), IBM_EINVAL, "more than 2^31 unknowns with padding and membrane ghosts");
    hipStream_t s = c.cs;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int nl = (int)c.lv.size();
    Level &Z = c.lv[0];
    c.ng = st->ng;
    c.nm = st->nm;
    c.nrows = st->ng + st->nm;
    c.n_fallback = st->nfallback;
    const long long R = c.nrows, nm = c.nm, N = c.N;
    const SlotMap sm{nx, ny, Z.H, Z.Nh, N, c.N2};
    {
        const long long p = st->pin;
        const int i = (int)(p % nx), j = (int)((p / nx) % ny), k = (int)(p / ((long long)nx * ny));
        c.pin = host_slot(Z.H, ny, Z.Nh, i, j, k);
        c.vol_pin = Z.hw[0][i] * Z.hw[1][j] * Z.hw[2][k];
    }
    // the captured iterations and the vectors below may change
    IBM_HIP(hipStreamSynchronize(s));
    c.drop_graphs();
    const bool w8 = nx % 8 == 0 && ((uintptr_t)flags & 7) == 0;
    const Walk WF = make_walk(w8 ? Z.Nh / 4 : Z.Nh);
    if (w8) k_setup_flags0<true><<<WF.nb, TPB, 0, s>>>(Z.lv, WF, flags, Z.m.p, c.part.p);
    else k_setup_flags0<false><<<WF.nb, TPB, 0, s>>>(Z.lv, WF, flags, Z.m.p, c.part.p);
    k_fin<<<1, 1024, 0, s>>>(c.part.p, PSTRIDE, WF.nb, FIN_SUM, 0, 0.0, c.ssum.p->volume);  // fluid volume
    // ghost and membrane rows
    const long long R1 = std::max<long long>(R, 1), M1 = std::max<long long>(nm, 1);
    reserve(c.rslot, std::max<long long>(c.ng, 1));
    reserve(c.rcol, R1 * 8);
    reserve(c.rw, R1 * 8);
    reserve(c.rsG, R1);
    reserve(c.rdlb, R1);
    reserve(c.gtmp, R1);
    reserve(c.gtmp2, R1);
    reserve(c.mtmp, M1);
    reserve(c.rmrow, R1 * 8);
    reserve(c.mslot, M1);
    reserve(c.mcol, M1 * 6);
    reserve(c.mcolor, M1);
    auto blocks = [](long long n) { return (int)std::min<long long>(std::max<long long>((n + TPB - 1) / TPB, 1), 4096); };
    if (R) {
        k_setup_rows<<<blocks(8 * R), TPB, 0, s>>>(sm, c.ng, R, st->cell.p, st->col.p, st->w.p, st->sG.p, st->dlb.p,
                                                  c.rslot.p, c.rcol.p, c.rw.p, c.rsG.p, c.rdlb.p);
    }
    if (nm) IBM_HIP(hipMemsetAsync(&c.ssum.p->err, 0, sizeof(int), s));
    if (nm)
        k_setup_membrane<<<blocks(nm), TPB, 0, s>>>(sm, nz, nm, st->cell.p + c.ng, flags, c.mslot.p, c.mcol.p,
                                                    c.mcolor.p, &c.ssum.p->err);
    if (R && nm)
        k_map_mrows<<<blocks(8 * R), TPB, 0, s>>>(8 * R, st->col.p, N, flags, st->cell.p + c.ng, nm, c.rmrow.p);
    // the slots those rows read (the first half-sweep of a V-cycle zeroes
    // these, not every black slot)
    if (R) k_mark_read<<<blocks(8 * R), TPB, 0, s>>>(8 * R, c.rcol.p, c.N2, Z.m.p);
    if (nm) k_mark_read<<<blocks(6 * nm), TPB, 0, s>>>(6 * nm, c.mcol.p, c.N2, Z.m.p);
    // the coarse masks level by level with their active volumes
    for (int l = 1; l < nl; ++l) {
        Level &F = c.lv[l - 1], &C = c.lv[l];
        const uint8_t *fine = l == 1 ? flags : c.hact[l & 1].p;
        uint8_t *ha = c.hact[(l + 1) & 1].p;
        k_coarse_active<<<blocks(C.N), TPB, 0, s>>>(F.n[0], F.n[1], C.n[0], C.n[1], C.N, fine, l == 1, ha);
        k_coarse_mask<<<C.walk.nb, TPB, 0, s>>>(C.lv, C.walk, ha, C.m.p, c.part.p, PSTRIDE);
        k_fin<<<1, 1024, 0, s>>>(c.part.p, PSTRIDE, C.walk.nb, FIN_SUM, l, 0.0, c.ssum.p->volume);
        k_fin<<<1, 1024, 0, s>>>(c.part.p + PSTRIDE, PSTRIDE, C.walk.nb, FIN_SUM, l, 0.0, c.ssum.p->inactive);
    }
    IBM_LAUNCH_CHECK();
    // lists that smoothing takes: their counts come back with the sums, in one wait
    c.flat = c.opts.precond == IBM_PRECOND_MG && c.N < WALK_MIN_CELLS &&
             (c.nrows <= FLAT_ROWS || (c.ng && c.nm));
    std::unique_ptr<CellLists> adjacent, units;
    if (R && walk_wanted(c)) {
        const long long nu = (long long)((Z.H + 3) / 4) * ((ny + 3) / 4) * ((nz + 3) / 4);
        for (auto &q : c.ubits) reserve(q, nu);
        units.reset(new CellLists(c.ubits[0].p, nu, 2, UB_LIST, UB_NEAR));
        count_units(c, *units, s);
    }
    if (c.ng && (c.flat || (walk_wanted(c) && c.nrows <= FEW_ROWS))) {
        k_mark_adjacent<<<Z.walk.nb, TPB, 0, s>>>(Z.lv, Z.walk, Z.m.p);
        IBM_LAUNCH_CHECK();
        adjacent.reset(new CellLists(Z.m.p, c.N2, 1, F_ADJ));
        adjacent->count(&c.ssum.p->adjacent, s);
    }
    SetupSums hs;
    IBM_HIP(hipMemcpyAsync(&hs, c.ssum.p, sizeof hs, hipMemcpyDeviceToHost, s));
    IBM_HIP(hipStreamSynchronize(s));
    IBM_REQUIRE(!nm || hs.err == 0, IBM_EGEOM, "cut link without ghost");
    plan_walk(c, units.get(), hs.units, s);
    c.few = c.walk && c.nrows <= FEW_ROWS;
    if (c.few || c.flat) code_rows(c, st, adjacent.get(), hs.adjacent, s);
    c.vol_fluid = hs.volume[0];
    for (int l = 1; l < nl; ++l) {
        c.lv[l].volA = hs.volume[l];
        c.lv[l].n_inactive = (long long)hs.inactive[l];
    }
    Sp &S = c.sp;
    S.N2 = c.N2;
    S.pin = c.pin;
    S.nrows = (int)R;
    S.ng = (int)c.ng;
    S.rslot = c.rslot.p; S.rcol = c.rcol.p; S.rw = c.rw.p; S.rsG = c.rsG.p;
    S.nm = (int)nm;
    S.mslot = c.mslot.p; S.mcol = c.mcol.p; S.mcolor = c.mcolor.p;
    S.rmrow = c.rmrow.p;
    // vectors over the unknowns: exact size at set-up; when an update needs
    // more, every held vector is reallocated with headroom for later updates
    const long long Nt = c.N2 + nm;
    const bool first = !c.x.p;
    c.Nt = Nt;
    c.W0 = make_walk(Nt);
    c.Wp = make_walk(Z.Nh + nm);
    c.W4 = make_walk((Nt + 3) / 4, W4MAXB);
    const long long cap = first ? Nt : Nt + nm / 4 + 1024;
    DBuf<double> *dv[] = {&c.x, &c.r, &c.b, &c.t, &c.rh, &c.p, &c.v, &c.ph, &c.sh, &c.rsp, &c.d64, &c.r2};
    DBuf<float> *fv[] = {&c.fr, &c.frh, &c.fp, &c.fv, &c.fph, &c.fsh, &c.ft, &c.frsp};
    if (first) {
        c.x.alloc(Nt); c.r.alloc(Nt); c.b.alloc(Nt); c.t.alloc(Nt);
        if (!c.mixed) {
            c.rh.alloc(Nt); c.p.alloc(Nt); c.v.alloc(Nt); c.ph.alloc(Nt); c.sh.alloc(Nt); c.rsp.alloc(Nt);
        } else {
            c.d64.alloc(Nt); c.fr.alloc(Nt); c.frh.alloc(Nt); c.fp.alloc(Nt); c.fv.alloc(Nt);
            c.fph.alloc(Nt); c.fsh.alloc(Nt); c.ft.alloc(Nt); c.frsp.alloc(Nt);
        }
    } else {
        for (auto *q : dv)
            if (q->p && (long long)q->n < Nt) q->alloc(cap);
        for (auto *q : fv)
            if (q->p && (long long)q->n < Nt) q->alloc(cap);
    }
    std::vector<double> sc0(S_COUNT, 0.0);
    sc0[S_VPIN] = c.vol_pin;
    IBM_HIP(hipMemcpyAsync(c.sc.p, sc0.data(), S_COUNT * 8, hipMemcpyHostToDevice, s));
    IBM_HIP(hipStreamSynchronize(s));
    c.bytes = estimate_bytes(nx, ny, nz, c.nrows, c.opts.precision);
    IBM_REQUIRE(c.W0.nb <= PSTRIDE - 2048, IBM_EINVAL, "grid too large");
}

poisson_ctx *setup(const ibm_grid *grid, const uint8_t *flags, const ibm_stencils *st, const poisson_opts *opts)
{
    IBM_REQUIRE(flags && st, IBM_EINVAL, "null argument");
    std::unique_ptr<poisson_ctx> c(new poisson_ctx());
    if (opts) c->opts = *opts; else poisson_default_opts(&c->opts);
    poisson_opts &o = c->opts;
    IBM_REQUIRE(o.tol > 0 && o.max_iter > 0 && o.nu1 >= 1 && o.nu2 >= 0 && o.coarse_sweeps >= 1, IBM_EINVAL,
                "bad solver options");
    IBM_REQUIRE(o.precond == IBM_PRECOND_MG || (o.precond == IBM_PRECOND_SRJ && o.srj_sweeps >= 1 &&
                                                 o.srj_sweeps <= IBM_SRJ_MAX_SWEEPS),
                IBM_EINVAL, "bad preconditioner options");
    c->mixed = o.precision == IBM_PREC_MIXED;
    if (o.precond == IBM_PRECOND_SRJ) c->srj_w = srj_schedule(o.srj_sweeps);
    c->g = read_grid(grid);
    for (int d = 0; d < 3; ++d) IBM_REQUIRE(c->g.n[d] == st->n[d], IBM_EINVAL, "stencil table of another grid");
    IBM_HIP(hipStreamCreateWithFlags(&c->cs, hipStreamNonBlocking));
    IBM_HIP(hipEventCreate(&c->e0));
    IBM_HIP(hipEventCreate(&c->e1));
    IBM_HIP(hipEventCreateWithFlags(&c->ej, hipEventDisableTiming));
    c->hsc = pinned_slot();
    hipStream_t s = c->cs;
    const HostGrid &g = c->g;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    c->N = (long long)nx * ny * nz;
    // levels: halve while every dimension is even and the smallest exceeds 4
    int nl = 1;
    {
        int n[3] = {nx, ny, nz};
        while (nl < 16) {
            bool even = n[0] % 2 == 0 && n[1] % 2 == 0 && n[2] % 2 == 0;
            int mn = std::min(n[0], std::min(n[1], n[2]));
            if (!even || mn <= 4) break;
            for (int d = 0; d < 3; ++d) n[d] /= 2;
            ++nl;
        }
    }
    c->lv.resize(nl);
    Image I;  // every level's coefficients and maps: one copy instead of up to fifteen per level
    std::vector<double> faces[3];
    for (int d = 0; d < 3; ++d) faces[d] = g.f[d];
    for (int l = 0; l < nl; ++l) {
        Level &L = c->lv[l];
        for (int d = 0; d < 3; ++d) L.n[d] = g.n[d] >> l;
        if (l > 0)
            for (int d = 0; d < 3; ++d) {
                std::vector<double> cf(L.n[d] + 1);
                for (int i = 0; i <= L.n[d]; ++i) cf[i] = faces[d][2 * i];
                faces[d] = cf;
            }
        level_geometry(L, faces, I);
    }
    // level 0: shorter plane runs per thread (more tiles) measured faster;
    // the half-sweep addresses a tile's planes with 32-bit byte offsets
    c->lv[0].geo = make_geo(c->lv[0].H, c->lv[0].n[1], c->lv[0].n[2], 16384);
    c->lv[0].geo2 = make_geo_rows2(c->lv[0].H, c->lv[0].n[1], c->lv[0].n[2], 8192);
    IBM_REQUIRE(plane_span_ok((long long)c->lv[0].H * c->lv[0].n[1], std::max(c->lv[0].geo.kz, c->lv[0].geo2.kz),
                              sizeof(double)),
                IBM_EINVAL, "grid planes too large for the level-0 sweep's 32-bit offsets");
    c->N2 = 2 * c->lv[0].Nh;
    // prolongation maps of each level from its coarse parent
    for (int l = 1; l < nl; ++l) {
        Level &F = c->lv[l - 1], &C = c->lv[l];
        for (int d = 0; d < 3; ++d) {
            int nf = F.n[d], nc = C.n[d];
            std::vector<int> pi(nf);
            std::vector<double> pt(nf);
            for (int i = 0; i < nf; ++i) {
                double x = F.hc[d][i];
                x = std::min(std::max(x, C.hc[d][0]), C.hc[d][nc - 1]);
                int I0 = 0;
                while (I0 + 1 <= nc - 2 && C.hc[d][I0 + 1] <= x) ++I0;
                pi[i] = I0;
                pt[i] = (x - C.hc[d][I0]) / (C.hc[d][I0 + 1] - C.hc[d][I0]);
            }
            F.pi[d] = I.put(pi);
            F.pt[d] = I.put(pt);
        }
    }
    I.upload(c->coef, s);
    // tail start: the coarsest levels that fit one workgroup's LDS and, the
    // first of them, its registers (two cell pairs per thread; one below)
    for (int pass = 0; pass < 2; ++pass) {
        const size_t tsz = pass ? sizeof(double) : sizeof(float);
        int &t0 = pass ? c->tail0d : c->tail0;
        t0 = nl;
        for (int l = nl - 1; l >= 1 && (nl - l) <= 8; --l) {
            if (c->lv[l].Nh > TAIL_U * TAIL_T) break;
            int off = 0, m, xo, bo;
            for (int q = l; q < nl; ++q) tail_layout(c->lv[q], tsz, q == l, off, m, xo, bo);
            for (int q = l; q < nl; ++q) off += tail_coef_bytes(c->lv[q].n[0], c->lv[q].n[1], c->lv[q].n[2]);
            if (off > TAIL_LDS) break;
            t0 = l;
        }
    }
    if (!c->mixed) c->tail0 = c->tail0d;
    // device views, masks and coarse storage
    for (int l = 0; l < nl; ++l) {
        Level &L = c->lv[l];
        L.m.alloc(2 * L.Nh);
        Lv &v = L.lv;
        v.nx = L.n[0]; v.ny = L.n[1]; v.nz = L.n[2]; v.H = L.H; v.Nh = L.Nh;
        v.fH = make_fdiv(L.H);
        v.fy = make_fdiv(L.n[1]);
        for (int d = 0; d < 3; ++d) {
            v.cp[d] = (const double *)(c->coef.p + L.cp[d]);
            v.cm[d] = (const double *)(c->coef.p + L.cm[d]);
            v.w[d] = (const double *)(c->coef.p + L.w[d]);
        }
        v.f = L.m.p;
        if (l + 1 < nl)
            for (int d = 0; d < 3; ++d) {
                L.pm.pi[d] = (const int *)(c->coef.p + L.pi[d]);
                L.pm.pt[d] = (const double *)(c->coef.p + L.pt[d]);
            }
        if (l > 0) {
            L.br = make_brick(L.n[0], L.n[1], L.n[2]);
            L.brick = L.N <= BRICK_MAX_CELLS && ((long long)L.br.gx * L.br.gy * L.br.gz <= BRICK_MAX || L.n[0] <= BRICK_NARROW) &&
                      o.nu1 <= 2 && o.nu2 >= 1 && o.nu2 <= 2;
            if (c->mixed) { L.x32.alloc(2 * L.Nh); L.b16.alloc(2 * L.Nh); if (L.brick) L.k32.alloc(L.Nh); }
            else { L.x64.alloc(2 * L.Nh); L.b64.alloc(2 * L.Nh); if (L.brick) L.k64.alloc(L.Nh); }
        }
    }
    IBM_REQUIRE(c->lv[0].geo.nb <= PSTRIDE - 2048, IBM_EINVAL, "grid too large");
    for (auto &L : c->lv) {
        IBM_REQUIRE(L.geo.nb <= PSTRIDE && L.geon.nb <= PSTRIDE, IBM_EINVAL, "grid too large");
        IBM_REQUIRE(plane_span_ok((long long)L.H * L.n[1], L.geo.kz, sizeof(double)), IBM_EINVAL,
                    "grid planes too large for the sweeps' 32-bit offsets");
    }
    c->Wc = make_walk(c->N2);
    c->sc.alloc(S_COUNT);
    c->part.alloc((size_t)PSTRIDE * 4);
    c->ssum.alloc(1);
    if (nl > 1) {
        c->hact[0].alloc(c->lv[1].N);
        if (nl > 2) c->hact[1].alloc(c->lv[2].N);
    }
    setup_geometry(*c, flags, st);
    return c.release();
}

// ------------------------------------------------------------------ solve
struct StreamJoin {
    poisson_ctx &c;
    hipStream_t user;
    StreamJoin(poisson_ctx &cc, hipStream_t u) : c(cc), user(u)
    {
        IBM_HIP(hipEventRecord(c.ej, user));
        IBM_HIP(hipStreamWaitEvent(c.cs, c.ej, 0));
    }
    ~StreamJoin()
    {
        (void)hipEventRecord(c.ej, c.cs);
        (void)hipStreamWaitEvent(user, c.ej, 0);
    }
};

namespace {

void to_split(poisson_ctx &c, const double *nat, double *spl, long long tail, hipStream_t s)
{
    k_to_split<false><<<c.Wp.nb, TPB, 0, s>>>(c.L0(), c.Wp, nat, pairs_aligned(c.L0().nx, nat), spl, tail, nullptr);
    IBM_LAUNCH_CHECK();
}

template <int MODE>
void from_split(poisson_ctx &c, const double *spl, double *nat, long long tail, hipStream_t s)
{
    k_from_split<MODE><<<c.Wp.nb, TPB, 0, s>>>(c.L0(), c.Wp, spl, nat, pairs_aligned(c.L0().nx, nat), tail, c.pin,
                                               c.sc.p + S_TMP2);
    IBM_LAUNCH_CHECK();
}

// whether the na values from a and the nb values from b share memory
bool overlap(const double *a, long long na, const double *b, long long nb)
{
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + nb * sizeof(double) && y < x + na * sizeof(double);
}

// b (split, or NAT natural) from raw natural f and optional g; NAT: b overlaps neither
template <bool NAT = false>
void assemble_rhs(poisson_ctx &c, const double *f, const double *gval, double *b, hipStream_t s)
{
    const int nx = c.L0().nx;
    k_vsum<true, false><<<c.Wp.nb, TPB, 0, s>>>(c.L0(), c.Wp, f, pairs_aligned(nx, f), c.part.p);
    fin(c, c.Wp.nb, FIN_MEAN, S_TMP, c.vol_fluid, s);
    k_rhs<NAT><<<c.Wp.nb, TPB, 0, s>>>(c.L0(), c.Wp, c.pin, f, pairs_aligned(nx, f), c.sc.p + S_TMP, b,
                                       pairs_aligned(nx, b), c.nm);
    if (c.nrows) k_rhs_ghost<NAT><<<sparse_blocks(c.nrows), TPB, 0, s>>>(c.L0(), c.sp, c.rdlb.p, gval, b);
    IBM_LAUNCH_CHECK();
}

// FP64 storage of a mixed context, allocated on first need: the coarse FP64
// levels and the FP64 Krylov vectors (the FP64 cycle uses its own tail start)
void ensure_fp64(poisson_ctx &c)
{
    for (size_t l = 1; l < c.lv.size(); ++l) {
        Level &L = c.lv[l];
        if (!L.x64.p) L.x64.alloc(2 * L.Nh);
        if (!L.b64.p) L.b64.alloc(2 * L.Nh);
        if (L.brick && !L.k64.p) L.k64.alloc(L.Nh);
    }
    DBuf<double> *v[] = {&c.rh, &c.p, &c.v, &c.ph, &c.sh, &c.rsp, &c.r2};
    for (DBuf<double> *b : v)
        if (!b->p) b->alloc(c.Nt);
}

// true relative residual ||b - A x|| / ||b|| of the FP64 iterate (c.t is
// overwritten); for FP64 solves that end without a checked residual
double true_rel_residual(poisson_ctx &c, hipStream_t s)
{
    const Walk &W = c.W0;
    k_dot2<double><<<W.nb, TPB, 0, s>>>(W, c.b.p, c.b.p, c.part.p, PSTRIDE);
    k_fin<<<1, 1024, 0, s>>>(c.part.p, PSTRIDE, W.nb, FIN_SUM, S_TMP2, 0.0, c.sc.p);
    int np = launch_apply<double>(c, M_PINNED, true, 2, c.x.p, c.t.p, c.b.p, nullptr, c.b.p, nullptr, s);
    k_fin<<<1, 1024, 0, s>>>(c.part.p + PSTRIDE, PSTRIDE, np, FIN_SUM, S_TMP, 0.0, c.sc.p);
    IBM_LAUNCH_CHECK();
    read_scalars(c, s);
    const double bn2 = c.hsc[S_TMP2];
    return bn2 > 0.0 ? std::sqrt(c.hsc[S_TMP] / bn2) : 0.0;
}

// solve A x = b (assembled, in c.b, split) into c.x; returns status.  warm:
// c.x holds an initial guess (zero on inactive slots, zero at the pin)
int solve_core(poisson_ctx &c, poisson_stats *stats, hipStream_t s, bool warm = false)
{
    const poisson_opts &o = c.opts;
    int rc = IBM_ENOCONV, its = 0, outer = 0;
    double rel = 1.0;
    if (!c.mixed && !warm) {
        its = bicgstab<double, double>(c, c.b.p, c.x.p, c.r.p, c.rh.p, c.p.p, c.v.p, c.ph.p, c.sh.p, c.t.p, o.tol, o.max_iter,
                               true, &c.g64, s, &rc, &rel);
        if (log_enabled()) fprintf(stderr, "[ibm] fp64: %d iterations to %.3e (rc %d)\n", its, rel, rc);
    } else if (!c.mixed) {
        // FP64 from an initial guess: BiCGSTAB on the correction, A d = b - A x0
        const Walk &W = c.W0;
        reserve(c.d64, c.Nt);
        reserve(c.r2, c.Nt);
        k_dot2<double><<<W.nb, TPB, 0, s>>>(W, c.b.p, c.b.p, c.part.p, PSTRIDE);
        k_fin<<<1, 1024, 0, s>>>(c.part.p, PSTRIDE, W.nb, FIN_SUM, S_TMP2, 0.0, c.sc.p);
        int np = launch_apply<double>(c, M_PINNED, true, 2, c.x.p, c.r2.p, c.b.p, nullptr, c.b.p, nullptr, s);
        k_fin<<<1, 1024, 0, s>>>(c.part.p + PSTRIDE, PSTRIDE, np, FIN_SUM, S_TMP, 0.0, c.sc.p);
        IBM_LAUNCH_CHECK();
        read_scalars(c, s);
        const double bn2 = c.hsc[S_TMP2];
        const double rel0 = bn2 > 0.0 ? std::sqrt(c.hsc[S_TMP] / bn2) : 0.0;
        if (!std::isfinite(rel0)) {
            rc = IBM_EBREAKDOWN;
        } else if (bn2 == 0.0) {
            k_fill<double><<<W.nb, TPB, 0, s>>>(W, c.x.p, 0.0);
            rc = IBM_OK;
            rel = 0.0;
        } else if (rel0 <= o.tol) {
            rc = IBM_OK;
            rel = rel0;
        } else {
            double r1;
            its = bicgstab<double, double>(c, c.r2.p, c.d64.p, c.r.p, c.rh.p, c.p.p, c.v.p, c.ph.p, c.sh.p, c.t.p,
                                           o.tol / rel0, o.max_iter, true, &c.g64w, s, &rc, &r1);
            k_add<double><<<W.nb, TPB, 0, s>>>(W, c.x.p, c.d64.p);
            IBM_LAUNCH_CHECK();
            rel = r1 * rel0;
        }
        if (log_enabled())
            fprintf(stderr, "[ibm] fp64 from a guess (rel %.3e): %d iterations to %.3e (rc %d)\n", rel0, its, rel, rc);
    } else {
        // FP64 iterative refinement around FP32 inner solves
        const Walk &W = c.W0;
        if (!warm) k_fill<double><<<W.nb, TPB, 0, s>>>(W, c.x.p, 0.0);
        k_dot2<double><<<W.nb, TPB, 0, s>>>(W, c.b.p, c.b.p, c.part.p, PSTRIDE);
        k_fin<<<1, 1024, 0, s>>>(c.part.p, PSTRIDE, W.nb, FIN_SUM, S_TMP2, 0.0, c.sc.p);
        IBM_LAUNCH_CHECK();
        read_scalars(c, s);
        const double bn2 = c.hsc[S_TMP2];
        double prev = HUGE_VAL;
        bool inner_failed = false;
        for (outer = 0; outer <= o.max_outer; ++outer) {
            if (bn2 == 0.0) {
                k_fill<double><<<W.nb, TPB, 0, s>>>(W, c.x.p, 0.0);
                rc = IBM_OK;
                rel = 0.0;
                break;
            }
            // r64 = b - A x (pinned) and its norm
            int np = launch_apply<double>(c, M_PINNED, true, 2, c.x.p, c.r.p, c.b.p, nullptr, c.b.p, nullptr, s);
            k_fin<<<1, 1024, 0, s>>>(c.part.p + PSTRIDE, PSTRIDE, np, FIN_SUM, S_TMP, 0.0, c.sc.p);
            IBM_LAUNCH_CHECK();
            read_scalars(c, s);
            rel = std::sqrt(c.hsc[S_TMP] / bn2);
            if (!std::isfinite(rel)) { rc = IBM_EBREAKDOWN; break; }
            if (rel <= o.tol) { rc = IBM_OK; break; }
            if (rel > prev || inner_failed) {
                // refinement has stalled: either the FP32 correction made the
                // FP64 residual larger (the FP32 solves cannot resolve this
                // system: the condition number times the FP32 unit roundoff is
                // not small; that correction is undone), or the FP32 solve ran
                // out of iterations before its tolerance.  Finish with an FP64
                // BiCGSTAB on the remaining residual.
                const bool grew = rel > prev;
                if (grew) {
                    k_add<double><<<W.nb, TPB, 0, s>>>(W, c.x.p, c.d64.p, -1.0);
                    IBM_LAUNCH_CHECK();
                }
                const double base = grew ? prev : rel;
                if (log_enabled())
                    fprintf(stderr, "[ibm] outer %d: rel %.3e (previous %.3e, inner %s), refinement stalled: FP64 fallback\n",
                            outer, rel, prev, inner_failed ? "unconverged" : "converged");
                ensure_fp64(c);
                launch_apply<double>(c, M_PINNED, true, 2, c.x.p, c.r2.p, c.b.p, nullptr, c.b.p, nullptr, s);
                int frc;
                double frel;
                its += bicgstab<double, double>(c, c.r2.p, c.d64.p, c.r.p, c.rh.p, c.p.p, c.v.p, c.ph.p, c.sh.p,
                                                c.t.p, o.tol / base, o.max_iter, true, &c.g64, s, &frc, &frel);
                k_add<double><<<W.nb, TPB, 0, s>>>(W, c.x.p, c.d64.p);
                int np = launch_apply<double>(c, M_PINNED, true, 2, c.x.p, c.r.p, c.b.p, nullptr, c.b.p, nullptr, s);
                k_fin<<<1, 1024, 0, s>>>(c.part.p + PSTRIDE, PSTRIDE, np, FIN_SUM, S_TMP, 0.0, c.sc.p);
                IBM_LAUNCH_CHECK();
                read_scalars(c, s);
                rel = std::sqrt(c.hsc[S_TMP] / bn2);
                rc = frc == IBM_EBREAKDOWN ? frc : (rel <= o.tol ? IBM_OK : IBM_ENOCONV);
                if (log_enabled()) fprintf(stderr, "[ibm] fp64 fallback: rel %.3e (rc %d)\n", rel, rc);
                break;
            }
            if (outer == o.max_outer) { rc = IBM_ENOCONV; break; }
            prev = rel;
            // inner FP32 solve of A d = r64 (the inner residual vector starts as r64
            // rounded to FP32); it asks only for the reduction still needed,
            // never less than inner_tol
            int irc;
            double irel;
            const double itol = std::max(o.inner_tol, 0.5 * o.tol / rel);
            const int n_in = bicgstab<float, double>(c, (const double *)c.r.p, c.d64.p, c.fr.p, c.frh.p, c.fp.p, c.fv.p,
                                                     c.fph.p, c.fsh.p, c.ft.p, itol, o.max_iter, false, &c.g32, s,
                                                     &irc, &irel);
            its += n_in;
            if (log_enabled())
                fprintf(stderr, "[ibm] outer %d: rel %.3e, inner tol %.1e: %d iterations to %.2e (rc %d)\n", outer, rel,
                        itol, n_in, irel, irc);
            if (irc == IBM_EBREAKDOWN) { rc = irc; break; }
            inner_failed = irc == IBM_ENOCONV;
            k_add<double><<<W.nb, TPB, 0, s>>>(W, c.x.p, c.d64.p);
            IBM_LAUNCH_CHECK();
        }
    }
    // an FP64 solve that stopped at its iteration limit or at a breakdown
    // holds the recursively updated residual, not the true one
    if (!c.mixed && rc != IBM_OK && std::isfinite(rel)) rel = true_rel_residual(c, s);
    if (stats) {
        stats->iterations = its;
        stats->outer_steps = outer;
        stats->rel_residual = rel;
        stats->status = rc;
        stats->levels = (int)c.lv.size();
        stats->n_fallback = c.n_fallback;
    }
    return rc;
}

}  // namespace
}  // namespace ibm

// ------------------------------------------------------------------ C ABI
extern "C" void poisson_default_opts(poisson_opts *o)
{
    if (!o) return;
    o->precision = IBM_PREC_FP64;
    o->tol = 1e-10;
    o->max_iter = 200;
    o->nu1 = 2;
    o->nu2 = 2;
    o->coarse_sweeps = 32;
    o->inner_tol = 1e-3;
    o->max_outer = 10;
    o->use_graph = 1;
    o->precond = IBM_PRECOND_MG;
    o->srj_sweeps = 16;
}

extern "C" int32_t poisson_workspace_estimate(int32_t nx, int32_t ny, int32_t nz, int64_t n_rows, int32_t precision,
                                              size_t *bytes)
{
    return guarded([&] {
        IBM_REQUIRE(bytes && nx > 0 && ny > 0 && nz > 0, IBM_EINVAL, "bad arguments");
        *bytes = estimate_bytes(nx, ny, nz, n_rows, precision);
    });
}

extern "C" int32_t poisson_setup(const ibm_grid *grid, const uint8_t *flags_dev, const ibm_stencils *st,
                                 const poisson_opts *opts, size_t *workspace_bytes, poisson_ctx **out)
{
    return guarded([&] {
        IBM_REQUIRE(out, IBM_EINVAL, "null output");
        poisson_ctx *c = setup(grid, flags_dev, st, opts);
        if (workspace_bytes) *workspace_bytes = c->bytes;
        *out = c;
    });
}

extern "C" int32_t poisson_solve(poisson_ctx *c, const double *f_dev, const double *g_dev, double *x_dev,
                                 poisson_stats *stats, void *stream)
{
    return guarded([&] {
        IBM_REQUIRE(c && f_dev && x_dev, IBM_EINVAL, "null argument");
        StreamJoin j(*c, (hipStream_t)stream);
        hipStream_t s = c->cs;
        IBM_HIP(hipEventRecord(c->e0, s));
        assemble_rhs(*c, f_dev, g_dev, c->b.p, s);
        int rc = solve_core(*c, stats, s);
        // gauge: volume-weighted fluid mean removed from fluid, ghost and membrane-ghost values
        k_pinres<<<1, 64, 0, s>>>(c->L0(), c->pin, c->x.p, c->sc.p);
        k_vsum<false, false><<<c->Wp.nb, TPB, 0, s>>>(c->L0(), c->Wp, c->x.p, false, c->part.p);
        fin(*c, c->Wp.nb, FIN_MEAN, S_TMP2, c->vol_fluid, s);
        from_split<OUT_GAUGE>(*c, c->x.p, x_dev, c->nm, s);
        IBM_HIP(hipEventRecord(c->e1, s));
        read_scalars(*c, s);
        if (stats) {
            float ms = 0.f;
            IBM_HIP(hipEventElapsedTime(&ms, c->e0, c->e1));
            stats->solve_ms = ms;
            stats->pin_residual = c->hsc[S_TMP];
        }
        if (rc == IBM_ENOCONV) throw Error(IBM_ENOCONV, "iteration limit reached");
        if (rc == IBM_EBREAKDOWN) throw Error(IBM_EBREAKDOWN, "BiCGSTAB breakdown or non-finite values");
    });
}

extern "C" int32_t poisson_solve_from(poisson_ctx *c, const double *f_dev, const double *g_dev, const double *x0_dev,
                                      int64_t n_x0, double *x_dev, poisson_stats *stats, void *stream)
{
    return guarded([&] {
        IBM_REQUIRE(c && f_dev && x0_dev && x_dev, IBM_EINVAL, "null argument");
        IBM_REQUIRE(n_x0 == c->N || n_x0 == c->N + c->nm, IBM_EINVAL, "initial guess must hold N or N + n_mghost values");
        StreamJoin j(*c, (hipStream_t)stream);
        hipStream_t s = c->cs;
        IBM_HIP(hipEventRecord(c->e0, s));
        assemble_rhs(*c, f_dev, g_dev, c->b.p, s);
        // initial guess: the cells (and membrane ghost unknowns when given)
        // from x0, inactive slots zero, shifted to a zero pin value
        const bool ghosts = n_x0 > c->N;
        to_split(*c, x0_dev, c->x.p, ghosts ? c->nm : 0, s);
        if (c->nm && !ghosts)
            k_warm_membrane<<<(int)std::min<long long>((c->nm + TPB - 1) / TPB, 4096), TPB, 0, s>>>(c->sp, c->x.p);
        k_zero_inactive<<<c->Wc.nb, TPB, 0, s>>>(c->L0(), c->Wc, c->x.p);
        k_shift<double><<<c->W0.nb, TPB, 0, s>>>(c->L0(), c->W0, c->pin, c->x.p);
        k_shift_pin<<<1, 1, 0, s>>>(c->pin, c->x.p);
        IBM_LAUNCH_CHECK();
        int rc = solve_core(*c, stats, s, true);
        k_pinres<<<1, 64, 0, s>>>(c->L0(), c->pin, c->x.p, c->sc.p);
        k_vsum<false, false><<<c->Wp.nb, TPB, 0, s>>>(c->L0(), c->Wp, c->x.p, false, c->part.p);
        fin(*c, c->Wp.nb, FIN_MEAN, S_TMP2, c->vol_fluid, s);
        from_split<OUT_GAUGE>(*c, c->x.p, x_dev, c->nm, s);
        IBM_HIP(hipEventRecord(c->e1, s));
        read_scalars(*c, s);
        if (stats) {
            float ms = 0.f;
            IBM_HIP(hipEventElapsedTime(&ms, c->e0, c->e1));
            stats->solve_ms = ms;
            stats->pin_residual = c->hsc[S_TMP];
        }
        if (rc == IBM_ENOCONV) throw Error(IBM_ENOCONV, "iteration limit reached");
        if (rc == IBM_EBREAKDOWN) throw Error(IBM_EBREAKDOWN, "BiCGSTAB breakdown or non-finite values");
    });
}

extern "C" int32_t poisson_update(poisson_ctx *c, const uint8_t *flags_dev, const ibm_stencils *st)
{
    return guarded([&] {
        IBM_REQUIRE(c && flags_dev && st, IBM_EINVAL, "null argument");
        setup_geometry(*c, flags_dev, st);
    });
}

extern "C" int32_t ibm_fill_fresh(const ibm_grid *grid, const uint8_t *flags_old_dev, const uint8_t *flags_new_dev,
                                  double *x_dev, int64_t *n_fresh, void *stream)
{
    return guarded([&] {
        IBM_REQUIRE(grid && flags_old_dev && flags_new_dev && x_dev, IBM_EINVAL, "null argument");
        const HostGrid g = read_grid(grid);
        const long long N = (long long)g.n[0] * g.n[1] * g.n[2];
        hipStream_t s = (hipStream_t)stream;
        DBuf<int> cnt(1);
        IBM_HIP(hipMemsetAsync(cnt.p, 0, sizeof(int), s));
        const int nb = (int)std::min<long long>(std::max<long long>((N + TPB - 1) / TPB, 1), 8192);
        k_fill_fresh<<<nb, TPB, 0, s>>>(g.n[0], g.n[1], g.n[2], flags_old_dev, flags_new_dev, x_dev, cnt.p);
        IBM_LAUNCH_CHECK();
        int h = 0;
        IBM_HIP(hipMemcpyAsync(&h, cnt.p, sizeof(int), hipMemcpyDeviceToHost, s));
        IBM_HIP(hipStreamSynchronize(s));
        if (n_fresh) *n_fresh = h;
    });
}

extern "C" int32_t poisson_solve_assembled(poisson_ctx *c, const double *b_dev, double *x_dev, poisson_stats *stats,
                                           void *stream)
{
    return guarded([&] {
        IBM_REQUIRE(c && b_dev && x_dev, IBM_EINVAL, "null argument");
        StreamJoin j(*c, (hipStream_t)stream);
        hipStream_t s = c->cs;
        IBM_HIP(hipEventRecord(c->e0, s));
        to_split(*c, b_dev, c->b.p, c->nm, s);
        int rc = solve_core(*c, stats, s);
        from_split<OUT_PLAIN>(*c, c->x.p, x_dev, c->nm, s);
        IBM_HIP(hipEventRecord(c->e1, s));
        IBM_HIP(hipStreamSynchronize(s));
        if (stats) {
            float ms = 0.f;
            IBM_HIP(hipEventElapsedTime(&ms, c->e0, c->e1));
            stats->solve_ms = ms;
        }
        if (rc != IBM_OK) throw Error(rc, rc == IBM_ENOCONV ? "iteration limit reached" : "breakdown");
    });
}

extern "C" int32_t poisson_apply(poisson_ctx *c, const double *x_dev, double *y_dev, void *stream)
{
    return guarded([&] {
        IBM_REQUIRE(c && x_dev && y_dev, IBM_EINVAL, "null argument");
        StreamJoin j(*c, (hipStream_t)stream);
        hipStream_t s = c->cs;
        const long long n = c->N + c->nm;
        if (!overlap(x_dev, n, y_dev, n)) {
            const bool v2 = pairs_aligned(c->L0().nx, x_dev) && pairs_aligned(c->L0().nx, y_dev);
            const int nsp = (int)(c->nrows + c->nm);
            const Geo &G = c->lv[0].geo;
            if (v2) k_apply_nat<true><<<G.nb, TPB, 0, s>>>(c->L0(), G, c->pin, x_dev, y_dev);
            else k_apply_nat<false><<<G.nb, TPB, 0, s>>>(c->L0(), G, c->pin, x_dev, y_dev);
            if (nsp) k_sparse_nat<<<sparse_blocks(nsp), TPB, 0, s>>>(c->L0(), c->sp, x_dev, y_dev);
            IBM_LAUNCH_CHECK();
            return;
        }
        // in place: through split copies
        to_split(*c, x_dev, c->r.p, c->nm, s);
        launch_apply<double>(*c, M_PINNED, false, 0, c->r.p, c->t.p, nullptr, nullptr, nullptr, nullptr, s);
        from_split<OUT_PLAIN>(*c, c->t.p, y_dev, c->nm, s);
    });
}

extern "C" int32_t poisson_assemble_rhs(poisson_ctx *c, const double *f_dev, const double *g_dev, double *b_dev,
                                        void *stream)
{
    return guarded([&] {
        IBM_REQUIRE(c && f_dev && b_dev, IBM_EINVAL, "null argument");
        StreamJoin j(*c, (hipStream_t)stream);
        hipStream_t s = c->cs;
        const long long n = c->N + c->nm;
        if (!overlap(f_dev, c->N, b_dev, n) && !(g_dev && overlap(g_dev, c->nrows, b_dev, n))) {
            assemble_rhs<true>(*c, f_dev, g_dev, b_dev, s);
            return;
        }
        assemble_rhs(*c, f_dev, g_dev, c->r.p, s);
        from_split<OUT_PLAIN>(*c, c->r.p, b_dev, c->nm, s);
    });
}

extern "C" int32_t poisson_precond(poisson_ctx *c, const double *b_dev, double *x_dev, void *stream)
{
    return guarded([&] {
        IBM_REQUIRE(c && b_dev && x_dev, IBM_EINVAL, "null argument");
        IBM_REQUIRE(!c->mixed, IBM_EINVAL, "poisson_precond needs an FP64 context");
        StreamJoin j(*c, (hipStream_t)stream);
        hipStream_t s = c->cs;
        k_to_split<true><<<c->Wp.nb, TPB, 0, s>>>(c->L0(), c->Wp, b_dev, pairs_aligned(c->L0().nx, b_dev), c->r.p, c->nm,
                                                  c->part.p);
        fin(*c, c->Wp.nb, FIN_SINK, S_SINKP, 0.0, s);
        precond<double>(*c, c->r.p, c->t.p, c->sh.p, c->sc.p + S_SINKP, s);
        // shift: every active unknown minus the pin value, then the pin itself
        from_split<OUT_SHIFT>(*c, c->t.p, x_dev, c->nm, s);
        IBM_LAUNCH_CHECK();
    });
}

// Test hook, not part of the interface: what a mixed context's inner iterations
// apply, x = V-cycle(b) in FP32 with BF16 coarse right-hand sides, unshifted
// (poisson_precond takes FP64 contexts only).  first_phase != 0: the iterate
// of level 0 after the smoothing steps before the coarse correction instead
// (of the fused pass only its black cells leave the kernel: the rest is zero).
// b and x hold N + n_mghost doubles; b is rounded to FP32 on the way in.
extern "C" int32_t ibm_test_inner_precond(poisson_ctx *c, const double *b_dev, double *x_dev, int32_t first_phase,
                                          void *stream)
{
    return guarded([&] {
        IBM_REQUIRE(c && b_dev && x_dev && c->mixed && c->opts.precond == IBM_PRECOND_MG, IBM_EINVAL,
                    "needs a mixed multigrid context");
        StreamJoin j(*c, (hipStream_t)stream);
        hipStream_t s = c->cs;
        k_to_split<true><<<c->Wp.nb, TPB, 0, s>>>(c->L0(), c->Wp, b_dev, pairs_aligned(c->L0().nx, b_dev), c->r.p, c->nm,
                                                  c->part.p);
        fin(*c, c->Wp.nb, FIN_SINK, S_SINKP, 0.0, s);
        k_copy<double, float><<<c->W0.nb, TPB, 0, s>>>(c->W0, c->r.p, c->fp.p);
        const double *sink = c->sc.p + S_SINKP;
        if (!first_phase) {
            vcycle<float>(*c, c->fp.p, c->fph.p, c->ft.p, sink, s);
            k_copy<float, double><<<c->W0.nb, TPB, 0, s>>>(c->W0, c->fph.p, c->t.p);
        } else {
            k_fill<double><<<c->W0.nb, TPB, 0, s>>>(c->W0, c->t.p, 0.0);
            if (c->walk) {
                (void)walk_down<float>(*c, c->fp.p, c->ft.p, c->frsp.p, c->fph.p, sink, s);
                const int nu = c->near.nb();
                if (nu) k_near_merge<float><<<nu, NU_T, 0, s>>>(c->L0(), c->near, c->ft.p, c->frsp.p);
                const Walk Wb = make_walk(c->L0().Nh);
                k_copy<float, double><<<Wb.nb, TPB, 0, s>>>(Wb, c->frsp.p, c->t.p + c->L0().Nh);
            } else {
                if (c->flat)
                    rows_out<float>(*c, c->fph.p, c->fp.p,
                                    half_sweeps<float, false>(*c, c->fph.p, c->fp.p, sink, 2 * c->opts.nu1, true, s),
                                    (float *)nullptr, s);
                else
                    for (int it = 0; it < c->opts.nu1; ++it) fine_smooth<float>(*c, c->fph.p, c->fp.p, sink, it == 0, s);
                k_copy<float, double><<<c->W0.nb, TPB, 0, s>>>(c->W0, c->fph.p, c->t.p);
            }
        }
        from_split<OUT_PLAIN>(*c, c->t.p, x_dev, c->nm, s);
        IBM_LAUNCH_CHECK();
    });
}

extern "C" int32_t poisson_kernel_timing(poisson_ctx *c, int32_t kernel, int32_t reset, double *total_ms,
                                         int64_t *launches)
{
    return guarded([&] {
        IBM_REQUIRE(c, IBM_EINVAL, "null context");
        IBM_REQUIRE(kernel >= -1 && kernel <= PK_WALK_UP, IBM_EINVAL, "unknown kernel id");
        if (total_ms) *total_ms = c->prof_ms;
        if (launches) *launches = c->prof_count;
        if (reset) { c->prof_ms = 0.0; c->prof_count = 0; c->prof_used = 0; }
        c->prof_kernel = kernel;
    });
}

extern "C" int32_t poisson_level_info(poisson_ctx *c, int32_t *levels, int64_t *n_unknowns, int64_t *n_ghost,
                                      int64_t *n_mghost)
{
    return guarded([&] {
        IBM_REQUIRE(c, IBM_EINVAL, "null context");
        if (levels) *levels = (int32_t)c->lv.size();
        if (n_unknowns) *n_unknowns = c->N + c->nm;
        if (n_ghost) *n_ghost = c->ng;
        if (n_mghost) *n_mghost = c->nm;
    });
}

namespace ibm {
namespace {
// the context's large per-call scratch (Krylov vectors, level iterates and
// right-hand sides): every buffer currently held, in a fixed order
template <class F>
void for_scratch(poisson_ctx &c, F &&f)
{
    DBuf<double> *d[] = {&c.x, &c.r, &c.b, &c.t, &c.rh, &c.p, &c.v, &c.ph, &c.sh, &c.rsp, &c.d64, &c.r2};
    for (auto *q : d) f(*q);
    DBuf<float> *fl[] = {&c.fr, &c.frh, &c.fp, &c.fv, &c.fph, &c.fsh, &c.ft, &c.frsp};
    for (auto *q : fl) f(*q);
    for (size_t l = 1; l < c.lv.size(); ++l) {
        f(c.lv[l].x64);
        f(c.lv[l].b64);
        f(c.lv[l].x32);
        f(c.lv[l].b16);
        f(c.lv[l].k64);
        f(c.lv[l].k32);
    }
}
constexpr size_t WS_ALIGN = 256;
size_t ws_round(size_t b) { return (b + WS_ALIGN - 1) / WS_ALIGN * WS_ALIGN; }
}  // namespace
}  // namespace ibm

extern "C" int32_t poisson_workspace_size(poisson_ctx *c, size_t *bytes)
{
    return guarded([&] {
        IBM_REQUIRE(c && bytes, IBM_EINVAL, "null argument");
        size_t total = 0;
        for_scratch(*c, [&](auto &b) { total += ws_round(b.bytes()); });
        *bytes = total;
    });
}

extern "C" int32_t poisson_bind_workspace(poisson_ctx *c, void *ws_dev, size_t bytes)
{
    return guarded([&] {
        IBM_REQUIRE(c && ws_dev, IBM_EINVAL, "null argument");
        IBM_REQUIRE(((uintptr_t)ws_dev % WS_ALIGN) == 0, IBM_EINVAL, "workspace must be 256-byte aligned");
        size_t need = 0;
        for_scratch(*c, [&](auto &b) { need += ws_round(b.bytes()); });
        IBM_REQUIRE(bytes >= need, IBM_ENOMEM, "workspace too small: " + std::to_string(bytes) + " < " +
                                                   std::to_string(need));
        IBM_HIP(hipStreamSynchronize(c->cs));
        // captured iterations hold the old addresses
        c->drop_graphs();
        char *base = (char *)ws_dev;
        size_t off = 0;
        for_scratch(*c, [&](auto &b) {
            if (!b.n) return;
            const size_t n = b.n, sz = ws_round(b.bytes());
            typedef typename std::remove_reference<decltype(*b.p)>::type E;
            b.view(reinterpret_cast<E *>(base + off), n);
            off += sz;
        });
    });
}

extern "C" void poisson_destroy(poisson_ctx *c)
{
    if (c) {
        (void)hipStreamSynchronize(c->cs);
        delete c;
    }
}
