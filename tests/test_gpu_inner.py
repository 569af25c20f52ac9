"""The inner preconditioner of the mixed form (FP32 iterates, BF16 coarse
right-hand sides) by itself: refinement and the FP64 fallback of a whole solve
would hide a fault in it.  Through the library's test hook, at the edges of
bricks, tiles and units and on every route of level 0."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2605_04335_amd import workloads as W
from tests import refpy
from tests.test_gpu_fused import box_case, walk_case

pytestmark = pytest.mark.gpu


def inner(P, sol, b, first_phase=0):
    import torch
    bt = torch.from_numpy(b).cuda()
    x = torch.full_like(bt, float("nan"))
    fn = P.lib().ibm_test_inner_precond
    fn.restype = ctypes.c_int32
    rc = fn(sol.h, ctypes.c_void_p(bt.data_ptr()), ctypes.c_void_p(x.data_ptr()), ctypes.c_int32(first_phase),
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, P.lib().ibm_last_error()
    return x


def case(shape, bodies):
    f, bl = walk_case(shape, bodies)
    if "large" in bodies:
        L = [m / max(shape) for m in shape]
        bl = [W.sphere([0.5 * e for e in L], 0.4 * min(L), freq=12)]
    if "many" in bodies:  # nearly every unit near a body
        L = [m / max(shape) for m in shape]
        bl = [W.sphere((L[0] * (i + 0.5) / 4, L[1] * (j + 0.5) / 4, L[2] * (k + 0.5) / 4), 0.08 * min(L), freq=3)
              for i in range(4) for j in range(4) for k in range(4)]
    if "small" in bodies:
        L = [m / max(shape) for m in shape]
        bl = [W.sphere((0.3 * L[0], 0.5 * L[1], 0.5 * L[2]), 0.05, freq=6),
              W.plate((0.7 * L[0], 0.5 * L[1], 0.5 * L[2]), 0.1, 0.2, 12, 30, 0.02, 0.4)]
    return f, bl


# The V-cycle of the inner solves against the oracle's in FP64, by the residual
# of their difference d: what is not FP32 rounding (2^-24 of the iterate) comes
# from rounding each coarse right-hand side to BF16 (2^-9 of it, on at most
# seven levels), so A d stays within 7 * 2^-9 < 2^-5 of the largest right-hand
# side at every row; without smoothing after the interpolation, whose own
# second differences are up to four times the coarse operator's, within 2^-3.
# A row relaxed with a wrong neighbour, or not at all, is off by the right-hand
# side itself.
# The right-hand side has no net flux, so that the pin's sink (which would
# outgrow every other row) is zero to rounding.
@pytest.mark.parametrize("shape,bodies,nu1,nu2", [
    ((24, 40, 56), "sphere plate", 2, 2),      # bricks, tail, rows in the half-sweeps
    ((50, 42, 62), "sphere plate", 1, 1),      # an odd coarsest level on bricks
    ((40, 34, 38), "wall", 3, 1),
    ((32, 32, 32), "sphere plate", 2, 2),      # two cell pairs per thread in the tail
    ((124, 120, 116), "many", 2, 2),           # more rows than the recomputing half-sweeps take
    ((128, 128, 128), "sphere plate", 2, 2),   # a fifth of the units near a body: one-sweep kernels
    ((96, 152, 148), "sphere", 2, 2),          # the pass, few rows
    ((176, 160, 152), "large", 2, 2),          # the pass, many rows
    ((160, 116, 116), "plate", 2, 2),
    ((32, 264, 260), "", 2, 2),                # narrower than a tile, cut tiles
    ((264, 92, 90), "wall", 2, 2),
    ((128, 128, 132), "many", 2, 2),           # too many near units: one-sweep kernels
    ((128, 128, 132), "sphere plate", 1, 2),   # step counts that the pass does not take
    ((128, 128, 132), "plate", 2, 0),
    ((128, 132, 128), "sphere", 3, 3),
    ((208, 204, 200), "small", 2, 2),          # few rows, their units beside the pass
])
def test_inner_vcycle_matches_fp64_oracle(shape, bodies, nu1, nu2):
    import torch
    import paper_2605_04335_amd as P
    print("[case] inner", shape, bodies, nu1, nu2, flush=True)
    f, bl = case(shape, bodies)
    O = oracle.setup(*f, bl)
    flags, st, sol, _ = P.setup(*f, bl, nu1=nu1, nu2=nu2, precision="mixed")
    act = refpy.active_mask(O.flags, O.st.nm)
    fluid = np.zeros(len(act), bool)
    fluid[:len(O.flags)] = (O.flags & 1) == 0
    b = np.where(fluid, W.noise_rhs(len(act), 51), 0.0)
    b[fluid] -= b[fluid].mean()  # (equal volumes)
    b = b.astype(np.float32).astype(np.float64)
    z = inner(P, sol, b)
    assert torch.equal(z, inner(P, sol, b))
    z = z.cpu().numpy()
    assert np.all(z[~act] == 0.0)
    zo = oracle.vcycle(*f, O.flags, O.st, b, nu1, nu2, 32)
    pin = int(np.nonzero(O.flags & 8)[0][0])
    d = np.where(act, z - z[pin] - zo, 0.0)
    r = oracle.apply(*f, O.flags, O.st, d)
    r[pin] = 0.0
    assert np.abs(r).max() < (2.0 ** -5 if nu2 else 2.0 ** -3) * np.abs(b).max()


def smoothed(f, b, sink, steps):
    """The smoothing steps from zero in FP64 arithmetic, every half-sweep's
    values rounded to FP32: no bodies, the pin in cell 0.  b: [z, y, x]."""
    nb, dg = [], 0.0
    for ax, face in zip((2, 1, 0), f):
        w, c = np.diff(face), refpy.centres(face)
        cp, cm = np.zeros(len(w)), np.zeros(len(w))
        cp[:-1], cm[1:] = 1.0 / (w[:-1] * np.diff(c)), 1.0 / (w[1:] * np.diff(c))
        sh = [1, 1, 1]
        sh[ax] = -1
        m = b.shape[ax]
        nb.append((ax, cp[:m].reshape(sh), cm[:m].reshape(sh)))
        dg = dg + cp[:m].reshape(sh) + cm[:m].reshape(sh)
    b = b.copy()
    b[0, 0, 0] -= sink
    red = np.indices(b.shape).sum(0) % 2 == 0
    x = np.zeros_like(b)
    for q in range(2 * steps):
        s = np.zeros_like(b)
        for ax, cp, cm in nb:
            p = np.pad(x, [(1, 1) if a == ax else (0, 0) for a in range(3)])
            n = b.shape[ax]
            s += cp * np.take(p, range(2, n + 2), ax) + cm * np.take(p, range(n), ax)
        x = np.where(red == (q % 2 == 0), ((s - b) / dg).astype(np.float32).astype(np.float64), x)
    return x, red


# The steps before the coarse correction on level 0, cell by cell: FP64
# arithmetic between FP32 iterates leaves the order of six products open, so a
# value may differ where it lies within 2^-52 of a rounding boundary: one cell in
# 2^28 and half-sweep, and that cell's neighbours afterwards.  64 cells allowed.
@pytest.mark.parametrize("shape,nu1", [((128, 128, 128), 2), ((32, 264, 260), 2), ((264, 92, 90), 2), ((25, 31, 27), 2),
                                       ((64, 20, 36), 3), ((128, 128, 132), 1)])
def test_inner_smoothing_cell_by_cell(shape, nu1):
    import paper_2605_04335_amd as P
    print("[case] smoothing", shape, nu1, flush=True)
    f, _ = box_case(*shape, "")
    flags, st, sol, _ = P.setup(*f, [], nu1=nu1, precision="mixed")
    b = W.noise_rhs(shape[0] * shape[1] * shape[2], 52).astype(np.float32).astype(np.float64)
    z = inner(P, sol, b, 1).cpu().numpy().reshape(shape[::-1])
    want, red = smoothed(f, b.reshape(shape[::-1]), b.sum(), nu1)
    cells = ~red if b.size >= 1 << 21 and nu1 == 2 else np.ones_like(red)
    assert np.count_nonzero((z != want) & cells) <= 64
    assert np.abs(z - want)[cells].max() <= 2.0 ** -20 * np.abs(want).max()


# Routes of level 0 in FP64 that the fused tests leave out: few rows with their
# units beside the pass, too many near units for it, step counts that it does
# not take.  Compared modulo a constant at the V-cycle's parity bound, as there.
@pytest.mark.parametrize("shape,bodies,nu1,nu2", [
    ((208, 204, 200), "small", 2, 2),
    ((128, 128, 132), "many", 2, 2),
    ((128, 128, 132), "sphere plate", 1, 2),
    ((128, 128, 132), "plate", 2, 0),
    ((128, 132, 128), "sphere", 3, 3),
    ((124, 120, 116), "many", 2, 2),
])
def test_other_routes_of_level_0(shape, bodies, nu1, nu2):
    import torch
    import paper_2605_04335_amd as P
    print("[case] route", shape, bodies, nu1, nu2, flush=True)
    f, bl = case(shape, bodies)
    O = oracle.setup(*f, bl)
    flags, st, sol, _ = P.setup(*f, bl, nu1=nu1, nu2=nu2)
    b = oracle.assemble_rhs(*f, O.flags, O.st, W.noise_rhs(len(O.flags), 53))
    bt = torch.from_numpy(b).cuda()
    z = sol.precond(bt)
    assert torch.equal(z, sol.precond(bt))
    zo = oracle.vcycle(*f, O.flags, O.st, b, nu1, nu2, 32)
    d = (z.cpu().numpy() - zo)[zo != 0.0]
    assert np.linalg.norm(d - d.mean()) < 1e-11 * np.linalg.norm(zo)


# The pin's right-hand side less the sink is not an FP32 number and is used in
# FP64 in every half-sweep: the pin's neighbours after two steps of the fused
# pass, over draws, equal the half-sweeps' to the bit (a corner of eight cells
# per axis holds all they depend on).
def test_the_sink_stays_in_fp64():
    import paper_2605_04335_amd as P
    shape, n = (128, 128, 128), 8
    f, _ = box_case(*shape, "")
    flags, st, sol, _ = P.setup(*f, [], precision="mixed")
    off = []
    for seed in range(24):
        b = W.noise_rhs(shape[0] ** 3, 60 + seed).astype(np.float32).astype(np.float64)
        z = inner(P, sol, b, 1).cpu().numpy().reshape(shape[::-1])
        want, _ = smoothed(f, b.reshape(shape[::-1])[:n, :n, :n], b.sum(), 2)
        off += [z[k] - want[k] for k in ((0, 0, 1), (0, 1, 0), (1, 0, 0))]
    assert not np.any(off), "%d of %d values off, by up to %.1e" % (np.count_nonzero(off), len(off), np.abs(off).max())
