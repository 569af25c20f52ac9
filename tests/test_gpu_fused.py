"""Fused kernels against the FP64 oracle at the sizes where they can go wrong
(edges of bricks and tiles, remainders, the ends of the option ranges)."""
import numpy as np
import pytest

import oracle
from paper_2605_04335_amd import workloads as W

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def box_case(nx, ny, nz, bodies, stretched=False):
    n = (nx, ny, nz)
    L = [m / max(n) for m in n]
    f = [W.stretched_faces(m, 1.05, e)[0] if stretched else W.uniform_faces(m, e) for m, e in zip(n, L)]
    s, c = min(L), [0.5 * e for e in L]
    out = []
    if "sphere" in bodies:
        out.append(W.sphere((c[0] - 0.2 * s, c[1], c[2]), 0.2 * s, freq=6))
    if "plate" in bodies:
        out.append(W.plate((c[0] + 0.15 * s, c[1], c[2]), 0.2 * s, 0.5 * s, 12, 30, 0.05 * s, 0.4))
    return f, out


# coarse levels smoothed on bricks: levels smaller than a brick, of one and a
# half bricks, odd in every direction (the coarsest level of a ragged box, all
# its sweeps on bricks), with masked cells and closed faces; every count of
# smoothing steps that takes the fused launches and one (3) that does not.
# The V-cycle is a fixed linear map whose global sums are reduced in another
# order than the oracle's: the bound of the V-cycle's parity test, 1e-11.
@pytest.mark.parametrize("shape,bodies,nu1,nu2,ncs", [
    ((24, 40, 56), "sphere plate", 2, 2, 32),
    ((24, 40, 56), "sphere plate", 1, 2, 32),
    ((24, 40, 56), "sphere plate", 2, 1, 33),
    ((24, 40, 56), "sphere", 3, 1, 32),
    ((50, 42, 30), "sphere", 2, 2, 32),
    ((50, 42, 62), "sphere plate", 1, 1, 31),
    ((82, 34, 26), "", 2, 2, 1),
    ((82, 34, 26), "plate", 2, 2, 2),
    ((128, 32, 16), "sphere", 2, 2, 32),
])
def test_vcycle_on_bricks_matches_oracle(shape, bodies, nu1, nu2, ncs):
    import torch
    import paper_2605_04335_amd as P
    print("[case] bricks", shape, bodies, nu1, nu2, ncs, flush=True)
    f, bl = box_case(*shape, bodies, stretched=shape[0] == 24)
    O = oracle.setup(*f, bl)
    flags, st, sol, _ = P.setup(*f, bl, nu1=nu1, nu2=nu2, coarse_sweeps=ncs)
    b = oracle.assemble_rhs(*f, O.flags, O.st, W.noise_rhs(len(O.flags), 41))
    z = sol.precond(torch.from_numpy(b).cuda()).cpu().numpy()
    assert rel(z, oracle.vcycle(*f, O.flags, O.st, b, nu1, nu2, ncs)) < 1e-11


# level 0 smoothed by the fused pass: tiles cut in every direction, a level
# narrower than a tile, no body at all (no near unit), bodies at the walls and
# through them, a membrane.  Compared modulo a constant: the shift to a zero
# pin value carries the rounding of the sink's sum over all cells (the oracle
# adds 2 million terms one after the other), which the pinned cycle does not
# resolve; the one-sweep kernels are as far from the oracle by that constant.
# The bound is the V-cycle's parity test's.
WALK = [
    ((128, 128, 128), "sphere plate"),
    ((160, 116, 116), "plate"),
    ((96, 152, 148), "sphere"),
    ((32, 264, 260), ""),
    ((264, 92, 90), "wall"),
]


def walk_case(shape, bodies):
    f, bl = box_case(*shape, bodies)
    if "wall" in bodies:
        L = [m / max(shape) for m in shape]
        bl = [W.sphere((0.02, 0.5 * L[1], 0.4 * L[2]), 0.1, freq=6), W.plate((0.5, 0.5 * L[1], 0.5 * L[2]), 0.2, 0.6, 30, 90)]
    return f, bl


@pytest.mark.parametrize("shape,bodies", WALK)
def test_fused_pass_matches_oracle(shape, bodies):
    import torch
    import paper_2605_04335_amd as P
    print("[case] walk", shape, bodies, flush=True)
    f, bl = walk_case(shape, bodies)
    O = oracle.setup(*f, bl)
    flags, st, sol, _ = P.setup(*f, bl)
    b = oracle.assemble_rhs(*f, O.flags, O.st, W.noise_rhs(len(O.flags), 43))
    bt = torch.from_numpy(b).cuda()
    z = sol.precond(bt)
    zo = oracle.vcycle(*f, O.flags, O.st, b)
    act = zo != 0.0
    d = z.cpu().numpy() - zo
    assert np.all(d[~act] == 0.0)  # the pin and inactive cells
    assert np.linalg.norm(d[act] - d[act].mean()) < 1e-11 * np.linalg.norm(zo)
    assert torch.equal(z, sol.precond(bt))


# thin boxes: a coarse level of more bricks than they pay for (one-sweep
# kernels), and as many on a level too narrow for those (bricks).  The same.
@pytest.mark.parametrize("shape", [(440, 440, 10), (300, 6, 312), (600, 6, 600), (6, 600, 600)])
def test_thin_boxes_match_oracle(shape):
    import torch
    import paper_2605_04335_amd as P
    print("[case] thin", shape, flush=True)
    f, _ = box_case(*shape, "")
    O = oracle.setup(*f, [])
    flags, st, sol, _ = P.setup(*f, [])
    b = oracle.assemble_rhs(*f, O.flags, O.st, W.noise_rhs(len(O.flags), 50))
    z = sol.precond(torch.from_numpy(b).cuda()).cpu().numpy()
    zo = oracle.vcycle(*f, O.flags, O.st, b)
    d = (z - zo)[zo != 0.0]
    assert np.linalg.norm(d - d.mean()) < 1e-11 * np.linalg.norm(zo)


# a box of more than 2^16 rows, or pairs of cells to a row, beyond the places a
# pass can hold.  The same bound and comparison; the sink's sum is of the same
# size as above.
@pytest.mark.parametrize("shape", [(6, 65540, 6), (131080, 6, 6)])
def test_longest_boxes_match_oracle(shape):
    import torch
    import paper_2605_04335_amd as P
    print("[case] long", shape, flush=True)
    f = [W.uniform_faces(m, m / 64.0) for m in shape]
    O = oracle.setup(*f, [])
    flags, st, sol, _ = P.setup(*f, [])
    b = oracle.assemble_rhs(*f, O.flags, O.st, W.noise_rhs(len(O.flags), 47))
    z = sol.precond(torch.from_numpy(b).cuda()).cpu().numpy()
    zo = oracle.vcycle(*f, O.flags, O.st, b)
    act = zo != 0.0
    d = (z - zo)[act]
    assert np.linalg.norm(d - d.mean()) < 1e-11 * np.linalg.norm(zo)


def test_update_across_the_row_limit_equals_fresh_setup():
    """A context below the pass's size takes the half-sweeps with their rows or
    the one-sweep kernels by the count of rows: an update to more rows than the
    limit, and back, preconditions bit for bit as a fresh context, and as the
    oracle (the V-cycle's parity bound)."""
    import torch
    import paper_2605_04335_amd as P
    shape = (124, 120, 116)
    f, small = box_case(*shape, "sphere")
    L = [m / max(shape) for m in shape]
    big = [W.sphere((L[0] * (i + 0.5) / 3, L[1] * (j + 0.5) / 3, L[2] * (k + 0.5) / 3), 0.125, freq=6)
           for i in range(3) for j in range(3) for k in range(3)]
    _, _, sol, _ = P.setup(*f, small)
    for bodies in (big, small):
        flags, st, fresh, _ = P.setup(*f, bodies)
        assert (sum(st.info()[:2]) > 45000) == (bodies is big)
        sol.update(flags, st)
        O = oracle.setup(*f, bodies)
        b = oracle.assemble_rhs(*f, O.flags, O.st, W.noise_rhs(len(O.flags), 48))
        x = torch.from_numpy(b).cuda()
        z = sol.precond(x)
        assert torch.equal(z, fresh.precond(x))
        zo = oracle.vcycle(*f, O.flags, O.st, b)
        d = (z.cpu().numpy() - zo)[zo != 0.0]
        assert np.linalg.norm(d - d.mean()) < 1e-11 * np.linalg.norm(zo)


def test_fused_pass_after_update_equals_fresh_setup():
    """The near units follow the bodies: a context updated to another geometry
    (and back to none) preconditions bit for bit as a fresh one."""
    import torch
    import paper_2605_04335_amd as P
    f, a = walk_case((128, 128, 128), "sphere plate")
    _, b = walk_case((128, 128, 128), "plate")
    _, _, sol, _ = P.setup(*f, a)
    for bodies in (b, [], a):
        flags, st, fresh, _ = P.setup(*f, bodies)
        sol.update(flags, st)
        x = torch.from_numpy(W.noise_rhs(fresh.n_unknowns, 44)).cuda()
        assert torch.equal(sol.precond(x), fresh.precond(x))


# half-sweeps with the sparse rows in the same launch: closed ghosts, membranes
# and both, next to each other and at the walls, odd edges (padding slots),
# one to three steps before and none to three after the coarse correction, a
# box of a single block of cells, no rows at all; and a box with enough rows
# for the one-sweep row kernels beside the fused pass.  The same bound and the
# same comparison modulo a constant.
@pytest.mark.parametrize("shape,bodies,nu1,nu2", [
    ((8, 6, 4), "", 2, 2),
    ((16, 16, 16), "plate", 1, 1),
    ((25, 31, 27), "sphere plate", 2, 2),
    ((40, 34, 38), "touching", 2, 2),
    ((40, 34, 38), "touching", 3, 1),
    ((36, 28, 46), "wall", 1, 3),
    ((36, 28, 46), "wall", 2, 0),
    ((176, 160, 152), "large", 2, 2),
])
def test_fused_rows_match_oracle(shape, bodies, nu1, nu2):
    import torch
    import paper_2605_04335_amd as P
    print("[case] rows", shape, bodies, nu1, nu2, flush=True)
    f, bl = walk_case(shape, bodies)
    L = [m / max(shape) for m in shape]
    c, s = [0.5 * e for e in L], min(L)
    if "touching" in bodies:  # the membrane's edge one cell from the sphere
        bl = [W.sphere((c[0], c[1], c[2]), 0.2 * s, freq=6),
              W.plate((c[0], c[1], c[2] + 0.2 * s + 1.5 / max(shape)), 0.3 * s, 0.5 * s, 12, 30)]
    if "large" in bodies:
        bl = [W.sphere((c[0], c[1], c[2]), 0.4 * s, freq=12)]
    O = oracle.setup(*f, bl)
    flags, st, sol, _ = P.setup(*f, bl, nu1=nu1, nu2=nu2)
    assert bodies != "large" or O.st.ng + O.st.nm > 1 << 15
    b = oracle.assemble_rhs(*f, O.flags, O.st, W.noise_rhs(len(O.flags), 45))
    bt = torch.from_numpy(b).cuda()
    z = sol.precond(bt)
    zo = oracle.vcycle(*f, O.flags, O.st, b, nu1, nu2, 32)
    act = zo != 0.0
    d = z.cpu().numpy() - zo
    assert np.linalg.norm(d[act] - d[act].mean()) < 1e-11 * np.linalg.norm(zo)
    assert torch.equal(z, sol.precond(bt))


# the coarse tail: a first level of one and of two cell pairs per thread, a
# coarsest level swept by one wavefront, by the block, and alone in the tail,
# odd edges, closed faces and masked cells, no post-smoothing.  The bound of
# the V-cycle's parity test.
@pytest.mark.parametrize("shape,bodies,nu1,nu2,ncs", [
    ((32, 32, 32), "sphere plate", 2, 2, 32),
    ((32, 32, 32), "", 3, 0, 5),
    ((32, 24, 28), "plate", 1, 1, 32),
    ((10, 10, 10), "sphere", 2, 2, 32),
    ((30, 26, 22), "sphere", 2, 2, 9),
    ((64, 20, 36), "sphere plate", 2, 3, 32),
    ((4, 4, 4), "", 2, 2, 1),
])
def test_coarse_tail_matches_oracle(shape, bodies, nu1, nu2, ncs):
    import torch
    import paper_2605_04335_amd as P
    print("[case] tail", shape, bodies, nu1, nu2, ncs, flush=True)
    f, bl = box_case(*shape, bodies, stretched=True)
    O = oracle.setup(*f, bl)
    flags, st, sol, _ = P.setup(*f, bl, nu1=nu1, nu2=nu2, coarse_sweeps=ncs)
    b = oracle.assemble_rhs(*f, O.flags, O.st, W.noise_rhs(len(O.flags), 46))
    bt = torch.from_numpy(b).cuda()
    z = sol.precond(bt)
    assert rel(z.cpu().numpy(), oracle.vcycle(*f, O.flags, O.st, b, nu1, nu2, ncs)) < 1e-11
    assert torch.equal(z, sol.precond(bt))


# the kernels that a program times per launch: half-sweeps on every grid, also
# where passes take their place in untimed solves; the pass only there
@pytest.mark.parametrize("shape,passes", [((64, 48, 40), False), ((128, 128, 128), True)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_kernel_timing_counts_launches(shape, passes, precision):
    import torch
    import paper_2605_04335_amd as P
    f, bl = box_case(*shape, "plate")
    flags, st, sol, _ = P.setup(*f, bl, precision=precision, tol=1e-9)
    rhs = torch.from_numpy(W.noise_rhs(len(flags), 49)).cuda()
    x, _ = sol.solve(rhs)
    counts = []
    for kernel in (P.KERNEL_SWEEP0, P.KERNEL_APPLY0, P.KERNEL_XR, P.KERNEL_WALK_UP):
        sol.kernel_timing(kernel)
        y, stats = sol.solve(rhs)
        ms, n = sol.kernel_timing(-1)
        counts.append(n)
        assert (ms > 0.0) == (n > 0)
        assert float((x - y).norm() / x.norm()) < 1e-6  # a solve to the same tolerance
    # per iteration two V-cycles of two phases, two steps of two half-sweeps each; what starts from zero is not
    # timed: the first half-sweep (with its rows), or the first step (one-sweep kernels)
    per = 12 if passes else 14
    its = stats.iterations
    assert counts[1] == counts[2] == its and counts[3] == (2 * its if passes else 0)
    assert counts[0] % per == 0 and abs(counts[0] // per - its) <= 2
