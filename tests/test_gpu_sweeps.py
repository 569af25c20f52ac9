"""Two Jacobi sweeps of the advection-diffusion solve in one pass, against the
FP64 oracle at the sizes where it can go wrong."""
import numpy as np
import pytest

import oracle
from paper_2605_04335_amd import workloads as W

pytestmark = pytest.mark.gpu


# two sweeps per pass: tiles cut in every direction, narrower than a ring,
# walls in every tile, an odd count of sweeps per cycle (one of them by
# itself), bodies at and through the walls, none; the iterate starts from noise
# and the solve stops after its cycles.  Every row is evaluated in the order of
# its definition on both sides: rounding of 24 sweeps at most, 1e-13.
@pytest.mark.parametrize("shape,bodies,sweeps", [((4, 4, 4), "", 2), ((65, 9, 11), "", 3), ((64, 8, 70), "plate", 4),
                                                 ((67, 33, 130), "sphere plate", 2), ((130, 17, 6), "", 5),
                                                 ((40, 44, 36), "walls", 8), ((23, 19, 21), "sphere", 1)])
def test_ad_sweep_pairs_match_oracle(shape, bodies, sweeps):
    import torch
    import paper_2605_04335_amd as P
    print("[case] pairs", shape, bodies, sweeps, flush=True)
    L = [m / max(shape) for m in shape]
    f = [W.uniform_faces(m, e) for m, e in zip(shape, L)]
    s, c = min(L), [0.5 * e for e in L]
    bl = []
    if "sphere" in bodies:
        bl.append(W.sphere((c[0] - 0.15 * s, c[1], c[2]), 0.2 * s, freq=4))
    if "plate" in bodies:
        bl.append(W.plate((c[0] + 0.2 * s, c[1], c[2]), 0.3 * s, 0.4 * s, 8, 8, 0.02 * s, 0.3))
    if "walls" in bodies:
        bl += [W.sphere((0.05, c[1], c[2]), 0.2, freq=4), W.plate((0.6, c[1], c[2]), 0.2, 1.2 * L[1], 8, 24, 0.0, 0.4)]
    flags, _ = P.classify(*f, bl)
    st = P.build_ghost_stencils(*f, bl, flags, bc="dirichlet")
    O = oracle.stencils(*f, bl, flags.cpu().numpy(), bc="dirichlet")
    N = len(flags)
    dg = oracle.max_cell_scale(*f)
    beta = 4.0 / dg
    sol = P.AdSolver(*f, flags, st, beta, tol=1e-300, sweeps=sweeps, max_cycles=3)
    rhs, g = W.noise_rhs(N, 5), W.noise_rhs(max(O.ng + O.nm, 1), 6)
    u0 = W.noise_rhs(N + O.nm, 7)
    u = torch.from_numpy(u0.copy()).cuda()
    sol.solve(torch.from_numpy(rhs).cuda(), torch.from_numpy(g).cuda(), u, check=False)
    fl = flags.cpu().numpy()
    u0[:N][((fl & 1) != 0) & ((fl & 2) == 0)] = 0.0
    want, cyc, _, _ = oracle.ad_solve(*f, fl, O, beta, oracle.ad_rhs(*f, fl, O, rhs, g if bl else None),
                                      oracle.ad_schedule(sweeps, beta, dg), tol=1e-300, maxcyc=3, x0=u0)
    assert cyc == 3
    assert np.linalg.norm(u.cpu().numpy() - want) < 1e-13 * np.linalg.norm(want)


# the reported residual, from pairs of cells (even rows) and single ones (odd
# rows, or an iterate off 16-byte alignment), against the operator's: sums of a
# few thousand squares, 1e-12
@pytest.mark.parametrize("shape", [(4, 4, 4), (130, 9, 37), (66, 21, 18), (35, 20, 17)])
@pytest.mark.parametrize("shift", [0, 1])
def test_ad_residual_of_the_last_iterate(shape, shift):
    import torch
    import paper_2605_04335_amd as P
    print("[case] residual", shape, shift, flush=True)
    L = [m / max(shape) for m in shape]
    f = [W.uniform_faces(m, e) for m, e in zip(shape, L)]
    s, c = min(L), [0.5 * e for e in L]
    bl = [] if min(shape) < 8 else [W.sphere((c[0], c[1], c[2]), 0.25 * s, freq=4),
                                    W.plate((c[0] - 0.3, c[1], c[2]), 0.3 * s, 0.4 * s, 6, 6, 0.0, 0.3)]
    flags, _ = P.classify(*f, bl)
    st = P.build_ghost_stencils(*f, bl, flags, bc="dirichlet")
    fl = flags.cpu().numpy()
    O = oracle.stencils(*f, bl, fl, bc="dirichlet")
    beta = 4.0 / oracle.max_cell_scale(*f)
    sol = P.AdSolver(*f, flags, st, beta, tol=1e-300, sweeps=2, max_cycles=1)
    n = len(fl) + O.nm
    rhs = W.noise_rhs(len(fl), 8)
    u = torch.zeros(n + 1, dtype=torch.float64, device="cuda")[shift:shift + n]
    _, stats = sol.solve(torch.from_numpy(rhs).cuda(), None, u, check=False)
    b = oracle.ad_rhs(*f, fl, O, rhs, None)
    r = b - oracle.ad_apply(*f, fl, O, beta, u.cpu().numpy())
    assert abs(stats.rel_residual / (np.linalg.norm(r) / np.linalg.norm(b)) - 1.0) < 1e-12
