"""3D mesh step and metrics at the edges of their tiles: the monitor (30 x 14
columns), filter passes (26 x 16 columns three a launch, 28 x 18 two, 30 x 20 one)
and Jacobi sweeps (28 x 12 two a launch, 30 x 14 one), over one and several z
chunks, on grids around the tile sizes and smaller than a halo, with every kind
of face, against the oracle at the FP64 parity bar."""
import numpy as np
import pytest
import torch

import oracle
from paper_2202_07989_amd import inputs as I
from gpu_util import TOL_FP64, dev, host, say

pytestmark = pytest.mark.gpu

PER, REF, OUT, INF = I.BC_PERIODIC, I.BC_REFLECT, I.BC_OUTFLOW, I.BC_INFLOW
FACES = {
    "periodic": None,
    "walls": [(REF, REF)] * 3,
    "mixed": [(PER, PER), (REF, REF), (OUT, INF)],
}
STIFF = dict(gamma=(3.0, 1.4), cv=(1.0, 1.0), pinf=(100.0, 0.0))


@pytest.mark.parametrize("faces", list(FACES))
@pytest.mark.parametrize("n", [(3, 3, 3), (28, 13, 5), (29, 12, 3), (31, 15, 17), (33, 11, 40), (5, 26, 9),
                               (27, 17, 6), (30, 20, 4), (61, 15, 7)])
@pytest.mark.parametrize("smooth,sweeps", [(0, 0), (0, 1), (1, 2), (2, 3), (3, 4), (7, 5)])
def test_mesh_step(faces, n, smooth, sweeps):
    say(f"[mesh tiles 3D] {faces} {n} smooth={smooth} sweeps={sweeps}")
    bc = FACES[faces]
    sp = I.make_spec(3, 2, n, chi=I.CHI_SHOCK, bc=bc, wall=[(0.0, 1.0)] * 3 if bc else None, **STIFF)
    if faces == "mixed":
        sp["inflow"] = {(2, 1): [1.0, 0.5, -0.3, 0.1, 0.2, 400.0]}
    rho, v, p = I.random_state(sp, 3, noise=0.2, p_range=(50.0, 200.0))
    rng = np.random.default_rng(3)
    x = [np.broadcast_to(xi, rho[0].shape) + 0.2 * sp["dxi"][k] * rng.uniform(-1, 1, size=rho[0].shape)
         for k, xi in enumerate(I.xi_nodes(sp))]    # nodes moved by up to a fifth of a spacing
    JU, J, xp = I.assemble(sp, I.conserved(sp, rho, v, p), np.ones_like(rho[0]), x)
    o = oracle.Oracle(sp)
    o.fill_ghosts_state(JU, J)
    o.fill_ghosts_x(xp)
    from paper_2202_07989_amd import es
    ctx = es.Context(sp)
    h = min(sp["dxi"])
    for mon in (dict(sigma=[0], alpha=[100.0]), dict(sigma=[5, 3], alpha=[6.0, 12.0], psi=[12.0, 2.0])):
        mon = dict(mon, n_smooth=smooth, n_sweeps=sweeps)
        rc, disp, tau, resid = o.mesh_redistribute(mon, JU, J, xp)
        assert rc == 0
        gd = torch.full_like(dev(xp), float("nan"))
        gt = torch.zeros(1, dtype=torch.float64, device="cuda")
        gr = torch.full((max(1, sweeps),), -1.0, dtype=torch.float64, device="cuda")
        for want in (gr if sweeps else None, None):
            ctx.mesh_redistribute(mon, dev(JU), dev(J), dev(xp), gd, gt, want)
            assert np.abs(host(gd) - disp).max() <= TOL_FP64 * h, (mon, np.abs(host(gd) - disp).max() / h)
            assert abs(float(host(gt)[0]) - tau) <= TOL_FP64
        if sweeps:
            assert np.abs(host(gr) - resid).max() <= TOL_FP64 * h


@pytest.mark.parametrize("faces", list(FACES))
@pytest.mark.parametrize("n", [(3, 3, 3), (26, 10, 9), (27, 11, 20), (25, 9, 40), (53, 21, 8)])
@pytest.mark.parametrize("w", [1, 2, 3])
def test_metrics(faces, n, w):
    """Columns (26 x 10 a block) and z chunks of the metrics, with and without a
    displacement and the time metrics, ghost layers included."""
    say(f"[metric tiles 3D] {faces} {n} w={w}")
    bc = FACES[faces]
    sp = I.make_spec(3, 2, n, w=w, bc=bc, wall=[(0.0, 1.0)] * 3 if bc else None, **STIFF)
    if faces == "mixed":
        sp["inflow"] = {(2, 1): [1.0, 0.5, -0.3, 0.1, 0.2, 400.0]}
    o = oracle.Oracle(sp)
    rng = np.random.default_rng(5)
    x, disp = I.zeros(sp, 3), I.zeros(sp, 3)
    Iin = I.interior(sp)
    for k, xi in enumerate(I.xi_nodes(sp)):
        x[k][Iin[1:]] = xi + 0.2 * sp["dxi"][k] * rng.uniform(-1, 1, size=xi.shape)
        disp[k][Iin[1:]] = 0.1 * sp["dxi"][k] * rng.uniform(-1, 1, size=xi.shape)
    o.fill_ghosts_x(x)
    o.fill_ghosts_kind(disp, 3, 2)
    # a product is of size dxi and carries about 4 roundings; its differences over
    # dxi^2 then carry 16 eps / dxi, on either side
    tol = 32 * np.finfo(float).eps / min(sp["dxi"])
    from paper_2202_07989_amd import es
    ctx = es.Context(sp)
    dt = torch.tensor([0.01], dtype=torch.float64, device="cuda")
    for d, cs, t in ((disp, 0.5, True), (disp, 0.0, True), (None, 0.0, True), (disp, 1.0, False)):
        jx, jt = o.metrics(x, d, c_s=cs, dt=0.01)
        gx = torch.full_like(dev(jx), float("nan"))
        gt = torch.full_like(dev(jt), float("nan"))
        ctx.es_metrics(dev(x), None if d is None else dev(d), cs, dt, gx, gt if t else None)
        assert np.abs(host(gx) - jx).max() <= tol * np.abs(jx).max(), (cs, t)
        if t:
            assert np.abs(host(gt) - jt).max() <= tol * np.abs(jx).max() * 10 * max(sp["dxi"]), cs
        else:
            assert torch.isnan(gt).all()
