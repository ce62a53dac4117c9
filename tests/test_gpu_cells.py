"""The velocity cycle's launches by cells (pre-smoothing tiles of 62 x 6 cells, post-smoothing 60 x 4,
residual and restriction 30 x 2 coarse cells and, from 256^2 on, 30 x 6) at grids where their tiles
end: one cell past a tile (60, 120), ragged last tiles (112, 160), and both sides of the rule that
gives the restriction its larger tile; and the pressure part's (descent 29 x 5 coarse nodes, ascent
60 x 12, from 512^2 on 29 x 13 and 60 x 28; the one-launch coarse end from 64^2 down, with the output
where it starts on the finest level): a grid with one level (5), a coarse end alone (6 to 64, dense
levels of 16 to 256 unknowns), one and more levels above it.  The matrix-free preconditioner equals the one on the
assembled operators (fsi_set_smoother) up to the order of the sums, in velocity and pressure each (a
few hundred roundings of a well conditioned cycle): one application in both precisions, and one
and two inner steps in FP64."""
import numpy as np
import pytest

from paper_2301_10041_amd import fsi, inputs

from gpu_helpers import rel, to_dev, to_host, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 6, 8, 24, 36, 60, 64, 112, 120, 160, 256, 320, 512])
def test_cell_launches_equal_assembled(n):
    print(f"[cell launches n={n}]", flush=True)
    torch = torch_dev()
    wl = inputs.small_workload(n, 4, (0.5, 0.5), 0.2)
    ctx = fsi.Context.from_workload(wl)
    xy, _ = wl.solid_mesh()
    ctx.assemble_coupling(to_dev(np.concatenate([xy[:, 0], xy[:, 1]])))
    r = to_dev(np.random.default_rng(71 + n).uniform(-1, 1, ctx.sizes["N"]))   # boundary rows too
    sz = ctx.sizes
    for prec, tol in ((fsi.FP64, 1e-12), (fsi.FP32, 1e-5)):
        for mode, maxit in ((fsi.INNER_FIXED_DIAG, 1), (fsi.INNER_MINRES, 1), (fsi.INNER_MINRES, 2)):
            if mode == fsi.INNER_MINRES and (n < 60 or n > 320 or prec == fsi.FP32):
                continue   # MINRES coefficients that nearly cancel magnify the rounding (1e4 times at 8^2)
            out = []
            for kind in (fsi.SMOOTH_CSR, fsi.SMOOTH_STENCIL):
                ctx.set_smoother(kind)
                ctx.set_inner_mode(mode)
                ctx.set_inner(1e-30, maxit)
                z = torch.zeros_like(r)
                ctx.apply_precond(r, z, fsi.PC_DIAG, prec)
                out.append(to_host(z))
            for name, lo, hi in (("u", 0, sz["off_p"]), ("p", sz["off_p"], sz["off_Xx"])):
                d = rel(out[1][lo:hi], out[0][lo:hi])
                print(f"  prec {prec} mode {mode} maxit {maxit} {name}: rel diff {d:.2e}", flush=True)
                assert d <= tol
    ctx.close()
