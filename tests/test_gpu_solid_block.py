"""The closed form of A22 in its forms: one block per system and component with the rows in registers
(1, 2 and 3 rows per thread: 127, 1,261 and 2,977 solid nodes), with the rows read again in every
step (several systems of 3,367 and 7,057 nodes) and one launch per step (single systems from 3,367
nodes, all from 7,351).  Its result satisfies C_s z_X = -dt r_lam and C_s z_lam = A_s z_X - r_X to the
rounding level (the spectrum of D^{-1} C_s lies in [1/2, 2]), and a batch equals its systems alone,
bitwise."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_2301_10041_amd import fsi, inputs

from gpu_helpers import to_dev, to_host, torch_dev

pytestmark = pytest.mark.gpu


def _position(wl):
    xy, _ = wl.solid_mesh()
    return to_dev(np.concatenate([xy[:, 0], xy[:, 1]]))


@pytest.mark.parametrize("m", [1, 6, 20, 31, 33, 48, 49])
def test_a22_solves_its_equations(m):
    print(f"[A22 of {3 * m * m + 3 * m + 1} solid nodes]", flush=True)
    torch = torch_dev()
    wl = inputs.small_workload(16, m, (0.5, 0.5), 0.2)
    ctx = fsi.Context.from_workload(wl)
    ctx.assemble_coupling(_position(wl))
    sz, ns = ctx.sizes, ctx.sizes["Ns"]
    r = np.random.default_rng(m).uniform(-1, 1, sz["N"])
    z = torch.zeros(sz["N"], dtype=torch.float64, device="cuda")
    ctx.set_inner(1e-2, 1)
    ctx.apply_precond(to_dev(r), z, fsi.PC_DIAG, fsi.FP64)
    z = to_host(z)
    rp, col, cs = ctx.export_csr("CS")
    Cs = sp.csr_matrix((cs[:, 0], col, rp), shape=(ns, ns))
    As = sp.csr_matrix((ctx.export_csr("AS")[2][:, 0], col, rp), shape=(ns, ns))
    for c in ("x", "y"):
        X, lam = (slice(sz[f"off_{k}{c}"], sz[f"off_{k}{c}"] + ns) for k in ("X", "l"))
        d = Cs @ z[X] + wl.dt * r[lam]
        assert np.linalg.norm(d) <= 1e-13 * wl.dt * np.linalg.norm(r[lam])
        q = As @ z[X]
        d = Cs @ z[lam] - (q - r[X])
        assert np.linalg.norm(d) <= 1e-13 * (np.linalg.norm(q) + np.linalg.norm(r[X]))
    ctx.close()


@pytest.mark.parametrize("ms", [(6, 31), (33, 20), (48, 33), (49, 6)])
def test_a22_batch_equals_alone(ms):
    print(f"[A22 batch of {ms}]", flush=True)
    torch = torch_dev()
    wls = [inputs.small_workload(16, m, (0.5, 0.5), 0.25) for m in ms]
    opts = fsi.Opts(rtol=1e-8, maxit=4)   # a few outer steps: convergence is not the point
    ctxs = [fsi.Context.from_workload(wl) for wl in wls]
    us = [to_dev(np.random.default_rng(k).uniform(-1, 1, 2 * c.sizes["N2"])) for k, c in enumerate(ctxs)]
    Xs = [_position(wl) for wl in wls]
    alone = []
    for c, u, X in zip(ctxs, us, Xs):
        out = torch.zeros(c.sizes["N"], dtype=torch.float64, device="cuda")
        try:
            c.step(u, X, out, opts)
        except fsi.FsiError as e:
            assert e.code == fsi.FSI_E_NOCONV
        alone.append(to_host(out))
    outs = [torch.zeros(c.sizes["N"], dtype=torch.float64, device="cuda") for c in ctxs]
    fsi.step_batch(ctxs, us, Xs, outs, opts)
    for a, b in zip(alone, outs):
        assert np.array_equal(a, to_host(b))
    for c in ctxs:
        c.close()
