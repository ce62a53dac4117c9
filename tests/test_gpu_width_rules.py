"""The cell launches on grids where the rules by size choose other forms than on the small ones, and the
paper's pair inside MINRES.

 * Paper's pair above 256^2 cells: the 64-wide first smoothing without the restriction, the restriction with
   two rows of cells per wavefront and the 64-wide post-smoothing (tiles of 62 x 6, 30 x 6 coarse and 60 x 4
   cells), on ragged last tiles (288) and one cell past a tile (480).  The preconditioner
   M = diag(V, S~^{-1}) has to be linear and symmetric.  V has 6 levels of at most 8 products, each within
   about 30 roundings of |D^{-1} A| <= 4: 6e-13 in FP64.
 * Paper's pair, the A11 rows and updates of an inner step: MINRES run here in NumPy, with A11 the
   assembled operator (apply_operator) and M as above (its factor leaves the iterates as they are), gives
   the iterate of three inner steps.  A rounding grows by the norms lost from one Lanczos vector to the next
   (1e4 at 8^2 in one step): 1e-9 of the largest entry in FP64, 2e-3 in FP32, where M rounds at
   1e-7.  A wrong number of A_f, B or B^T changes its rows by 1/100 or more.  480^2 has more parts of
   beta^2 than the A11 launch sums itself.
 * Triangle batches of more than 65,536 cells on grids of 129 to 256 cells: the 64-wide restriction with one
   row of cells per wavefront (160, 192) and with two (256), bit for bit the systems alone, whose first launch
   restricts."""
import numpy as np
import pytest

from paper_2301_10041_amd import fsi

from gpu_helpers import soa, to_dev, to_host, torch_dev
from test_gpu_batch import alone, batch, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch_dev()
    fsi.lib()


class Fluid:
    """A11 and the preconditioner of a Q2 context on [u | p], as NumPy functions."""

    def __init__(self, n, prec):
        from paper_2301_10041_amd import inputs
        xy, quad = inputs.quad_bar(4, 2, 0.3, 0.7, 0.4, 0.6)
        self.ctx, self.prec = fsi.Context(n, xy, quad, pair=fsi.PAIR_Q2P1DISC), prec
        self.ctx.assemble_coupling(to_dev(soa(xy)))
        self.nf, self.pin = self.ctx.sizes["off_Xx"], self.ctx.sizes["off_p"]
        self.r0 = None

    def _full(self, v):
        x = np.zeros(self.ctx.sizes["N"])
        x[: self.nf] = v
        return to_dev(x)

    def _precond(self, v):
        torch = torch_dev()
        z = torch.zeros(self.ctx.sizes["N"], dtype=torch.float64, device="cuda")
        self.ctx.apply_precond(self._full(v), z, fsi.PC_DIAG, self.prec)
        return to_host(z)[: self.nf]

    def A(self, v):
        torch = torch_dev()
        y = torch.zeros(self.ctx.sizes["N"], dtype=torch.float64, device="cuda")
        self.ctx.apply_operator(self._full(v), y)
        return to_host(y)[: self.nf]

    def M(self, v):
        """M v, scaled so that M r0 is one step's iterate; self.lin: how far from linear."""
        if self.r0 is None:
            self.r0 = np.random.default_rng(99).uniform(-1, 1, self.nf)
            self.x0 = self.inner(self.r0, 1)
        a = np.linalg.norm(self.r0) / np.linalg.norm(v)
        x1, x3 = self.inner(a * v, 1), self.inner(a * v + self.r0, 1)
        c, *_ = np.linalg.lstsq(np.stack([x1, self.x0], 1), x3, rcond=None)
        self.lin = np.linalg.norm(c[0] * x1 + c[1] * self.x0 - x3) / np.linalg.norm(x3)
        return c[0] / c[1] / a * x1

    def inner(self, v, steps):
        self.ctx.set_inner(1e-30, steps)
        return self._precond(v)


def minres(A, M, b, steps):
    """`steps` steps of preconditioned MINRES from 0 (Paige and Saunders 1975)."""
    r1, r2, y = np.zeros_like(b), b, M(b)
    beta = phibar = np.sqrt(b @ y)
    oldb = dbar = eps = sn = 0.0
    cs = -1.0
    w1 = w2 = x = np.zeros_like(b)
    for k in range(steps):
        v = y / beta
        y = A(v)
        if k:
            y = y - beta / oldb * r1
        alfa = v @ y
        y = y - alfa / beta * r2
        r1, r2, y = r2, y, M(y)
        oldb, beta = beta, np.sqrt(r2 @ y)
        delta, gbar = cs * dbar + sn * alfa, sn * dbar - cs * alfa
        eps, oldeps, dbar = sn * beta, eps, -cs * beta
        gamma = np.hypot(gbar, beta)
        cs, sn = gbar / gamma, beta / gamma
        phi, phibar = cs * phibar, sn * phibar
        w1, w2 = w2, (v - oldeps * w1 - delta * w2) / gamma
        x = x + phi * w2
    return x


@pytest.mark.parametrize("prec,tol", [(fsi.FP64, 1e-12), (fsi.FP32, 1e-4)])
@pytest.mark.parametrize("n", [288, 480])
def test_q2_cycle_above_256(n, prec, tol):
    print(f"[Q2 cycle n={n} prec={prec}]", flush=True)
    f = Fluid(n, prec)
    rng = np.random.default_rng(n)
    r1, r2 = rng.uniform(-1, 1, f.nf), rng.uniform(-1, 1, f.nf)
    m1, lin1 = f.M(r1), f.lin
    m2, lin2 = f.M(r2), f.lin
    f.ctx.close()
    sym = abs(r1 @ m2 - r2 @ m1) / (np.linalg.norm(r1) * np.linalg.norm(m2))
    print(f"  linearity {lin1:.1e} {lin2:.1e}, symmetry {sym:.1e}", flush=True)
    assert lin1 <= tol and lin2 <= tol and sym <= tol
    assert r1 @ m1 > 0 and r2 @ m2 > 0


@pytest.mark.parametrize("prec,tol", [(fsi.FP64, 1e-9), (fsi.FP32, 2e-3)])
@pytest.mark.parametrize("n", [24, 40, 128, 160, 288, 480])
def test_q2_inner_steps(n, prec, tol):
    print(f"[Q2 inner steps n={n} prec={prec}]", flush=True)
    f = Fluid(n, prec)
    b = np.random.default_rng(3 + n).uniform(-1, 1, f.nf)
    want, got = minres(f.A, f.M, b, 3), f.inner(b, 3)
    f.ctx.close()
    for name, s in (("u", slice(0, f.pin)), ("p", slice(f.pin, f.nf))):
        d = np.abs(got[s] - want[s]).max() / np.abs(want[s]).max()
        print(f"  {name}: {d:.1e}", flush=True)
        assert d <= tol


@pytest.mark.parametrize("n, K", [(160, 3), (192, 2), (256, 2)])
@pytest.mark.parametrize("prec", [fsi.FP64, fsi.FP32])
def test_batch_with_wide_restrictions(n, K, prec):
    assert K * n * n > 256 * 256
    print(f"[wide restriction n={n} K={K} prec={prec}]", flush=True)
    opts = fsi.Opts(prec=prec, pc=fsi.PC_TRI, rtol=1e-8)
    wls = workloads(n, K, seed=31)
    ctxs = [fsi.Context.from_workload(wl) for wl in wls]
    states, stats, rcs = batch(ctxs, wls, opts)
    assert rcs == [fsi.FSI_OK] * K
    for k in (0, K - 1):
        a, sa = alone(wls[k], opts, False)
        assert np.array_equal(states[k], a) and stats[k]["inner_its"] == sa["inner_its"], k
    for c in ctxs:
        c.close()
