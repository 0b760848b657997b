"""Rounding of the FP64 and FP32 right-hand side where viscosity dominates: the
Laplacian is a sum of large terms that nearly cancel, so an order of its terms
with larger partial sums is further off.  The measure is the same stencils in
numpy in the element type, one axis after the other and every product rounded:
the kernel, which fuses its products, may not be further from the extended
precision value (root mean square) than that."""
import numpy as np
import pytest

from paper_1912_05371_amd import cases, inputs, wacm

from gpu_util import log, to_pool

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TW = ("0.77088238051821737976", "-0.16670590441457390381", "0.020843142770310142619")


def _rhs(U, h, nu, c0, cg, ng, T):
    """rhs of padded blocks U (nb, 4, P, P, P) in element type T."""
    U = U.astype(T)
    bs = U.shape[2] - 2 * ng
    a = [T(np.longdouble(q)) for q in TW]
    d2 = [T(T(-5) / T(2)), T(T(4) / T(3)), T(T(-1) / T(12))]
    ih, ih2 = (T(1) / h.astype(T)).reshape(-1, 1, 1, 1), (T(1) / (h * h).astype(T)).reshape(-1, 1, 1, 1)

    def at(c, axis, o):
        i = [slice(ng, ng + bs)] * 3
        i[2 - axis] = slice(ng + o, ng + o + bs)  # arrays are [z][y][x]
        return U[(slice(None), c) + tuple(i)]

    def first(c, d):
        return sum(a[m] * (at(c, d, m + 1) - at(c, d, -m - 1)) for m in range(3)) * ih

    def second(c, d):
        v = d2[2] * at(c, d, -2)
        for o in (-1, 0, 1, 2):
            v = v + d2[abs(o)] * at(c, d, o)
        return v

    u = [at(c, 0, 0) for c in range(4)]
    out = []
    for c in range(3):
        lap = ((second(c, 0) + second(c, 1)) + second(c, 2)) * ih2
        conv = u[0] * first(c, 0) + u[1] * first(c, 1) + u[2] * first(c, 2)
        out.append(-conv + T(nu) * lap - first(3, c))
    div = first(0, 0) + first(1, 1) + first(2, 2)
    out.append(-T(c0 * c0) * div - T(cg) * u[3])
    return np.stack(out, 1)


@pytest.mark.parametrize("bs,prec,schedule", [(16, wacm.F64, {}), (24, wacm.F64, dict(tile_rows=8)),
                                              (24, wacm.F64, dict(tile_rows=0)), (16, wacm.F32, {})])
def test_viscous_rhs_rounds_like_the_plain_order(bs, prec, schedule):
    ng, nu, c0, cg = 4, 1.0, 1.0, 1.0
    lev, ix, iy, iz = inputs.random_balanced_leaves(3, 1, 3, 30)
    codes = [wacm.treecode_encode(*q) for q in zip(lev, ix, iy, iz)]
    g = wacm.Grid(bs, ng, 1.0, 1, 3, codes, lev, prec)
    g.set_schedule(**schedule)
    log(f"rounding of the rhs bs {bs} dtype {prec} {schedule}")
    U = to_pool(g, inputs.pack(inputs.fourier_fields(4, bs, 1.0, lev, ix, iy, iz, kmax=3), bs, ng))
    g.sync_ghosts(U)
    dU = g.pool()
    g.rhs_acm(cases.params(nu=nu, c0=c0, c_gamma=cg), 0.0, U, dU)
    i = slice(ng, ng + bs)
    got = dU[:len(lev), :, i, i, i].cpu().numpy().astype(np.longdouble)
    host = U[:len(lev)].cpu().numpy()
    T = np.float64 if prec == wacm.F64 else np.float32
    h = np.longdouble(1) / (np.longdouble(bs) * (np.longdouble(2) ** np.asarray(lev)))
    exact = _rhs(host, h, nu, c0, cg, ng, np.longdouble)
    plain = _rhs(host, h, nu, c0, cg, ng, T).astype(np.longdouble)
    rms = [float(np.sqrt(np.mean(((v - exact) / np.abs(exact[:, :3]).max()) ** 2)))
           for v in (got, plain)]
    log(f"  rms error: kernel {rms[0]:.3e}, plain order {rms[1]:.3e}")
    assert rms[0] <= rms[1]


def test_step_adjoint_keeps_what_four_stages_add_together():
    """A sponge on every point takes 8e-8 of lambda = 1 per step, at most a third
    of it in one stage: less than half of lambda's last place (2^-25), so a sum
    that starts from lambda loses every stage's part.  Summed among themselves
    the stages' parts reach lambda: an error of half a last place per kernel that
    writes it (two), 2^-24 per step."""
    steps, dt = 64, 1e-6
    lev, ix, iy, iz = inputs.uniform_leaves(1)
    codes = [wacm.treecode_encode(*q) for q in zip(lev, ix, iy, iz)]
    g = wacm.Grid(16, 4, 1.0, 1, 1, codes, lev, wacm.F32)
    prm = cases.params(nu=0.0, c0=1.0, c_gamma=0.0, sponge=1, l_sp=0.6, c_sp=dt / 8e-8,
                       u_inf=(0.0, 0.0, 0.0), p_inf=0.0)
    U, lam, work = g.pool(), g.pool(), g.adj_work()
    lam.fill_(1.0)
    th = torch.zeros(3, dtype=torch.float64, device="cuda")
    for n in range(steps):
        g.rk4_step_adj(prm, n * dt, dt, U, lam, th, None, None, work)
    i = slice(4, 20)
    got = lam[:8, :, i, i, i].double()
    err = float((got - np.exp(-8e-8 * steps)).abs().max())
    log(f"lambda after {steps} steps: error {err:.2e} of {8e-8 * steps:.2e}")
    assert err <= steps * 2.0 ** -24
