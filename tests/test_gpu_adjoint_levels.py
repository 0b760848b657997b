"""GPU adjoint of one RK4 step on trees whose blocks meet coarser and finer
leaves on every side, for each block size (whole blocks at 16, tiles of 8 rows
at 24 and 32), with each kind of penalization term, against the oracle's
adjoint.  Tolerances: FP64 1e-12 of the largest adjoint value (1e-10 for
theta, 1e-11 for the solid velocity, as for the plate), FP32 1e-5."""
import numpy as np
import pytest

from paper_1912_05371_amd import cases, inputs, wacm

from gpu_util import from_pool, log, to_pool

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PLATE = dict(mask=2, c_eta=1e-3, w=0.02, x_le=(0.5, 0.5, 0.5), lo=(0.0, -0.25, -0.02),
             hi=(0.2, 0.25, 0.02), amp=0.6, freq=1.0, phase=0.3)
SPHERE = dict(mask=1, c_eta=1e-3, w=0.02, sph_c=(0.45, 0.5, 0.55), sph_r=0.2)
SPONGE = dict(sponge=1, l_sp=0.2, c_sp=5e-3, u_inf=(0.3, -0.2, 0.1), p_inf=0.05)


@pytest.mark.parametrize("bs,ng,levels,blocks,terms,dtype", [
    (16, 3, (1, 4), 90, PLATE, wacm.F64),
    (16, 5, (1, 3), 60, {**SPHERE, **SPONGE}, wacm.F32),
    (16, 4, (1, 1), 8, {}, wacm.F64),          # no face next to another level
    (24, 4, (1, 3), 40, {**PLATE, **SPONGE}, wacm.F64),
    (24, 3, (1, 3), 40, PLATE, wacm.F32),
    (32, 4, (1, 3), 30, SPONGE, wacm.F64),
    (32, 3, (1, 2), 22, {**SPHERE, "clip": 1}, wacm.F32),
])
def test_step_adjoint_on_mixed_levels(orc, bs, ng, levels, blocks, terms, dtype):
    lev, ix, iy, iz = inputs.random_balanced_leaves(17 + bs, levels[0], levels[1], blocks)
    log(f"step adjoint bs {bs} ng {ng} blocks {len(lev)} levels {np.bincount(lev).tolist()}")
    og = orc.Grid(bs, ng, 1.0, levels[0], levels[1], lev, ix, iy, iz)
    codes = [wacm.treecode_encode(*q) for q in zip(lev, ix, iy, iz)]
    gg = wacm.Grid(bs, ng, 1.0, levels[0], levels[1], codes, lev, dtype)
    prm = cases.params(nu=1e-2, c0=5.0, c_gamma=1.0, **terms)
    rng = np.random.default_rng(bs)
    rnd = (lambda a: a) if dtype == wacm.F64 else (lambda a: a.astype(np.float32).astype(float))
    U = rnd(inputs.pack(inputs.fourier_fields(3, bs, 1.0, lev, ix, iy, iz, kmax=3), bs, ng))
    lam = rnd(rng.standard_normal(U.shape))
    dus = rnd(0.05 * rng.standard_normal((og.nb, 3, bs ** 3)))
    t, dt = 0.05, 0.3 / (bs << levels[1]) / 5.0
    lam_o, th_o, db_o = lam.copy(), [0.0, 0.0, 0.0], np.zeros_like(dus)
    og.rk4_step_adj(prm, t, dt, U, lam_o, th_o, db_o, dus)
    lam_g = to_pool(gg, lam)
    th = torch.zeros(3, dtype=torch.float64, device="cuda")
    db = torch.zeros((gg.capacity, 3, bs ** 3), dtype=torch.float64, device="cuda")
    d = torch.from_numpy(dus).to("cuda", gg.torch_dtype())
    work = gg.adj_work()
    gg.rk4_step_adj(prm, t, dt, to_pool(gg, U), lam_g, th, db, d, work)
    i = slice(ng, ng + bs)
    lg = from_pool(lam_g, np.arange(og.nb))[..., i, i, i]
    lo = lam_o[..., i, i, i]
    tol = (1e-12, 1e-10, 1e-11) if dtype == wacm.F64 else (1e-5, 1e-5, 1e-5)
    err = [np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-30) for a, b in
           ((lg, lo), (th.cpu().numpy(), np.array(th_o)), (db.cpu().numpy(), db_o))]
    log(f"  lambda {err[0]:.2e} theta {err[1]:.2e} dus {err[2]:.2e}")
    assert all(e < q for e, q in zip(err, tol))
    # without the solid velocity's adjoint: the same lambda and theta
    lam2, th2 = to_pool(gg, lam), torch.zeros_like(th)
    gg.rk4_step_adj(prm, t, dt, to_pool(gg, U), lam2, th2, None, d, work)
    assert torch.equal(th, th2)
    assert torch.equal(lam_g[..., i, i, i], lam2[..., i, i, i])
