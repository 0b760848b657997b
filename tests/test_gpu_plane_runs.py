"""The stage kernel with a block's planes cut into 1, 2 or 4 runs (few tiles
for the resident workgroups, or a last round nearly empty): two CFL steps in
one call, so that the second one's time step comes from the runs' maxima,
against the oracle.  Tolerances as for one step: FP64 1e-12 of the largest
value, FP32 1e-5, twice that for two steps."""
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


@pytest.mark.parametrize("bs,blocks,terms,dtype,schedule", [
    (16, 8, {}, wacm.F64, {}),
    (16, 300, {**PLATE, **SPONGE}, wacm.F64, dict(wg_per_cu=1)),
    (16, 300, SPHERE, wacm.F32, dict(wg_per_cu=1, xcd_map=2)),
    (16, 520, {}, wacm.F64, dict(wg_per_cu=1)),
    (24, 8, PLATE, wacm.F32, {}),
    (24, 100, SPONGE, wacm.F64, dict(tile_rows=8, wg_per_cu=1)),
    (24, 71, SPHERE, wacm.F64, dict(tile_rows=8, xcd_map=2)),
    (32, 30, {**PLATE, "clip": 1}, wacm.F64, {}),
    (32, 30, {}, wacm.F32, dict(tile_rows=8)),
])
def test_two_steps_match_the_oracle(orc, bs, blocks, terms, dtype, schedule):
    jmax = 1 if blocks == 8 else 4
    lev, ix, iy, iz = inputs.random_balanced_leaves(5 + bs, 1, jmax, blocks)
    log(f"plane runs bs {bs} blocks {len(lev)} {schedule}")
    og = orc.Grid(bs, 4, 1.0, 1, jmax, lev, ix, iy, iz)
    codes = [wacm.treecode_encode(*q) for q in zip(lev, ix, iy, iz)]
    gg = wacm.Grid(bs, 4, 1.0, 1, jmax, codes, lev, dtype)
    gg.set_schedule(**schedule)
    prm = cases.params(nu=1e-3, c0=5.0, c_gamma=1.0, **terms)
    U = inputs.pack(inputs.fourier_fields(9, bs, 1.0, lev, ix, iy, iz, kmax=3), bs, 4)
    if dtype == wacm.F32:
        U = U.astype(np.float32).astype(float)
    pool, work = to_pool(gg, U), gg.work()
    t = torch.zeros(1, dtype=torch.float64, device="cuda")
    dt = torch.zeros(1, dtype=torch.float64, device="cuda")
    gg.rk4_steps(prm, t, dt, pool, work, 2)
    t_o = 0.0
    for _ in range(2):
        dt_o = og.dt(prm, U)
        og.rk4_step(prm, t_o, dt_o, U)
        t_o += dt_o
    i = slice(4, 4 + bs)
    a, b = from_pool(pool, np.arange(og.nb))[..., i, i, i], U[..., i, i, i]
    err = np.max(np.abs(a - b)) / np.max(np.abs(b))
    tol = 2e-12 if dtype == wacm.F64 else 2e-5
    log(f"  rel {err:.2e} t {t.item():.6e} vs {t_o:.6e}")
    assert err < tol and abs(t.item() - t_o) < tol * t_o
