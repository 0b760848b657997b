"""Edges of the kernels that predict ghost values and of the low-pass of the
transform: box edges odd and even, two wave tiles, the smallest lattice; and
the schedule taken when none is set on a large grid."""
import numpy as np
import pytest

from paper_1912_05371_amd import cases, inputs, wacm

from gpu_util import from_pool, log, make_pair, to_pool

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DT = {"f64": wacm.F64, "f32": wacm.F32}
EPS = {"f64": np.finfo(np.float64).eps, "f32": np.finfo(np.float32).eps}


@pytest.mark.parametrize("bs,ng,prec", [(16, 5, "f64"), (16, 4, "f32"), (24, 3, "f32"),
                                        (24, 5, "f64"), (32, 3, "f64"), (32, 5, "f32")])
def test_ghost_regions_in_coarser_leaves(orc, bs, ng, prec):
    c = cases.random_octree(bs=bs, ng=ng, target=60, j0=1, jmax=3, seed=bs + ng)
    og, gg = make_pair(orc, c, DT[prec])
    U = np.random.default_rng(ng).standard_normal((og.nb, 4, c.P, c.P, c.P))
    U = U.astype(np.float32).astype(np.float64) if prec == "f32" else U
    Uo = U.copy()
    og.sync(Uo)
    pool = to_pool(gg, U, fill=float("nan"))
    gg.sync_ghosts(pool)
    Ug = from_pool(pool, np.arange(og.nb))
    # three passes of 4-term sums with weight sums 1.25 per axis: rounding
    # below 3 eps (1.25 + 1.25^2 + 1.25^3) max|u| < 16 eps max|u|
    worst = np.max(np.abs(Ug - Uo))
    log(f"fill bs {bs} ng {ng} {prec}: {worst:.2e}")
    assert worst <= 16 * EPS[prec] * np.max(np.abs(Uo))  # (a NaN fails too)


@pytest.mark.parametrize("n,nlev,prec", [(8, 1, "f64"), (56, 3, "f32"), (128, 1, "f32"),
                                         (136, 2, "f64"), (260, 1, "f64")])
def test_lifted_transform(orc, n, nlev, prec):
    u = np.random.default_rng(n).standard_normal((1, n, n, n))
    u = u.astype(np.float32).astype(np.float64) if prec == "f32" else u
    expect = orc.mr_forward(u, nlev, wacm.CDF44)
    d = torch.from_numpy(u).to("cuda", torch.float64 if prec == "f64" else torch.float32)
    work = wacm.mr_work(d)
    wacm.mr_forward(d, nlev, wacm.CDF44, work)
    fwd = np.max(np.abs(d.double().cpu().numpy() - expect))
    wacm.mr_inverse(d, nlev, wacm.CDF44, work)
    back = np.max(np.abs(d.double().cpu().numpy() - u))
    # per level 3 axes of prediction (absolute weight sum 1.25) and 3 of
    # low-pass (sum of |h| 1208/512 < 2.4, 11 terms): an error of level k grows
    # at most 2.4^3 per later level in theory and far less in practice; 64 eps
    # per level and direction of the largest value
    tol = 64 * EPS[prec] * nlev * np.max(np.abs(expect))
    log(f"lifted transform n {n} levels {nlev} {prec}: {fwd:.2e} {back:.2e} (tol {tol:.1e})")
    assert fwd <= tol and back <= 2 * tol


@pytest.mark.parametrize("bs,ng,prec", [(16, 3, "f32"), (24, 4, "f64"), (32, 5, "f64")])
def test_two_steps_on_a_quadtree(orc, bs, ng, prec):
    lev, ix, iy = inputs.random_balanced_leaves2(bs, 1, 4, 40)
    prm = cases.three_vortex_params()
    c = cases.Case2("quadtree", bs, ng, 1.0, 1, 4, lev, ix, iy, prm)
    rng = np.random.default_rng(bs)
    c.fields = [0.1 * rng.standard_normal((len(lev), bs, bs)) for _ in range(3)]
    og = orc.Grid2D(bs, ng, 1.0, 1, 4, lev, ix, iy)
    gg = wacm.Grid.from_case(c, dtype=DT[prec])
    U = c.padded()
    U = U.astype(np.float32).astype(np.float64) if prec == "f32" else U
    pool = torch.zeros(gg.pool_shape(), dtype=gg.torch_dtype(), device="cuda")
    pool[:U.shape[0]] = torch.from_numpy(U).to("cuda", gg.torch_dtype())
    t, dt = (torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2))
    gg.rk4_steps(prm, t, dt, pool, gg.work(), 2, dt_mode=wacm.DT_CFL)
    t_o = 0.0
    for _ in range(2):
        dt_o = og.dt(prm, U)
        og.rk4_step(prm, dt_o, U)
        t_o += dt_o
    i = slice(ng, ng + bs)
    a, b = pool[:c.nb].double().cpu().numpy()[..., i, i], U[..., i, i]
    e = np.max(np.abs(a - b)) / np.max(np.abs(b))
    # one step is held to 1e-12 (FP32 1e-5), two to twice that
    tol = 2e-12 if prec == "f64" else 2e-5
    log(f"quadtree bs {bs} ng {ng} {prec}: {e:.2e}, t {t.item():.9e} vs {t_o:.9e}")
    assert e < tol and abs(t.item() - t_o) <= tol * t_o


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_schedule_of_a_large_grid_without_one_set(prec):
    lev, ix, iy, iz = inputs.random_balanced_leaves(3, 2, 6, 4200)
    codes = [wacm.treecode_encode(*q) for q in zip(lev, ix, iy, iz)]
    prm = cases.params(nu=1e-3, c0=5.0, c_gamma=1.0)
    got = []
    for sched in (None, dict(tile_rows=0, xcd_map=1)):
        g = wacm.Grid(24, 4, 1.0, 2, 6, codes, lev, DT[prec])
        if sched:
            g.set_schedule(**sched)
        gen = torch.Generator("cuda").manual_seed(1)
        U = torch.rand(g.pool().shape, generator=gen, device="cuda", dtype=g.torch_dtype())
        t, dt = (torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2))
        g.rk4_steps(prm, t, dt, U, g.work(), 2)
        got.append((U[:len(lev), :, 4:28, 4:28, 4:28].clone(), t.item(), dt.item()))
        del U, g
    assert torch.equal(got[0][0], got[1][0]) and got[0][1:] == got[1][1:]


@pytest.mark.parametrize("bs,ng,prec", [(16, 3, "f64"), (24, 4, "f32"), (32, 5, "f64")])
def test_filtered_steps_need_the_lattice_ghosts_alone(bs, ng, prec):
    from paper_1912_05371_amd import adaptive
    c = cases.random_octree(bs=bs, ng=ng, target=40, j0=1, jmax=3, seed=bs)
    g = wacm.Grid.from_case(c, dtype=DT[prec])
    U = np.random.default_rng(ng).standard_normal((c.nb, 4, c.P, c.P, c.P))
    prm = cases.params(nu=1e-3, c0=5.0, c_gamma=1.0)
    i = slice(ng, ng + bs)
    got = []
    for whole in (False, True):
        A = to_pool(g, U, fill=float("nan"))
        A[:, :, :ng] = A[:, :, ng + bs:] = float("nan")
        t, dt = (torch.full((1,), v, dtype=torch.float64, device="cuda") for v in (0.0, 1e-5))
        if whole:
            for _ in range(2):
                g.rk4_step(prm, t, dt, A, g.work(), dt_mode=wacm.DT_FIXED)
                g.sync_ghosts(A)
                g.filter_blocks(A, -1)
        else:
            adaptive.filtered_steps(g, prm, A, g.work(), t, dt, 2, -1, dt_mode=wacm.DT_FIXED)
        got.append(A[:c.nb, :, i, i, i].clone())
    assert torch.isfinite(got[0]).all() and torch.equal(got[0], got[1])
