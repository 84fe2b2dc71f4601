"""GPU parity of the HIP library against the FP64 CPU oracle, through the C ABI.

FP64 kernels must match the oracle within 1e-12 relative per field (max
abs difference over max |q|); FP32 kernels are compared with the FP64 GPU
path within per-field relative L2 tolerances measured and frozen here."""
import numpy as np
import pytest

import hlbm_inputs as hi
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2002_03644_amd import HLBM_EDIVERGED, HLBM_OK, HlbmError, Params, Solver  # noqa: E402

FIELDS = ("rho", "ux", "uy", "s")


def rel_max(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


def rel_l2(a, b, centre=False):
    ref = b - b.mean() if centre else b
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(ref), 1e-300))


def gpu_moments(S):
    return {k: v.double().cpu().numpy() for k, v in S.moments().items()}


def pair(nx, ny, fields, steps, gamma=1.4, **kw):
    """Run the oracle and the FP64 GPU path from the same s bytes."""
    r, u, v, t = fields
    s = oracle.entropy_from_theta(r, t, gamma)
    okw = {k: kw[k] for k in ("mu", "sigma", "bc_x", "bc_y", "phi_mode", "e1_centred",
                              "e2_off", "prandtl") if k in kw}
    O = oracle.OracleSolver(oracle.OracleParams(nx, ny, gamma=gamma, **okw), r, u, v, s=s)
    G = Solver(Params(nx, ny, dtype="f64", gamma=gamma, **kw), r, u, v, s=s)
    O.step(steps)
    G.step(steps)
    return O.moments(), gpu_moments(G), O, G


def assert_parity(mo, mg, tol=1e-12):
    """Per field max |gpu - oracle| / max |oracle|; both velocity components
    are scaled by the largest velocity magnitude (a component can be
    identically zero, e.g. u_y of a quasi-1D tube)."""
    vscale = max(np.abs(mo["ux"]).max(), np.abs(mo["uy"]).max(), 1e-300)
    for k in FIELDS:
        scale = vscale if k in ("ux", "uy") else np.abs(mo[k]).max()
        err = float(np.abs(mg[k] - mo[k]).max() / scale)
        assert err < tol, (k, err)


# ------------------------------------------------------------ FP64 vs oracle
@pytest.mark.parametrize("sigma", [0.0, 0.5])
def test_f64_vortex_several_tiles_ragged(sigma):
    """130 x 70 vortex: several workgroup tiles in x and y with ragged tails."""
    nx, ny = 130, 70
    f = hi.vortex(nx, ny, 60, 35, 8, 0.5, 0.25, noise=1e-6, seed=0)
    mo, mg, _, _ = pair(nx, ny, f, 60, mu=1e-3, sigma=sigma)
    assert_parity(mo, mg)


@pytest.mark.parametrize("sigma", [0.0, 0.5])
def test_f64_vortex_128_full_run(sigma):
    """Isentropic vortex, 128^2 periodic, Ma 0.5, vortex Mach 0.25, R = 10,
    nu = 1e-3, density noise 1e-6 (seed 0), 500 steps."""
    n = 128
    f = hi.vortex(n, n, 64, 64, 10, 0.5, 0.25, noise=1e-6, seed=0)
    mo, mg, _, _ = pair(n, n, f, 500, mu=1e-3, sigma=sigma)
    assert_parity(mo, mg)


def test_f64_sod_4096x4():
    """Sod tube 4096 x 4, x extrapolated, y periodic, nu = 1e-3, sigma = 0.4,
    finite-difference Phi.  After 100 steps the strict 1e-12 gate holds.  Over
    the full 2000 steps the under-resolved shock (cell Reynolds number ~200)
    amplifies rounding: the bound is ten times the oracle's own response to a
    1e-15 relative density perturbation, measured here."""
    nx, ny = 4096, 4
    f = hi.sod(nx, ny)
    kw = dict(mu=1e-3, sigma=0.4, phi_mode="fd", bc_x="extrapolate")
    mo, mg, O, G = pair(nx, ny, f, 100, **kw)
    assert_parity(mo, mg)
    O.step(1900)
    G.step(1900)
    mo, mg = O.moments(), gpu_moments(G)
    r, u, v, t = f
    s = oracle.entropy_from_theta(r, t, 1.4)
    noise = np.random.default_rng(0).uniform(-1, 1, (1, nx)).repeat(ny, 0)
    okw = {k: kw[k] for k in kw}
    B = oracle.OracleSolver(oracle.OracleParams(nx, ny, **okw), r * (1 + 1e-15 * noise), u, v,
                            s=s)
    B.step(2000)
    mb = B.moments()
    for k in ("rho", "ux", "s"):
        sens = rel_max(mb[k], mo[k])
        err = rel_max(mg[k], mo[k])
        print(f"sod 2000 steps {k}: gpu-oracle {err:.3e}, oracle 1e-15 sensitivity {sens:.3e}")
        assert err <= max(1e-12, 10 * sens), (k, err, sens)


@pytest.mark.parametrize("opts", [
    dict(bc_x="extrapolate", bc_y="extrapolate", phi_mode="fd", sigma=0.3),
    dict(bc_x="periodic", bc_y="extrapolate", sigma=0.9, prandtl=1.3),
    dict(e1_centred=True, e2_off=True, sigma=0.2),
    dict(precise_theta=True, sigma=0.5),
])
def test_f64_options(opts):
    nx, ny = 75, 66
    f = hi.random_smooth(nx, ny, seed=17, amp=0.05, u0=(0.2, -0.1))
    mo, mg, _, _ = pair(nx, ny, f, 40, mu=3e-3, **opts)
    assert_parity(mo, mg)


@pytest.mark.parametrize("shape", [(1, 1), (1, 9), (9, 1), (2, 3), (5, 2), (3, 200), (61, 2)])
def test_f64_degenerate_shapes(shape):
    """Grids thinner than the stencil radius and than one tile."""
    nx, ny = shape
    f = hi.random_smooth(nx, ny, seed=3, amp=0.03)
    for bc in ("periodic", "extrapolate"):
        mo, mg, _, _ = pair(nx, ny, f, 12, mu=2e-3, sigma=0.5, bc_x=bc, bc_y=bc)
        assert_parity(mo, mg)


def test_f64_supersonic_vortex():
    n = 96
    f = hi.vortex(n, n, 30, 48, 8, 1.3, 0.13)
    mo, mg, _, _ = pair(n, n, f, 80, mu=1e-3, sigma=0.0)
    assert_parity(mo, mg)


def test_f64_populations_match_oracle():
    n = 33
    f = hi.random_smooth(n, n, seed=5, amp=0.05)
    _, _, O, G = pair(n, n, f, 7, mu=2e-3, sigma=0.7)
    Fo, so = O.state()
    Fg = G.populations().cpu().numpy()
    assert np.abs(Fg - Fo).max() / np.abs(Fo).max() < 1e-12


# ------------------------------------------------------- tiles and determinism
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_tile_shape_invariance(dtype):
    """Per-node arithmetic does not depend on the tile, so every tile shape
    must give the same result; a difference means a race or halo bug.  FP64
    is built without contraction and is compared bitwise.  FP32 uses fused
    multiply-adds whose placement may differ between compiled copies of the
    row loop (a peeled iteration vs the loop body), so it is compared within
    a few units in the last place."""
    nx, ny = 301, 97
    r, u, v, t = hi.vortex(nx, ny, 150, 48, 9, 0.9, 0.3, noise=1e-4, seed=1)
    s = oracle.entropy_from_theta(r, t, 1.4)
    outs = []
    for tw, th in ((64, 8), (128, 32), (256, 5), (64, 97), (128, 1), (192, 16), (192, 7)):
        G = Solver(Params(nx, ny, dtype=dtype, mu=1e-3, sigma=0.3, tile_w=tw, tile_h=th),
                   r, u, v, s=s)
        G.step(25)
        outs.append(torch.cat([G.populations().flatten(), G.moments()["s"].flatten()]))
    for o in outs[1:]:
        if dtype == "f64":
            assert torch.equal(o, outs[0])
        else:
            assert (o - outs[0]).abs().max().item() < 2e-6


@pytest.mark.parametrize("nx,ny,dtype", [(64, 64, "f32"),
                                         (1031, 1100, "f32"),   # 4.5 MB planes: padded stride
                                         (800, 700, "f64")])    # 4.5 MB planes: padded stride
def test_checkpoint_resume_bitwise(nx, ny, dtype):
    r, u, v, t = hi.vortex(nx, ny, nx / 2, ny / 2, 6, 0.5, 0.25)
    A = Solver(Params(nx, ny, dtype=dtype, mu=1e-3), r, u, v, theta=t)
    A.step(10)
    snap = A.save_state()
    A.step(10)
    ref = A.populations().clone()
    B = Solver(Params(nx, ny, dtype=dtype, mu=1e-3), r, u, v, theta=t)
    B.load_state(snap)
    B.step(10)
    assert torch.equal(B.populations(), ref)
    # populations and entropy written back through the ABI give the same
    # state and the same next steps: exactly in FP64 (absolute storage),
    # within a few FP32 ulps where storage subtracts the rest state
    C = Solver(Params(nx, ny, dtype=dtype, mu=1e-3), r, u, v, theta=t)
    C.set_populations(ref, A.moments()["s"])
    A.step(3)
    C.step(3)
    if dtype == "f64":
        assert torch.equal(C.populations(), A.populations())
    else:
        scale = ref.abs().max().item()
        assert (C.populations() - A.populations()).abs().max().item() < 1e-6 * scale


# --------------------------------------------------------- conservation/status
def test_conservation_totals():
    n = 96
    r, u, v, t = hi.random_smooth(n, n, seed=9, amp=0.05)
    G = Solver(Params(n, n, dtype="f64", mu=2e-3, sigma=0.5), r, u, v, theta=t)
    t0 = G.totals()
    G.step(200)
    t1 = G.totals()
    assert abs(t1[0] - t0[0]) / t0[0] < 1e-13
    assert abs(t1[1] - t0[1]) / t0[0] < 1e-13
    assert abs(t1[2] - t0[2]) / t0[0] < 1e-13
    O = oracle.OracleSolver(oracle.OracleParams(n, n, mu=2e-3, sigma=0.5), r, u, v, theta=t)
    O.step(200)
    np.testing.assert_allclose(t1, O.totals(), rtol=1e-12, atol=1e-13)
    F = Solver(Params(n, n, dtype="f32", mu=2e-3, sigma=0.5), r, u, v, theta=t)
    f0 = F.totals()
    F.step(200)
    f1 = F.totals()
    assert abs(f1[0] - f0[0]) / f0[0] < 1e-6


def test_status_flags_divergence():
    n = 40
    r, u, v, t = hi.random_smooth(n, n, seed=2)
    G = Solver(Params(n, n, dtype="f64", mu=1e-3), r, u, v, theta=t)
    code, cfl = G.status()
    assert code == HLBM_OK and 0 < cfl < 1
    F = G.populations()
    m = G.moments()
    F[3, 5, 7] = float("nan")
    G.set_populations(F, m["s"])
    assert G.status()[0] == HLBM_EDIVERGED
    G.step(2)
    assert G.status()[0] == HLBM_EDIVERGED


def test_init_rejects_bad_fields():
    n = 16
    r, u, v, t = hi.random_smooth(n, n, seed=2)
    r = r.copy()
    r[3, 3] = -1.0
    with pytest.raises(HlbmError):
        Solver(Params(n, n, dtype="f64"), r, u, v, theta=np.abs(t))


def test_init_warns_cfl():
    r, u, v, t = hi.uniform(8, 8, 1.0, 0.9, 0.0, 0.3)
    G = Solver(Params(8, 8, dtype="f64"), r, u, v, theta=t)
    assert G.init_code == 1


# ----------------------------------------------------------- FP32 vs FP64
# Per-field relative L2 of FP32 vs the FP64 GPU path (rho and u centred on
# their mean), measured on MI355X and frozen with ~2x headroom.
#  - vortex, 128^2, 500 steps: rho 8.3e-5, ux 1.5e-4, uy 5.3e-5, s 2.5e-8.
#  - turbulence 1024^2, 1000 steps: rho 1.2e-4, u 5.7e-5, s 3.8e-7 (the FP64
#    run with FP32-rounded inputs alone differs by 7.8e-5 / 4.0e-5: chaotic flow).
#  - Sod 4096 x 4: 1.5e-6 after 100 steps; after 2000 steps 2.3e-2 / 1.2e-1 /
#    2.9e-3.  The under-resolved shock amplifies spatially varying rounding
#    ~1e9-fold over 2000 steps (FP64: 1e-15 noise -> 1.6e-6), so FP32's
#    per-step rounding (~1e-8) saturates at percent level.
FP32_TOL = {
    "vortex": dict(rho=2e-4, ux=3e-4, uy=2e-4, s=1e-7),
    "turbulence": dict(rho=3e-4, ux=2e-4, uy=2e-4, s=1e-6),
    "sod100": dict(rho=2.5e-6, ux=6e-5, s=8e-7),   # measured 6.4e-7, 1.5e-5, 2.1e-7
    "sod2000": dict(rho=5e-4, ux=3e-3, s=1e-4),   # measured 1.2e-4, 7.3e-4, 2.1e-5
    "mach2_300": dict(rho=6e-5, ux=1e-4, s=3e-7),     # measured 1.4e-5, 2.5e-5, 6.7e-8
    "mach2_2000": dict(rho=3.5e-3, ux=7e-3, s=1.4e-5),  # measured 8.6e-4, 1.7e-3, 3.3e-6
}


def f32_vs_f64(nx, ny, fields, steps, theta_ref=None, **kw):
    r, u, v, t = fields
    s = oracle.entropy_from_theta(r, t, kw.get("gamma", 1.4))
    A = Solver(Params(nx, ny, dtype="f64", **kw), r, u, v, s=s)
    extra = {} if theta_ref is None else dict(theta_ref=theta_ref)
    B = Solver(Params(nx, ny, dtype="f32", **extra, **kw), r, u, v, s=s)
    A.step(steps)
    B.step(steps)
    return gpu_moments(A), gpu_moments(B), A, B


def check_tol(name, ma, mb, fields):
    errs = {k: rel_l2(mb[k], ma[k], centre=k != "s") for k in fields}
    print(f"fp32 {name} rel L2:", {k: f"{e:.2e}" for k, e in errs.items()})
    for k in fields:
        assert errs[k] < FP32_TOL[name][k], (k, errs[k])


def test_f32_vortex_tolerance():
    n = 128
    f = hi.vortex(n, n, 64, 64, 10, 0.5, 0.25, noise=1e-6, seed=0)
    ma, mb, _, _ = f32_vs_f64(n, n, f, 500, mu=1e-3, sigma=0.5)
    check_tol("vortex", ma, mb, FIELDS)


def test_f32_turbulence_tolerance():
    n = 1024
    f = hi.turbulence(n, 0.5, hi.THETA_PAPER, seed=0)
    ma, mb, _, B = f32_vs_f64(n, n, f, 1000, mu=1e-3, sigma=0.0)
    assert B.status()[0] == HLBM_OK
    check_tol("turbulence", ma, mb, FIELDS)


def test_f32_mach2_shock_tolerance():
    """Mach-2 normal shock 2048 x 512 from Rankine-Hugoniot states (x
    extrapolated, seeded upstream perturbation, theta_ref at the upstream
    temperature): FP32 against FP64 after 300 and 2000 steps."""
    nx, ny = 2048, 512
    f = hi.normal_shock(nx, ny, mach=2.0, theta1=0.1, perturb=1e-3, seed=0)
    ma, mb, A, B = f32_vs_f64(nx, ny, f, 300, theta_ref=0.1, mu=1e-3, sigma=0.0,
                              phi_mode="fd", bc_x="extrapolate")
    check_tol("mach2_300", ma, mb, ("rho", "ux", "s"))
    A.step(1700)
    B.step(1700)
    assert A.status()[0] == HLBM_OK and B.status()[0] == HLBM_OK
    check_tol("mach2_2000", gpu_moments(A), gpu_moments(B), ("rho", "ux", "s"))


def test_f32_sod_tolerance():
    nx, ny = 4096, 4
    ma, mb, A, B = f32_vs_f64(nx, ny, hi.sod(nx, ny), 100, theta_ref=0.2, mu=1e-3, sigma=0.4,
                              phi_mode="fd", bc_x="extrapolate")
    check_tol("sod100", ma, mb, ("rho", "ux", "s"))
    A.step(1900)
    B.step(1900)
    check_tol("sod2000", gpu_moments(A), gpu_moments(B), ("rho", "ux", "s"))


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_theta_of_any_density(dt):
    """theta = rho^(gamma - 1) exp(s / c_v) of the fields, also where no flow gets:
    zero, negative, subnormal and infinite densities, entropies past the
    exponential's range (FP32: those whose deviation form is exact)."""
    inf = float("inf")
    rho = [1.0, 0.7, 3.0, -1.0, inf, 1.0, 1.0]
    s = [-1.0, 0.2, 0.5, 0.1, 0.1, inf, -inf]
    if dt == "f64":
        rho += [0.0, 1e-310, 1e300, 1.0, 1.0, 1.0]
        s += [0.3, -1.0, 0.1, 591.25, 600.0, -640.0]
    td = torch.float64 if dt == "f64" else torch.float32
    n = len(rho)
    one = np.ones((1, n))
    S = Solver(Params(n, 1, dtype=dt), one, 0 * one, 0 * one, theta=0.2 * one)
    F = torch.zeros(9, 1, n, dtype=td)
    F[0, 0] = torch.tensor(rho, dtype=td)
    sv = torch.tensor(s, dtype=td)[None]
    S.set_populations(F, sv)
    got = S.moments()["theta"].cpu().double()[0]
    cv = (1.0 / 3.0) / 0.4
    want = torch.exp(sv[0].double() / cv + 0.4 * torch.log(F[0, 0].double()))
    # the argument's rounding, twice: |x| up to 710, in FP32 up to 2
    tol = 1e-12 if dt == "f64" else 1e-5
    for k in range(n):
        assert torch.allclose(got[k], want[k], rtol=tol, atol=0.0, equal_nan=True), (
            rho[k], s[k], got[k], want[k])
