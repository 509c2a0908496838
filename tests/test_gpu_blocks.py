"""GPU reconstruction where the layout of the staged blocks changes: meshes
stretched along x, whose blocks have more distinct members, and order 6, whose
records are the longest, so that set-up halves the wavefronts per block or
stages one block instead of two.  Against the CPU oracle, with the bars of
test_gpu_parity.py: face states max_i |x - y| <= 1e-12 max_i |y|, flags exact
outside near ties.

Stretched meshes only with the TENO selection, which rejects the large stencil
across the jumps: at aspect 16 the nearest cells lie in one column, the
least-squares condition is 3e4, and for a scheme that keeps the large stencil
everywhere the oracle itself is 3e-10 from an 80-bit solution."""
import numpy as np
import pytest

from paper_2105_02127_amd import inputs
from parity_check import assert_adjoint, assert_states, check_flags
from test_blocks_host import _run, _write, driver  # noqa: F401  (the host driver's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,n", [(3, 5), (4, 64), (4, 65), (5, 64), (5, 65), (6, 64), (6, 65),
                                     (6, 90), (6, 91)])
def test_small_mesh_reconstruction_equals_blocks(order, n):
    """Small meshes are reconstructed a tile per workgroup, a wavefront per stencil
    (up to 512 tiles of 16 cells; 1,024 at order 3), batches always by blocks: the
    same bits, and those of the residual with its flags frozen."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_02127_amd import teno
    from paper_2105_02127_amd.batch import Batch
    print(f"[case] small order={order} n={n}", flush=True)
    m = (inputs.jittered_periodic_mesh(n, 43) if n > 5 else
         inputs.jittered_box_mesh(11, n, 43))       # 110 cells: a part of a block
    lm = teno.Mesh(m.xy, m.tri, period=m.period).setup(order=order, fallback=1)
    sv = teno.Solver(lm)
    U = torch.as_tensor(inputs.random_lines(m)[lm.perm], device="cuda")
    b = Batch([sv])
    b.set_tuning(order_mode=1, waves_per_cu=0, item_order=0, use_graph=0)
    dt = b.max_dt([U], 0.4)
    w = U.clone()
    flags = sv.empty_flags(3)
    sv.rk_step(w, dt.clone(), flags3=flags)
    b.rk_step([U], dt)
    torch.cuda.synchronize()
    assert torch.equal(w, U)
    f = sv.empty_flags()
    R = sv.residual(w, flags=f)
    assert torch.equal(sv.residual_frozen(w, f), R)


@pytest.mark.parametrize("order,n,aspect,variant,characteristic", [
    (3, 60, 32, 0, 0),   # four wavefronts, two blocks of 471 members
    (4, 60, 16, 0, 0),   # four, one block
    (6, 60, 1, 0, 0),    # eight, two blocks
    (6, 60, 1, 2, 1),
    (6, 26, 1, 0, 1),    # four, one block, in characteristic variables
    (6, 26, 1, 2, 0),
    (6, 26, 1, 1, 0),    # ... and no small stencils
    (6, 26, 8, 0, 0),    # two, one block
])
def test_block_layouts(oracle_mod, order, n, aspect, variant, characteristic):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_02127_amd import teno
    print(f"[case] order={order} n={n} aspect={aspect} variant={variant} "
          f"characteristic={characteristic}", flush=True)
    m = inputs.jittered_periodic_mesh(n, 41)
    U = inputs.make_state(m, "random_lines")
    xy = np.ascontiguousarray(m.xy * [1.0, 1.0 / aspect])
    period = (1.0, 1.0 / aspect)
    kw = dict(order=order, fallback=1, variant=variant, characteristic=characteristic)
    lm = teno.Mesh(xy, m.tri, period=period).setup(**kw)
    sv = teno.Solver(lm)
    om = oracle_mod.OracleMesh(xy, m.tri, period=period)
    om.setup(oracle_mod.params(**kw), all_cells=True)
    want = om.residual(U, want_fp=True)
    flags = sv.empty_flags()
    fs = sv.reconstruct(torch.as_tensor(U[lm.perm], device="cuda"), flags=flags)
    torch.cuda.synchronize()
    got = np.empty((m.n_cell, fs.shape[0], 4))
    got[lm.perm] = fs.permute(1, 0, 2).cpu().numpy()
    assert_states(got, want["fp"].reshape(m.n_cell, -1, 4), what="face states")
    if variant != 2:
        f = flags.cpu().numpy().view(np.uint16)
        fu = np.empty_like(f)
        fu[..., lm.perm] = f
        check_flags(fu, want["flags"], want["diag"]["tie_mask"])


@pytest.mark.parametrize("order,n", [(3, 9), (3, 127), (3, 128), (3, 129), (5, 104), (5, 105)])
def test_step_equals_batched_step(order, n):
    """Small meshes form fluxes and update in one launch (up to 32,768 cells with
    two points per face, 21,845 with three), batches in two: the same bits, and
    the next step's dt that of the new state."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_02127_amd import teno
    from paper_2105_02127_amd.batch import Batch
    print(f"[case] step order={order} n={n}", flush=True)
    m = inputs.jittered_periodic_mesh(n, 43)
    lm = teno.Mesh(m.xy, m.tri).setup(order=order, fallback=1)
    sv = teno.Solver(lm)
    U = torch.as_tensor(inputs.make_state(m, "random_lines")[lm.perm], device="cuda")
    b = Batch([sv])
    b.set_tuning(order_mode=1, waves_per_cu=0, item_order=0, use_graph=0)
    dt = b.max_dt([U], 0.4)
    w, d = U.clone(), dt.clone()
    sv.rk_step_dt(w, d, 0.4)
    b.rk_step([U], dt)
    torch.cuda.synchronize()
    assert torch.equal(w, U)
    assert torch.equal(d, sv.max_dt(w, 0.4))


@pytest.mark.parametrize("order,n", [(3, 13), (5, 13), (3, 14)])
def test_tetrahedral_residual_on_both_update_paths(order, n):
    """Tetrahedral meshes of up to 16,384 cells form fluxes and update in one
    launch, larger ones in two: residuals at sampled cells within 1e-12 of the
    flux scale, and conservation over the periodic mesh, on both sides (13,182
    cells, no multiple of a block's eight, and 16,464)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import tet
    from paper_2105_02127_amd import inputs3, teno3
    from test_gpu_tet import Case3
    m = inputs3.jittered_periodic_cube(n, 47)
    U = inputs3.random_planes3(m)
    c = Case3(teno3, tet, torch, m, U, order, f"update paths n={n}", oracle_all=False, fallback=1)
    R = c.user(c.sv.residual(c.Ud))
    cells = np.linspace(0, m.n_cell - 1, 60).astype(np.int32)
    want, _ = c.om.residual_cells(U, cells)
    scale = c.flux_scale()
    assert np.abs(R[cells] - want).max() <= 1e-12 * scale
    vol, _, _ = c.om.geometry()
    assert np.abs((vol[:, None] * R).sum(0)).max() <= 1e-12 * scale * vol.sum()


@pytest.mark.parametrize("order,variant", [(3, 0), (3, 1), (3, 2), (4, 0), (4, 2)])
def test_characteristic_past_the_first_blocks(oracle_mod, order, variant):
    """576,738 cells: about twelve blocks per resident workgroup, so that the
    Gram matrices of one block lie beside the staged members and the ids of the
    next ones."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_02127_amd import teno
    from test_gpu_parity import _sampled
    _sampled(teno, oracle_mod, torch, 6, n_sample=160, characteristic=1, variant=variant,
             order=order)


@pytest.mark.parametrize("order,n,aspect,variant,characteristic,tiles,buffers", [
    (6, 300, 4, 0, 0, 4, 1), (6, 200, 4, 0, 1, 4, 1), (6, 240, 1, 2, 1, 8, 2), (5, 200, 16, 0, 0, 4, 1), (6, 200, 16, 0, 0, 2, 1),
    (4, 250, 16, 0, 0, 4, 1), (4, 250, 16, 0, 1, 4, 1), (3, 300, 32, 0, 0, 4, 2), (3, 300, 48, 0, 1, 4, 1)])
def test_block_layouts_past_the_first_blocks(oracle_mod, driver, order, n, aspect, variant,  # noqa: F811
                                             characteristic, tiles, buffers):
    """Every layout of the staged blocks (asked of set-up) with more blocks than
    workgroups, so that buffers alternate or one is filled again: face states and
    flags at sampled cells, bars as above; stretched meshes with the TENO selection
    only, for the reason above."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_02127_amd import teno
    print(f"[case] past the first blocks order={order} n={n} aspect={aspect} variant={variant} "
          f"characteristic={characteristic}", flush=True)
    m = inputs.jittered_periodic_mesh(n, 41)
    U = inputs.make_state(m, "random_lines")
    m.xy = np.ascontiguousarray(m.xy * [1.0, 1.0 / aspect])
    m.period = (1.0, 1.0 / aspect)
    tmp, exe = driver
    _write(tmp, "b", m)
    w = _run(exe, "mesh", tmp, "b", order, variant, characteristic).split()
    layout = dict(zip(w[::2], map(int, w[1::2])))
    assert (layout["bwaves"], layout["nbuf"]) == (tiles, buffers), layout
    # a CU holds at most as many workgroups as its LDS
    assert layout["blocks"] > 256 * (160 * 1024 // layout["lds"])
    kw = dict(order=order, fallback=1, variant=variant, characteristic=characteristic)
    lm = teno.Mesh(m.xy, m.tri, period=m.period).setup(**kw)
    sv = teno.Solver(lm)
    om = oracle_mod.OracleMesh(m.xy, m.tri, period=m.period)
    om.setup(oracle_mod.params(**kw), all_cells=False)
    cells = np.unique(np.random.default_rng(order).integers(0, m.n_cell, 120))
    fp, ofl, _, odg = om.reconstruct_cells(U, cells)
    flags = sv.empty_flags()
    fs = sv.reconstruct(torch.as_tensor(U[lm.perm], device="cuda"), flags=flags)
    inv = np.empty(m.n_cell, np.int64)
    inv[lm.perm] = np.arange(m.n_cell)
    got = fs[:, torch.as_tensor(inv[cells], device="cuda")].permute(1, 0, 2).cpu().numpy()
    assert_states(got, fp.reshape(len(cells), -1, 4), what="face states")
    if variant != 2:
        gfl = flags.cpu().numpy().view(np.uint16)[..., inv[cells]]
        check_flags(gfl.T if characteristic else gfl, ofl, odg["tie_mask"])


def _graded(order, angle, growth, **kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_02127_amd import teno
    print(f"[case] graded order={order} {angle} rad e^{growth} {kw}", flush=True)
    m = inputs.graded_sector_mesh(40, 3, angle, growth)
    U = inputs.conservative(1.0 + 0.3 * m.rng.uniform(-1, 1, m.n_cell), 0.3, 0.2, 1.0)
    lm = teno.Mesh(m.xy, m.tri, period=m.period).setup(order=order, **kw)
    return torch, m, U, lm, teno.Solver(lm)


@pytest.mark.parametrize("order", [3, 4, 5, 6])
@pytest.mark.parametrize("angle,growth", [(1.5, 4.0), (1.5, 8.0), (4.0, 4.0)])
def test_graded_mesh_large_stencils(driver, order, angle, growth):  # noqa: F811
    """Graded meshes, where set-up keeps the operators of some stencils: face
    states of the linear scheme against 128 bits.  The operators' own rounding of
    the differences (0.6, 41 rows of entries up to about 50 with basis values up to
    32) allows 1e-11 of the state; the normal matrices' bound, 1e-12, adds less."""
    torch, m, U, lm, sv = _graded(order, angle, growth, variant=1)
    tmp, exe = driver
    _write(tmp, "g", m)
    np.ascontiguousarray(U).tofile(tmp + "/g.u")
    _run(exe, "faces", tmp, "g", order, 13)
    cells = np.fromfile(tmp + "/g.cells", np.int32)
    want = np.fromfile(tmp + "/g.faces").reshape(len(cells), -1, 4)
    fs = sv.reconstruct(torch.as_tensor(U[lm.perm], device="cuda"))
    got = np.empty((m.n_cell, fs.shape[0], 4))
    got[lm.perm] = fs.permute(1, 0, 2).cpu().numpy()
    scale = max(np.abs(want).max(), 1.0)
    assert np.abs(got[cells] - want).max() <= 1e-11 * scale


@pytest.mark.parametrize("variant,characteristic", [(0, 0), (2, 0), (0, 1), (2, 1)])
def test_graded_mesh_small_stencils(oracle_mod, variant, characteristic):
    """The same at order 3, where the oracle's operators keep 1e-13 on such a mesh:
    selections and combinations of the small stencils, and the adjoint."""
    torch, m, U, lm, sv = _graded(3, 1.5, 4.0, variant=variant, characteristic=characteristic,
                                  fallback=1)
    om = oracle_mod.OracleMesh(m.xy, m.tri, period=m.period)
    om.setup(oracle_mod.params(order=3, variant=variant, characteristic=characteristic, fallback=1))
    want = om.residual(U, want_fp=True)
    flags = sv.empty_flags()
    Ud = torch.as_tensor(U[lm.perm], device="cuda")
    fs = sv.reconstruct(Ud, flags=flags)
    got = np.empty((m.n_cell, fs.shape[0], 4))
    got[lm.perm] = fs.permute(1, 0, 2).cpu().numpy()
    assert_states(got, want["fp"].reshape(m.n_cell, -1, 4), what="face states")
    if variant == 2:
        return
    f = flags.cpu().numpy().view(np.uint16)
    fu = np.empty_like(f)
    fu[..., lm.perm] = f
    check_flags(fu, want["flags"], want["diag"]["tie_mask"])
    if characteristic:
        return
    lam = m.rng.normal(size=U.shape)
    g = sv.vjp_residual(Ud, flags, torch.as_tensor(lam[lm.perm], device="cuda"))
    gu = np.empty_like(U)
    gu[lm.perm] = g.cpu().numpy()
    assert_adjoint(gu, om.vjp(U, fu, lam), om.vjp_scale(U, fu, lam), what="graded vjp")


@pytest.mark.parametrize("order", [3, 5, 6])
def test_graded_mesh_adjoint_is_the_transpose(order):
    """<lam, dR v> by central differences of the linear scheme's residual against
    <vjp, v>.  The oracle's own central difference at order 6 on this mesh is 7e-6
    off at a step of 1e-4 and 7e-8 at 1e-5 (the one-sided large stencils raise the
    perturbation a hundredfold, and the error falls with its square), 5e-10 at
    1e-6, where rounding adds 1e-9: step 1e-6, bar 1e-7."""
    torch, m, U, lm, sv = _graded(order, 1.5, 8.0, variant=1)
    U = inputs.conservative(1.0 + 0.02 * m.rng.uniform(-1, 1, m.n_cell), 0.3, 0.2, 1.0)
    Ud = torch.as_tensor(U[lm.perm], device="cuda")
    flags = sv.empty_flags()
    sv.reconstruct(Ud, flags=flags)
    vol = torch.as_tensor(np.ascontiguousarray(_areas(m)[lm.perm]), device="cuda")[:, None]
    g = torch.Generator(device="cuda").manual_seed(5)
    lam = vol * torch.randn(U.shape, generator=g, dtype=torch.float64, device="cuda")
    v = torch.randn(U.shape, generator=g, dtype=torch.float64, device="cuda")
    e = 1e-6
    dR = (sv.residual(Ud + e * v) - sv.residual(Ud - e * v)) / (2 * e)
    a, b = (lam * dR), sv.vjp_residual(Ud, flags, lam) * v
    assert abs(a.sum().item() - b.sum().item()) <= 1e-7 * a.abs().sum().item()


@pytest.mark.parametrize("order_mode", [0, 1])
def test_graded_meshes_in_a_batch(order_mode):
    """Batched steps of graded meshes of two orders and a jittered one: the bits of
    stepping them alone."""
    from paper_2105_02127_amd.batch import Batch
    from paper_2105_02127_amd import teno
    torch, m, U, lm, sv = _graded(4, 1.5, 8.0, fallback=1)
    svs, Us = [sv], [U[lm.perm]]
    lm = teno.Mesh(m.xy, m.tri, period=m.period).setup(order=5, fallback=1)
    svs.append(teno.Solver(lm))
    Us.append(U[lm.perm])
    p = inputs.jittered_periodic_mesh(20, 3)
    lm = teno.Mesh(p.xy, p.tri).setup(order=3, fallback=1)
    svs.append(teno.Solver(lm))
    Us.append(inputs.random_lines(p)[lm.perm])
    Us = [torch.as_tensor(u, device="cuda") for u in Us]
    alone = [u.clone() for u in Us]
    b = Batch(svs)
    b.set_tuning(order_mode=order_mode, waves_per_cu=0, item_order=0, use_graph=1)
    dt = b.max_dt(Us, 0.4)
    for _ in range(3):
        b.rk_step(Us, dt)
        for k, (s, u) in enumerate(zip(svs, alone)):
            s.rk_step(u, dt[k:k + 1].clone())
        torch.cuda.synchronize()
        for u, w in zip(Us, alone):
            assert torch.equal(u, w)


def _areas(m):
    x = m.xy[m.tri]
    d1, d2 = x[:, 1] - x[:, 0], x[:, 2] - x[:, 0]
    return 0.5 * np.abs(d1[:, 0] * d2[:, 1] - d1[:, 1] * d2[:, 0])
