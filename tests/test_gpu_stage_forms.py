"""The stage kernel's tile shapes on meshes where a tile's surface is most of
its faces: blocks of eight cells that are their own periodic neighbours,
outflow edges, unequal cell widths and both Riemann solvers.  Every fused shape
gives the split form's bits, and both stay within the parity bar of the
oracle, whose update is written cell by cell."""
import numpy as np
import pytest

from paper_2609_37859_amd import workloads as W
from tests.parity import TOL, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tdh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_37859_amd import tdh as T
    T.lib()
    return T


def _case(name, table):
    if name == "one_block":  # a single 8^3 block, periodic on itself
        cfg = W.Config()
        mesh = W.uniform_mesh(1, 1, 1, 8, (0.125, 0.1, 0.15))
    elif name == "row_outflow_hlle":  # outflow edges at every block, dual energy, HLLE
        cfg = W.Config(dual=1, riemann=1)
        mesh = W.uniform_mesh(3, 1, 2, 8, 0.05, bc=(1, 1, 0))
    elif name == "mixed_edges":  # 8^3 beside 16^3 blocks
        cfg = W.Config(dual=1)
        split = np.zeros((1, 2, 2), dtype=bool)
        split[0, 1, 0] = True
        mesh = W.mixed_mesh((2, 2, 1), 16, split, 0.03, bc=(1, 0, 1))
    else:  # the table EOS, seeded
        cfg = W.Config(eos_kind=1, dual=1, rho_floor=1e-12, p_floor=0.0, e_floor=table.e_floor)
        mesh = W.uniform_mesh(2, 1, 1, 8, 1e10, bc=(0, 1, 0))
        rng = np.random.default_rng(4)
        U = np.empty(int(mesh.offsets(6)[-1]))
        for b in range(mesh.nblocks):  # states over five decades in density and two in temperature
            q = W.unpack_block(mesh, 6, U, b)
            rho = 10.0 ** rng.uniform(-9, -4, q.shape[1:])
            e = W.saha_pe(rho, 10.0 ** rng.uniform(4, 6, q.shape[1:]))[1]
            v = rng.uniform(-1e7, 1e7, (3,) + q.shape[1:])
            q[0], q[1:4], q[5] = rho, rho * v, rho * e
            q[4] = q[5] + 0.5 * rho * (v ** 2).sum(0)
        return cfg, mesh, U
    return cfg, mesh, W.random_smooth_state(mesh, cfg, 11, amp=0.3)


@pytest.mark.parametrize("name", ["one_block", "row_outflow_hlle", "mixed_edges", "table"])
def test_tile_shapes_on_small_meshes(tdh, orc, saha, name):
    cfg, mesh, U = _case(name, saha)
    table = saha if cfg.eos_kind == 1 else None
    out = {}
    shapes = tdh.tile_shapes()
    for t, dims in enumerate(shapes):
        if dims[0] and any(int(n) % d for n in mesh.blk[:, 0] for d in dims[:3]):
            continue
        for mode in (0, 3, 4) if table is not None else (0,):
            ctx = tdh.Context(cfg, mesh, U, table=table, inv_mode=mode)
            ctx.set_tile(t)
            tdh.run_sync_steps(ctx, 3)
            out[t, mode] = ctx.get_state()
            ctx.close()
    split = next(t for t, d in enumerate(shapes) if d[0] == 0)
    for key, g in out.items():
        assert np.array_equal(g, out[split, 0]), (key, shapes[key[0]])
    o, _ = orc.run_sync(cfg, mesh, U, 3, table=table)
    err = rel_err(cfg.nv, mesh, out[split, 0], o)
    assert np.all(err <= TOL), err


def test_seeds_after_each_stage_are_the_states_cells(tdh, saha):
    """The cells that modes 2, 3 and 4 hold after steps without a CFL reduction
    are those of the state (the search in the stage ends at the exact cell)."""
    cfg, mesh, U = _case("table", saha)
    cells = []
    for mode in (2, 3, 4):
        ctx = tdh.Context(cfg, mesh, U, table=saha, inv_mode=mode)
        _, dt, _, _ = ctx.reduce_dt()
        for _ in range(2):
            ctx.step_level(0, 0.5 * dt)
        cells.append(ctx.seed_cells())
        state = ctx.get_state()
        ctx.close()
    exact = np.empty(mesh.ncells, dtype=np.int64)
    k = 0
    for b in range(mesh.nblocks):
        q = W.unpack_block(mesh, 6, state, b).reshape(6, -1)
        kin = 0.5 * (q[1] ** 2 + q[2] ** 2 + q[3] ** 2) / q[0]
        Uc = q[4] - kin
        Ue = np.maximum(np.where((Uc > 0) & (Uc > cfg.eta1 * q[4]), Uc, q[5]), q[0] * cfg.e_floor)
        x = np.clip((np.log10(q[0]) - saha.lr0) / saha.dlr, 0, saha.nrho - 1)
        i = np.minimum(x.astype(int), saha.nrho - 2)
        w = x - i
        col = (1 - w)[:, None] * saha.le[i] + w[:, None] * saha.le[i + 1]
        j = (col <= np.log10(Ue / q[0])[:, None]).sum(1) - 1
        exact[k:k + q.shape[1]] = np.clip(j, 0, saha.nT - 2)
        k += q.shape[1]
    for c in cells:
        # a target within rounding of a node may fall to either side
        assert np.mean(c != exact) < 1e-3 and np.max(np.abs(c - exact)) <= 1
        assert np.array_equal(c, cells[0])


@pytest.mark.parametrize("dual", [0, 1])
@pytest.mark.parametrize("riemann", [0, 1])
@pytest.mark.parametrize("dense", [0, 1])
def test_stage_minima_are_the_reductions(tdh, dual, riemann, dense):
    """Ideal gas: the time step from the minima the last second stage left (where
    it leaves any: not with dense ghosts, nor the split form) equals the one
    reduced from the state, bit for bit."""
    cfg = W.Config(dual=dual, riemann=riemann, ghost_dense=dense)
    split = np.zeros((1, 2, 1), dtype=bool)
    split[0, 1, 0] = True
    mesh = W.mixed_mesh((1, 2, 1), 16, split, 0.03, bc=(1, 0, 1))
    for tile in (0, tdh.tile_shapes().index(next(d for d in tdh.tile_shapes() if d[0] == 0))):
        ctx = tdh.Context(cfg, mesh, W.random_smooth_state(mesh, cfg, 5, amp=0.3))
        ctx.set_tile(tile)
        for _ in range(2):
            r = ctx.reduce_dt()
            ctx.run_window(r[1] * 2 ** r[3], batched=True)
        a, b = ctx.reduce_dt(), ctx.reduce_dt(static=True)
        assert np.array_equal(a[0], b[0]) and a[1] == b[1]
        ctx.close()


@pytest.mark.parametrize("var, dual", [(0, 0), (0, 1), (1, 1), (4, 1)])
@pytest.mark.parametrize("riemann", [0, 1])
@pytest.mark.parametrize("value", [1e160, 1e200, 1e290, np.inf, -np.inf, np.nan])
def test_slopes_that_overflow_stay_infinite(tdh, orc, var, dual, riemann, value):
    """The limiter's quotient where the product of the differences overflows, and
    on infinities and NaN: a stage turns the same values NaN and infinite as the
    oracle's 2 a b / (a + b) does, so a state that blows up is not hidden."""
    cfg = W.Config(dual=dual, riemann=riemann)
    mesh = W.uniform_mesh(1, 1, 1, 8, 0.1, bc=(1, 1, 1))
    U = W.uniform_state(mesh, cfg)
    q = W.unpack_block(mesh, cfg.nv, U, 0)
    for k, f in ((3, 0.25), (4, 1.0), (5, 3.0)):  # a rising flank: equal signs either side of the middle cell
        q[var, 4, 4, k] = f * value
    ctx = tdh.Context(cfg, mesh, U)
    ctx.step_level(0, 1e-4)
    g = ctx.get_state()
    ctx.close()
    o, _ = orc.run_sync(cfg, mesh, U, 1, dts=[1e-4])
    for kind in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(kind(g), kind(o)), (kind.__name__, int(kind(g).sum()), int(kind(o).sum()))


@pytest.mark.parametrize("name", ["levels", "refined"])
def test_network_finds_the_cells_of_a_window_without_any(tdh, saha, name):
    """Mode 4 with the network on, windows with levels on one and on two refinement
    levels: a state set after its reduction holds no table cells, so the window
    starts with the network's pass (one launch more than a window whose cells are
    held), and gives mode 0's bits whatever the network predicts."""
    box = (6, 8, 8, 10, 4, 6)
    if name == "levels":
        cfg, mesh, U = W.debris_stream_c5(saha, box=box)
    else:
        cfg, mesh, U = W.debris_stream_amr(saha, box=box)
    out = {}
    for mode, params in ((0, None), (4, 5), (4, 6)):
        ctx = tdh.Context(cfg, mesh, U, table=saha, inv_mode=mode)
        if params is not None:
            ctx.mlp_init(W.mlp_init_params(params), W.seed_ranges(saha))
            ctx.mlp_enable_seed(True)
        _, dt0, _, lmax = ctx.reduce_dt()
        assert lmax > 0
        launches = []
        for held in (False, True):
            if not held:
                ctx.set_state(U)
            before = ctx.stats()["kernel_launches"]
            ctx.run_window(dt0 * 2 ** lmax, batched=True)
            launches.append(ctx.stats()["kernel_launches"] - before)
            out.setdefault((mode, params), []).append(ctx.get_state())
        assert launches[0] - launches[1] == (1 if mode == 4 else 0)
        ctx.close()
    for a, b in zip(out[4, 5] + out[4, 6], 2 * out[0, None]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("split", [0.75, 1.0])
def test_flux_correction_on_many_blocks(tdh, orc, split):
    """More blocks than a wave per 64 cells of every face would fill the chip with
    (65536 waves): a wave takes several parts of a face of 32^2 cells, and blocks of
    16^3 beside them take fewer.  Random levels, so that most faces are corrected."""
    cfg = W.Config(n_lat=1)
    rng = np.random.default_rng(12)
    cut = rng.random((1, 10, 13)) < split
    cut[0, 3, 4] = cut[0, 3, 5] = False
    mesh = W.mixed_mesh((13, 10, 1), 32, cut, 1.0 / 64, bc=(1, 0, 1))
    assert 6 * 16 * mesh.nblocks > 65536
    U = W.random_smooth_state(mesh, cfg, 2, amp=0.3)
    levels = rng.integers(0, 2, mesh.nblocks)
    ctx = tdh.Context(cfg, mesh, U)
    ctx.set_levels(levels)
    ctx.run_window(2e-3, batched=True)
    g = ctx.get_state()
    ctx.close()
    o, _ = orc.lat_window(cfg, mesh, U, levels, 1e-3)
    assert np.all(rel_err(cfg.nv, mesh, g, o) <= TOL)
