"""Restart remap, Galilean boost and frame acceleration on the GPU (through the
C ABI) against the oracle."""
import numpy as np
import pytest

from paper_2609_37859_amd import workloads as W
from tests.parity import TOL, rel_err
from tests.test_oracle_remap import _vortex_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tdh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_37859_amd import tdh as T
    T.lib()
    return T


def _remap_gpu(T, cfg, src, U, dst, t=0.0):
    a = T.Context(cfg, src, U)
    a.time = t
    b = T.Context(cfg, dst, W.uniform_state(dst, cfg))
    b.remap_from(a)
    out, tb = b.get_state(), b.time
    a.close()
    b.close()
    assert tb == t
    return out


@pytest.mark.parametrize("case", ["identity", "refine_shifted", "coarsen", "outside_excision", "band_both_sides"])
def test_remap_matches_the_oracle(tdh, orc, case):
    if case == "identity":
        cfg = W.Config(dual=1)
        src, dst = W.uniform_mesh(2, 2, 2, 16, 1.0 / 32), W.uniform_mesh(4, 4, 4, 8, 1.0 / 32)
        t = 0.0
    elif case == "refine_shifted":
        cfg = W.Config(dual=1)
        src = W.uniform_mesh(2, 2, 2, 16, 1.0 / 32, bc=(0, 1, 1))
        dst = W.mixed_mesh((2, 2, 2), 32, np.eye(2, dtype=bool)[None].repeat(2, 0), 0.6 / 32,
                           x0=(0.1 / 3, 0.05, 0.0), bc=(0, 1, 1))
        t = 0.0
    elif case == "coarsen":
        cfg = W.Config()
        src, dst = W.uniform_mesh(2, 2, 2, 16, 1.0 / 32), W.uniform_mesh(2, 2, 2, 8, 1.0 / 16)
        t = 0.0
    elif case == "band_both_sides":  # larger target on both x faces and the high y face, finer, table-free
        cfg = W.Config(dual=1, rho_floor=1e-6, p_floor=1e-8)
        src = W.uniform_mesh(2, 2, 2, 8, 1.0 / 16, bc=(1, 1, 0))
        dst = W.uniform_mesh(5, 3, 2, 8, 1.0 / 24, x0=(-0.3, 0.1, 0.0), bc=(1, 1, 0))
        t = 0.0
    else:
        cfg = W.Config(dual=1, grav_kind=2, gm_bh=1.0, r_soft=0.01, r_exc=0.1, bh_x0=(0.5, 0.5, 0.5),
                       v_frame=(0.2, 0.0, 0.0), rho_floor=1e-6, p_floor=1e-8)
        src, dst = W.uniform_mesh(2, 2, 2, 8, 1.0 / 16, bc=(1, 1, 1)), W.uniform_mesh(3, 2, 2, 8, 1.0 / 16, bc=(1, 1, 1))
        t = 0.5
    U = _vortex_state(src, cfg)
    g = _remap_gpu(tdh, cfg, src, U, dst, t)
    o = orc.remap(cfg, src, U, dst, t=t)
    err = rel_err(cfg.nv, dst, g, o)
    print(case, "remap rel err", err, "bitwise", np.array_equal(g, o))
    assert np.all(err <= TOL)
    if case in ("identity", "outside_excision"):
        assert np.array_equal(g, o)


@pytest.mark.parametrize("ratio", [(0.3, 0.3, 0.3), (1.9, 1.9, 1.9), (2.0, 1.0, 0.7), (3.8, 3.8, 3.8), (4.0, 1.0, 1.0)])
@pytest.mark.parametrize("n", [8, 16, 32])
@pytest.mark.parametrize("dual", [0, 1])
def test_remap_over_spacing_ratios(tdh, orc, ratio, n, dual):
    """Target spacings of 0.3 to 4 source spacings (three taps per axis below
    1.95, four from there, the cell-by-cell kernel from 3.9), on blocks of every
    tile shape, shifted against the source and partly outside it."""
    cfg = W.Config(dual=dual, rho_floor=1e-6, p_floor=1e-8)
    src = W.mixed_mesh((2, 1, 2), 32, np.array([[[True, False]], [[False, True]]]), 1.0 / 32, bc=(0, 1, 1))
    dx = np.array(ratio) / 32
    dst = W.uniform_mesh(*[max(1, round(m / (n * r))) for m, r in zip((64, 32, 64), ratio)], n, tuple(dx),
                         x0=(0.013, -0.021, 0.37 / 32), bc=(0, 1, 1))
    U = _vortex_state(src, cfg)
    g = _remap_gpu(tdh, cfg, src, U, dst)
    err = rel_err(cfg.nv, dst, g, orc.remap(cfg, src, U, dst))
    print(ratio, n, dual, "remap rel err", err)
    assert np.all(err <= TOL)


@pytest.mark.parametrize("x0, bc", [
    ((-40.3, -17.0, -33.9), (1, 1, 1)),   # the source in the middle of the target
    ((0.2, 0.3, -60.0), (1, 1, 1)),       # from the target's low faces on
    ((-130.0, 1.0, 2.0), (1, 1, 1)),      # no target cell inside the source
    ((-50.0, 0.4, -50.0), (1, 0, 1)),     # periodic along y
])
@pytest.mark.parametrize("ratio", [0.9, 1.5, 1.9])
@pytest.mark.parametrize("dual", [0, 1])
def test_remap_onto_a_larger_domain(tdh, orc, x0, bc, ratio, dual):
    """Targets most of whose cells lie beyond the source (x0: the target's corner
    in source cells): the tiles cover only those inside, from the first whole
    tile on, and the others are floor states."""
    cfg = W.Config(dual=dual, rho_floor=1e-6, p_floor=1e-8)
    src = W.uniform_mesh(2, 3, 2, 16, 1.0 / 32, bc=bc)
    dst = W.uniform_mesh(3, 3, 3, 32, ratio / 32, x0=tuple(v / 32 for v in x0), bc=bc)
    U = _vortex_state(src, cfg)
    g = _remap_gpu(tdh, cfg, src, U, dst)
    o = orc.remap(cfg, src, U, dst)
    assert np.all(rel_err(cfg.nv, dst, g, o) <= TOL)
    floor = W.to_global(dst, cfg.nv, o)[0] == cfg.rho_floor
    assert np.array_equal(W.to_global(dst, cfg.nv, g)[0] == cfg.rho_floor, floor)


def test_galilean_boost_matches_the_oracle(tdh, orc):
    cfg = W.Config(dual=1)
    mesh = W.uniform_mesh(2, 2, 1, 16, 1.0 / 32)
    U = _vortex_state(mesh, cfg)
    V = np.array([0.3, -1.2, 2.0])
    ctx = tdh.Context(cfg, mesh, U)
    ctx.galilean_boost(V, 1.0)
    g = ctx.get_state()
    ctx.close()
    o = orc.galilean_boost(cfg, mesh, U, V, 1.0)
    assert np.all(rel_err(6, mesh, g, o) <= TOL)
    assert not np.array_equal(g, U)


def test_frame_acceleration_matches_the_oracle(tdh, orc):
    """The C5-shaped reduced debris stream with its point mass: the
    density-weighted field over dense, non-excised cells."""
    table = W.saha_table()
    cfg, mesh, U = W.debris_stream_c5(table, regions=(4, 3, 2), n_split=6, dxr=1.0)
    ctx = tdh.Context(cfg, mesh, U, table=table)
    ctx.time = 1234.5
    A = ctx.frame_acceleration(1e-6)
    ctx.close()
    o = orc.frame_acceleration(cfg, mesh, U, 1e-6, t=1234.5)
    print("frame acceleration", A, o)
    assert np.all(np.abs(A - o) <= 1e-12 * np.max(np.abs(o)))
    assert np.max(np.abs(o)) > 0
