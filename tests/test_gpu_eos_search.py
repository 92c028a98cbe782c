"""The table search without a seed, from its bin's start cell, on tables where
the start is far off (rows that differ by more than their own range, jumps,
the smallest table) and on every kind of target: inside, on the nodes, out of
range, infinite.  The cell and log T equal those of a full search of the
density-interpolated column, formed with the same operations; a batch's
pressures and sound speeds follow the table."""
import numpy as np
import pytest

from paper_2609_37859_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tdh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_37859_amd import tdh as T
    T.lib()
    return T


def _table(name):
    rng = np.random.default_rng(2)
    if name == "smallest":
        le = np.array([[0.0, 1.0], [3.0, 3.5]])
    elif name == "rows_apart":  # rows shifted by more than their range, one of them nearly flat
        le = np.cumsum(rng.uniform(0.01, 0.1, (5, 40)), axis=1) + np.array([0.0, 9.0, -4.0, 2.0, 2.1])[:, None]
        le[3] = 2.0 + 1e-9 * np.arange(40)
    elif name == "jumps":  # cells whose widths differ by twelve decades
        le = np.cumsum(10.0 ** rng.uniform(-11, 1, (4, 100)), axis=1)
    else:  # smooth
        le = 12.0 + np.linspace(0, 4, 64)[None, :] + 0.02 * np.arange(6)[:, None]
    n, m = le.shape
    return W.EosTable(n, m, -6.0, 0.7, 3.0, 0.1, le + 0.5, np.ascontiguousarray(le), le - 0.1, 0.0)


def _search(t, lr, le):
    """(cell, log T): the largest node of the column not above the target."""
    x = (np.clip(lr, t.lr0, t.lr0 + (t.nrho - 1) * t.dlr) - t.lr0) * (1.0 / t.dlr)
    i = np.clip(np.floor(x).astype(int), 0, t.nrho - 2)
    w = x - i
    col = (1.0 - w)[:, None] * t.le[i] + w[:, None] * t.le[i + 1]
    le = np.minimum(np.maximum(le, col[:, 0]), col[:, -1])
    j = np.clip((col <= le[:, None]).sum(1) - 1, 0, t.nT - 2)
    q = np.arange(len(j))
    return j, t.lT0 + (j + (le - col[q, j]) / (col[q, j + 1] - col[q, j])) * t.dlT


@pytest.mark.parametrize("name", ["smallest", "rows_apart", "jumps", "smooth"])
def test_search_without_a_seed(tdh, name):
    import torch
    t = _table(name)
    cfg = W.Config(eos_kind=1)
    mesh = W.uniform_mesh(1, 1, 1, 8, 1.0)
    ctx = tdh.Context(cfg, mesh, W.uniform_state(mesh, W.Config()), table=t)
    rng = np.random.default_rng(9)
    n = 4001
    lr = rng.uniform(t.lr0 - 0.5, t.lr0 + t.nrho * t.dlr, n)
    le = rng.uniform(t.le.min() - 0.5, t.le.max() + 0.5, n)
    on = rng.integers(0, t.nrho, n // 2)  # exactly on a node
    lr[:n // 2] = t.lr0 + on * t.dlr
    le[:n // 2] = t.le[on, rng.integers(0, t.nT, n // 2)]
    le[-2:] = np.inf, -np.inf
    j, lT = _search(t, lr, le)
    for mode in (0, 2):
        glT, gj, it = ctx.eos_invert(torch.from_numpy(lr), torch.from_numpy(le), mode=mode)
        assert np.array_equal(gj.cpu().numpy(), j)
        assert np.array_equal(glT.cpu().numpy(), lT)
        assert bool((it == (-1 if mode == 0 else 0)).all())
    ctx.close()


@pytest.mark.parametrize("n", [1, 255, 256, 257, 512, 513, 2048 * 512 + 1])
def test_eval_batch_sizes(tdh, n):
    """Every query of a batch is answered, whatever workgroup share it falls in.
    log P = log e + 1/2 and log c_s^2 = log e - 1/10 on the whole table, so P and
    c_s are known; the logarithm, the interpolation and the power each round a
    value below 20 a few times: 1e-13 relative covers ln 10 times 10 ulp of 16."""
    import torch
    t = _table("smooth")
    mesh = W.uniform_mesh(1, 1, 1, 8, 1.0)
    ctx = tdh.Context(W.Config(eos_kind=1), mesh, W.uniform_state(mesh, W.Config()), table=t)
    rng = np.random.default_rng(n)
    rho = 10.0 ** rng.uniform(-6.0, -2.6, n)
    e = 10.0 ** rng.uniform(12.2, 15.9, n)
    P, cs = (x.cpu().numpy() for x in ctx.eos_eval(torch.from_numpy(rho), torch.from_numpy(rho * e)))
    assert np.max(np.abs(P / (e * 10.0 ** 0.5) - 1.0)) < 1e-13
    assert np.max(np.abs(cs / np.sqrt(e * 10.0 ** -0.1) - 1.0)) < 1e-13
    ctx.close()


@pytest.mark.parametrize("n", [2 ** 19 - 1, 2 ** 19, 2 ** 19 + 257])
def test_eval_either_side_of_two_queries_per_thread(tdh, n):
    """The same bits from one query per thread and from two: the batch against
    its pieces of less than half the size."""
    import torch
    t = _table("smooth")
    mesh = W.uniform_mesh(1, 1, 1, 8, 1.0)
    ctx = tdh.Context(W.Config(eos_kind=1), mesh, W.uniform_state(mesh, W.Config()), table=t)
    rng = np.random.default_rng(n)
    rho = torch.from_numpy(10.0 ** rng.uniform(-6.5, -2.0, n))
    U = rho * torch.from_numpy(10.0 ** rng.uniform(11.5, 16.5, n))
    whole = ctx.eos_eval(rho, U)
    pieces = [ctx.eos_eval(r, u) for r, u in zip(rho.split(200001), U.split(200001))]
    for k in range(2):
        assert torch.equal(whole[k], torch.cat([p[k] for p in pieces]))
    ctx.close()


def test_table_buffer_without_start_cells(tdh, saha):
    """A buffer that holds the table but not the start cells: every search starts in
    the middle, with the same answers; a smaller one is refused."""
    import ctypes as C
    import torch
    cfg = W.Config(eos_kind=1, dual=1, rho_floor=1e-12, p_floor=0.0, e_floor=saha.e_floor)
    mesh = W.uniform_mesh(2, 1, 1, 8, 1e10)
    rho = np.geomspace(1e-9, 1e-5, 8)

    def fn(x, y, z):
        r = rho[(np.floor(x / 1e10).astype(int)) % 8] + 0 * y + 0 * z
        u = r * W.saha_pe(r, 2e4 + 0 * r)[1]
        return [r, 0 * r, 0 * r, 0 * r, u, u]

    U = W.pack_state(mesh, 6, fn)
    x = torch.from_numpy(W.seed_training_samples(saha, 5001, 4))
    lr, le = x[:, 0].contiguous(), x[:, 1].contiguous()
    full = tdh.lib().tdh_table_bytes(saha.nrho, saha.nT)
    least = full - (4 * (saha.nrho - 1) * saha.nT + 7) // 8 * 8
    buf = torch.zeros(full, dtype=torch.uint8, device="cuda")
    arrs = [np.ascontiguousarray(a) for a in (saha.lP, saha.le, saha.lc2)]
    out = []
    for nbytes in (full, least, least - 8):
        ctx = tdh.Context(cfg, mesh, U, table=saha, inv_mode=3)
        rc = ctx.L.tdh_set_eos_table(ctx.ctx, saha.nrho, saha.nT, saha.lr0, saha.dlr, saha.lT0, saha.dlT,
                                     *(a.ctypes.data_as(C.POINTER(C.c_double)) for a in arrs), buf.data_ptr(), nbytes)
        if nbytes < least:
            assert rc == -2  # TDH_ENOMEM
        else:
            assert rc == 0
            _, dt, _, _ = ctx.reduce_dt()
            ctx.step_level(0, dt)
            inv = ctx.eos_invert(lr, le, mode=0)
            pc = ctx.eos_eval(10.0 ** lr, 10.0 ** (lr + le))
            out.append([dt, ctx.get_state()] + [t.cpu().numpy() for t in inv + pc])
        ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
