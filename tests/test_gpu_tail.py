"""Single-workgroup tail V-cycle (cs_set_tail): the coarse levels of at most a
few thousand rows run Alg. 1 as one launch with workgroup barriers between the
steps.  Each row's arithmetic is the per-level kernels' own, in the same
order, so V-cycles and whole solves must be bit-identical with the tail on and
off - for point and block levels, every right-hand-side count, both working
precisions, a batch whose systems end on different levels (direct segments on
intermediate levels), graph replay, and the allocation-free entry point (which
always runs the per-level launches)."""
import numpy as np
import pytest

from synth import fd
from synth.batch import concatenate

pytestmark = pytest.mark.gpu


def _vcycle(s, b, tail):
    s.set_tail(tail)
    return s.vcycle(b).cpu().numpy()


def _check_vcycle(s, b, label):
    s.set_tail(4096)
    m, first = s.tail()
    assert m == 4096 and first >= 0, (label, first)   # the tail is in use
    x0 = _vcycle(s, b, 0)
    x1 = _vcycle(s, b, 4096)
    x2 = _vcycle(s, b, 4096)   # the table is reused
    print(f"[tail] {label}: tail from level {first} of {len(s.sizes)}, |x| {np.linalg.norm(x0):.6e}")
    np.testing.assert_array_equal(x1, x0)
    np.testing.assert_array_equal(x2, x0)
    return first


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nrhs", [1, 2, 4, 8])
def test_tail_vcycle_blocks8_3d(gpu_lib, precision, nrhs):
    p = fd.interface3d(32, nrhs=nrhs)
    s = gpu_lib.Solver(p.levels)
    s.setup(depth=3, precision=precision)
    _check_vcycle(s, p.rhs, f"interface3d_32 nb=8 {precision} nrhs={nrhs}")
    s.setup(depth=2, order="FF", n_pre=2, n_post=1, precision=precision)
    _check_vcycle(s, p.rhs, f"interface3d_32 FF V(2,1) {precision} nrhs={nrhs}")
    s.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_tail_vcycle_points_2d(gpu_lib, precision):
    p = fd.poisson2d(64, nrhs=2)   # levels of 4096, 1024, 256, 64 and 16 rows
    s = gpu_lib.Solver(p.levels)
    s.setup(depth=3, precision=precision)
    assert _check_vcycle(s, p.rhs, f"poisson2d_64 {precision}") == 0   # the whole V-cycle in one launch
    s.set_tail(1024)
    assert s.tail()[1] == 1
    x0 = _vcycle(s, p.rhs, 0)
    np.testing.assert_array_equal(_vcycle(s, p.rhs, 1024), x0)
    for method in ("ir", "cg"):   # with the tail from level 0 the refinement issues no early sweep
        s.set_tail(0)
        xa, ia = s.solve(p.rhs, rtol=1e-10, maxit=100, method=method)
        s.set_tail(4096)
        xb, ib = s.solve(p.rhs, rtol=1e-10, maxit=100, method=method)
        assert ib["iterations"] == ia["iterations"]
        np.testing.assert_array_equal(xb.cpu().numpy(), xa.cpu().numpy())
        np.testing.assert_array_equal(ib["history"], ia["history"])
    s.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_tail_vcycle_2d_blocks4(gpu_lib, precision):
    rng = np.random.default_rng(7)
    levels = fd.fv_hierarchy(np.exp(rng.standard_normal((64, 64))), bs=2, n_stop=4)
    b = rng.standard_normal((64 * 64, 2))
    s = gpu_lib.Solver(levels)
    s.setup(depth=2, precision=precision)
    _check_vcycle(s, b, f"lognormal 64^2 blocks 2x2 {precision}")
    s.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_tail_solves_identical(gpu_lib, precision):
    p = fd.interface3d(32, nrhs=4)
    s = gpu_lib.Solver(p.levels)
    s.setup(depth=3, precision=precision)
    for method in ("ir", "cg"):
        s.set_tail(0)
        x0, i0 = s.solve(p.rhs, rtol=1e-10, maxit=200, method=method)
        s.set_tail(4096)
        x1, i1 = s.solve(p.rhs, rtol=1e-10, maxit=200, method=method)
        assert i1["iterations"] == i0["iterations"]
        np.testing.assert_array_equal(x1.cpu().numpy(), x0.cpu().numpy())
        np.testing.assert_array_equal(i1["history"], i0["history"])
        print(f"[tail] solve {precision} {method}: {i0['iterations']} it, "
              f"{i0['solve_ms']:.2f} ms per-level, {i1['solve_ms']:.2f} ms tail")
    s.close()


def test_tail_batch_with_direct_segments(gpu_lib):
    sizes = [48, 64, 80, 16, 112, 32, 80, 8]
    bt = concatenate(fd.lognormal_batch(len(sizes), nrhs=4, sizes=sizes, config_id=14))
    s = gpu_lib.Solver(bt.levels)
    s.setup(depth=3, precision="fp32")
    s.set_systems(bt.sys_ptr)
    _check_vcycle(s, bt.rhs, "batch of 8 lognormal2d")
    s.set_tail(0)
    x0, i0 = s.solve(bt.rhs, rtol=1e-10, maxit=300, method="ir")
    st0 = s.system_stats()
    s.set_tail(4096)
    x1, i1 = s.solve(bt.rhs, rtol=1e-10, maxit=300, method="ir")
    st1 = s.system_stats()
    np.testing.assert_array_equal(x1.cpu().numpy(), x0.cpu().numpy())
    np.testing.assert_array_equal(st1[0], st0[0])
    np.testing.assert_array_equal(st1[1], st0[1])
    s.close()


def test_tail_with_graphs_and_noalloc(gpu_lib):
    p = fd.interface3d(32, nrhs=4)
    s = gpu_lib.Solver(p.levels)
    s.setup(depth=3, precision="fp32")
    s.set_tail(4096)
    import torch
    b = torch.as_tensor(p.rhs, device="cuda").contiguous()
    x0 = s.vcycle(b).cpu().numpy()
    xn = s.vcycle_noalloc(b, torch.empty_like(b)).cpu().numpy()   # per-level launches on the static array
    np.testing.assert_array_equal(xn, x0)
    x1 = s.vcycle(b).cpu().numpy()               # back on the context's buffers: table rebuilt
    np.testing.assert_array_equal(x1, x0)
    s.set_tail(0)
    s.set_graphs(False)
    xe, ie = s.solve(p.rhs, rtol=1e-10, maxit=200, method="ir")
    s.set_tail(4096)
    s.set_graphs(True)
    for _ in range(2):
        xg, ig = s.solve(p.rhs, rtol=1e-10, maxit=200, method="ir")
        assert ig["iterations"] == ie["iterations"]
        np.testing.assert_array_equal(xg.cpu().numpy(), xe.cpu().numpy())
    s.set_graphs(False)
    s.close()


def test_tail_settings(gpu_lib):
    p = fd.interface3d(32, nrhs=1)              # levels of 32768, 4096, 512 and 64 rows
    s = gpu_lib.Solver(p.levels)
    assert s.tail() == (0, -1)                 # off by default; no setup yet
    s.setup(depth=2)
    assert s.tail()[1] == -1
    s.set_tail(4096)
    assert s.tail()[1] == 1
    s.set_tail(1000)
    assert s.tail()[1] == 2
    s.set_tail(100)                             # only the bottom level is that small
    assert s.tail()[1] == -1
    s.set_tail(0)
    assert s.tail() == (0, -1)
    with pytest.raises(Exception, match="tail max_rows"):
        s.set_tail(-1)
    with pytest.raises(Exception, match="tail max_rows"):
        s.set_tail(1 << 20)
    s.close()


def test_autotune_picks_the_fastest_tail(gpu_lib):
    p = fd.poisson2d(64, nrhs=1)
    s = gpu_lib.Solver(p.levels)
    s.setup(depth=3, n_pre=2, n_post=2, precision="fp64")
    x0, i0 = s.solve(p.rhs, rtol=1e-10, maxit=100)
    s.autotune(1)
    cand = s.tail_candidates()
    rows, first = s.tail()
    print(f"[tail] autotune 64^2 V(2,2): {[(r, round(t, 4)) for r, t in cand]} -> max_rows {rows}, level {first}")
    assert cand[0][0] == 0 and len(cand) >= 2 and all(t > 0 for _, t in cand)
    assert rows == min(cand, key=lambda c: c[1])[0]
    x1, i1 = s.solve(p.rhs, rtol=1e-10, maxit=100)
    assert i1["iterations"] == i0["iterations"]
    np.testing.assert_array_equal(x1.cpu().numpy(), x0.cpu().numpy())
    s.close()


@pytest.mark.parametrize("family,n,nrhs,precision", [
    ("multiphase3d", 16, 2, "fp64"),    # 27-point rows (streamed), trilinear transfers, blocks of 8
    ("multiphase3d", 12, 1, "fp32"),
    ("stokes", 32, 1, "fp32"),          # saddle point, blocks of 4, up to 15 entries per row
    ("stokes", 24, 4, "fp64"),
    ("lognormal", 72, 8, "fp64"),       # 5184 rows: more than the registers hold, odd bottom (9^2)
    ("lognormal", 80, 1, "fp32"),
    ("interface", 28, 8, "fp32"),       # 21952 rows do not fit: starts at 2744, odd bottom (7^3)
    ("interface", 20, 2, "fp64"),
    ("poisson", 16, 1, "fp64"),         # a single tile per level
])
def test_tail_general_transfers_and_sizes(gpu_lib, family, n, nrhs, precision):
    """Hierarchies with general transfers, rows longer than the kernel holds in
    registers, row counts off its tiles and levels beyond the LDS."""
    from synth import fe, stokes
    rng = np.random.default_rng(n)
    levels = {"multiphase3d": lambda: fe.multiphase3d(n).levels, "stokes": lambda: stokes.mac2d(n).levels,
              "lognormal": lambda: fd.lognormal2d(n).levels, "interface": lambda: fd.interface3d(n).levels,
              "poisson": lambda: fd.poisson2d(n).levels}[family]()
    b = rng.standard_normal((levels[0].n, nrhs))
    s = gpu_lib.Solver(levels)
    s.setup(depth=3, order="FF" if family == "stokes" else "RF", n_pre=2, precision=precision)
    s.set_tail(65536)
    m, first = s.tail()
    assert m == 65536 and 0 <= first < len(levels) - 1
    x1 = s.vcycle(b).cpu().numpy()
    s.set_tail(0)
    np.testing.assert_array_equal(s.vcycle(b).cpu().numpy(), x1)
    s.close()


def test_tail_systems_of_ragged_sizes(gpu_lib):
    """A batch whose systems' rows straddle slices and end on different levels,
    each in its own workgroup, and the same rows declared one system."""
    bt = concatenate(fd.lognormal_batch(5, nrhs=2, sizes=[24, 40, 16, 56, 8], config_id=15))
    s = gpu_lib.Solver(bt.levels)
    s.setup(depth=2, precision="fp64")
    x0 = s.vcycle(bt.rhs).cpu().numpy()
    for sys_ptr in (None, bt.sys_ptr):
        s.set_systems(sys_ptr)
        s.set_tail(65536)
        assert s.tail()[1] >= 0
        np.testing.assert_array_equal(s.vcycle(bt.rhs).cpu().numpy(), x0)
    s.close()


def _nine_point_blocks(grids):
    """Levels of 16x16 blocks on g x g grids with nine-point block coupling (rows
    of 4, 6 and 9 blocks), four colours, 2x2 aggregation between the grids."""
    import scipy.sparse as sp

    from synth.problem import Level
    from synth.rng import TEST, stream
    rng = stream(31, TEST, grids[0])
    near = rng.uniform(-1, 1, size=(16, 16)) / 64
    diag = 2.0 * np.eye(16) + rng.uniform(-1, 1, size=(16, 16)) / 16
    levels = []
    for l, g in enumerate(grids):
        t = sp.diags([1.0, 1.0, 1.0], [-1, 0, 1], shape=(g, g))
        nine = sp.kron(t, t)
        A = sp.kron(nine - sp.eye(g * g), near) + sp.kron(sp.eye(g * g), diag)
        colour = (2 * (np.arange(g)[:, None] % 2) + np.arange(g)[None, :] % 2).astype(np.int32).ravel()
        P = None
        if l + 1 < len(grids):
            a = sp.csr_matrix((np.ones(g), (np.arange(g), np.arange(g) // 2)), shape=(g, g // 2))
            P = sp.csr_matrix(sp.kron(sp.kron(a, a), sp.eye(16)))
        levels.append(Level(sp.csr_matrix(A), 16, P, 0.25, colour))
    return levels


# 2 to 12 blocks a side: colours of 1 to 36 rows for 16 wavefronts
@pytest.mark.parametrize("order,n_pre,n_post,depth", [("FF", 1, 1, 3), ("RF", 1, 1, 2), ("RF", 2, 1, 1)])
@pytest.mark.parametrize("blocks,grids", [("sipg", (8,)), ("sipg", (12,)), ("nine_point", (2, 1)), ("nine_point", (4, 2)),
                                          ("nine_point", (8, 4, 2)), ("nine_point", (12, 6, 3))])
def test_tail_bf16_multicoloured(gpu_lib, blocks, grids, order, n_pre, n_post, depth):
    """The BF16 multicoloured levels in one launch: bit-identical with a launch
    per colour step, from a whole cycle or its coarse part, in a solve and under
    graph replay; more right-hand sides take the per-level launches."""
    from synth import dg
    levels = dg.sipg_q3(grids[0]).levels if blocks == "sipg" else _nine_point_blocks(grids)
    s = gpu_lib.Solver(levels)
    s.setup(depth=depth, mode="multiplicative", order=order, n_pre=n_pre, n_post=n_post, ridge=1e-3, precision="bf16")
    b = np.random.default_rng(5).uniform(-1, 1, size=(levels[0].n, 1))
    x0 = _vcycle(s, b, 0)
    for l, lv in enumerate(levels[:-1]):
        x1 = _vcycle(s, b, lv.n)
        assert s.tail() == (lv.n, l)
        np.testing.assert_array_equal(x1, x0)
        np.testing.assert_array_equal(_vcycle(s, b, lv.n), x0)
    kw = dict(rtol=1e-8, maxit=6, raise_on_noconv=False)
    s.set_tail(0)
    xa, ia = s.solve(b, **kw)
    b2 = np.hstack([b, 2 * b])
    y0 = s.vcycle(b2).cpu().numpy()
    s.set_tail(levels[0].n)
    np.testing.assert_array_equal(s.vcycle(b2).cpu().numpy(), y0)
    for graphs in (False, True):
        s.set_graphs(graphs)
        for _ in range(3):
            xb, ib = s.solve(b, **kw)
            assert ib["iterations"] == ia["iterations"]
            np.testing.assert_array_equal(xb.cpu().numpy(), xa.cpu().numpy())
    s.close()


@pytest.mark.parametrize("tail", [0, 4096])
def test_right_hand_side_counts_with_a_tail(gpu_lib, tail):
    """A V-cycle that is one tail launch refuses the counts that the per-level
    launches refuse."""
    p = fd.poisson2d(64)
    s = gpu_lib.Solver(p.levels)
    s.setup(depth=2)
    s.set_tail(tail)
    for nrhs in (3, 5, 16):
        with pytest.raises(gpu_lib.CascadeError, match="nrhs must be 1, 2, 4 or 8"):
            s.vcycle(np.ones((p.n, nrhs)))
    s.close()


def test_tail_level_is_reported_for_the_right_hand_sides_in_use(gpu_lib):
    """The BF16 multicoloured tail takes one right-hand side: with two the
    V-cycle runs per-level launches, and cs_get_tail says so."""
    from synth import dg
    levels = dg.sipg_q3(12).levels
    s = gpu_lib.Solver(levels)
    s.setup(depth=2, mode="multiplicative", order="FF", ridge=1e-3, precision="bf16")
    s.set_tail(levels[0].n)
    b = np.random.default_rng(3).uniform(-1, 1, size=(levels[0].n, 2))
    assert s.tail() == (levels[0].n, 0)      # no V-cycle yet: one
    for nrhs, first in ((2, -1), (1, 0)):
        s.trace(("tail",))
        s.vcycle(b[:, :nrhs])
        s.trace(())
        assert s.tail() == (levels[0].n, first)
        assert (s.trace_read()["tail"]["launches"] > 0) == (first == 0)
    s.close()


@pytest.mark.parametrize("family", ["points", "bf16"])
def test_tail_of_one_solver_beside_a_smaller_one(gpu_lib, family):
    """Two live solvers whose tails run the same kernel: the second one's, with
    less LDS, does not take the first one's away."""
    def make(n):
        if family == "points":
            p = fd.poisson2d(n)
            return p.levels, p.rhs, dict(depth=2)
        from synth import dg
        p = dg.sipg_q3(n)
        return p.levels, p.rhs, dict(depth=2, mode="multiplicative", order="FF", ridge=1e-3, precision="bf16")
    solvers = []
    for n in ((64, 16) if family == "points" else (12, 8)):
        levels, b, opts = make(n)
        s = gpu_lib.Solver(levels)
        s.setup(**opts)
        x0 = _vcycle(s, b[:, :1], 0)
        np.testing.assert_array_equal(_vcycle(s, b[:, :1], levels[0].n), x0)
        assert s.tail()[1] == 0
        solvers.append((s, b[:, :1], x0))
    for s, b, x0 in solvers:
        np.testing.assert_array_equal(s.vcycle(b).cpu().numpy(), x0)
        s.close()


@pytest.mark.parametrize("n,precision,first", [
    (12, "fp64", 0),     # 460 KB of A at level 0
    (16, "fp32", 0),     # 760 KB
    (16, "fp64", 1),     # 1,140 KB: from 512 rows
    (24, "fp32", 1),     # 307 KB at level 1
    (24, "fp64", -1),    # 460 KB there, and nothing below it to smooth
    (32, "fp32", 2),     # 760 KB at level 1: from 512 rows
])
def test_tail_covers_streamed_levels_up_to_a_size(gpu_lib, n, precision, first):
    """Long rows under general transfers: covered while one CU keeps up with a
    launch per step, whatever larger limit is set."""
    from synth import fe
    levels = fe.multiphase3d(n).levels
    b = np.random.default_rng(n).standard_normal((levels[0].n, 2))
    s = gpu_lib.Solver(levels)
    s.setup(depth=2, precision=precision)
    s.set_tail(4096)
    assert s.tail() == (4096, first)
    x1 = s.vcycle(b).cpu().numpy()
    s.set_tail(0)
    np.testing.assert_array_equal(s.vcycle(b).cpu().numpy(), x1)
    s.close()
