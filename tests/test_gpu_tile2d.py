"""Small D2Q9 boxes with the kernel left to the library: one launch per step,
or per two steps where the box is periodic and small, over tiles.  Results are
the two-pass kernels' bit for bit, for any number of steps between checks."""
import numpy as np
import pytest

from paper_2110_05197_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_05197_amd as M
    M.lib()
    return M


def make(M, model, prec, nx, ny, bc, kernel, cons=0):
    shape = (1, ny, nx)
    rng = np.random.default_rng(nx * 1000 + ny)
    rR, rB = inputs.droplet(shape, max(1.0, min(nx, ny) / 4.0), 1.0, 1.0)
    u = 0.01 * rng.standard_normal((3,) + shape)
    u[2] = 0.0
    kw = dict(lattice=M.D2Q9, model=model, precision=prec, nx=nx, ny=ny, nz=1, bc=bc, kernel=kernel)
    if model == M.CG:
        p = M.make_params(A=0.02, rho0_R=1.0, rho0_B=1.0, tau_R=0.8, conserve_mass=cons, **kw)
    elif model == M.SC_MP:
        p = M.make_params(G=-5.0, rho0_R=1.9, rho0_B=0.12, **kw)
        rR, rB = 0.12 + 1.78 * rR, None
    else:
        p = M.make_params(G_RB=1.2, **kw)
        rR, rB = 0.1 + rR, 0.1 + rB
    s = M.Sim(p)
    s.init_equilibrium(rR, rB, u)
    return s


SIZES = [(2, 2), (3, 5), (8, 8), (9, 17), (16, 4), (64, 64), (100, 75), (130, 126), (129, 131), (187, 203), (370, 400)]


@pytest.mark.parametrize("model,prec,cons", [("CG", 0, 0), ("CG", 1, 0), ("CG", 1, 1), ("CG", 2, 1), ("CG", 3, 0),
                                             ("SC_MP", 0, 0), ("SC_MP", 3, 0), ("SC_MC", 1, 0), ("SC_MC", 2, 0)])
def test_tiles_equal_two_pass_bitwise(M, model, prec, cons):
    m = getattr(M, model)
    for nx, ny in SIZES:
        for bc in ((0, 0, 0), (0, 1, 0), (1, 2, 0)):
            for runs in ((1, 2, 3), (4, 9), (11,)):   # steps between exports
                print(f"[tile2d] {model} prec={prec} {nx}x{ny} bc={bc} runs={runs}", flush=True)
                a = make(M, m, prec, nx, ny, bc, M.KERNEL_AUTO, cons)
                b = make(M, m, prec, nx, ny, bc, M.KERNEL_TWO_PASS, cons)
                assert a.kernel_used() == M.KERNEL_TWO_PASS
                for n in runs:
                    assert a.step(n) == (M.OK, n)
                    b.step(n)
                    fa, fb = a.export_f().cpu().numpy(), b.export_f().cpu().numpy()
                    assert np.array_equal(fa, fb, equal_nan=True)
                a.close()
                b.close()


def test_tiles_stop_at_checks_and_flag_divergence(M):
    """check_every splits the runs; a state gone bad inside a two-step launch
    is seen although the launch that flags it has moved on."""
    a = make(M, M.CG, M.FP64, 40, 24, (0, 0, 0), M.KERNEL_AUTO)
    b = make(M, M.CG, M.FP64, 40, 24, (0, 0, 0), M.KERNEL_TWO_PASS)
    assert a.step(23, check_every=5) == (M.OK, 23) and b.step(23) == (M.OK, 23)
    assert np.array_equal(a.export_f().cpu().numpy(), b.export_f().cpu().numpy())
    assert a.observables()["step"] == 23
    for s in (a, b):
        f = s.export_f()
        f[0, 0, 0, 3, 5] = float("nan")
        s.import_f(f)
        assert s.step(8, check_every=4) == (M.DIVERGED, 4)
        assert s.diverged()
        s.close()


def test_tile_steps_captured_in_a_graph(M):
    """An even number of captured steps leaves the buffers as they were, so
    that the graph replays: equal to eager two-pass steps after each replay."""
    import torch
    stream = torch.cuda.Stream()
    for k in (2, 6, 8):
        a = make(M, M.CG, M.FP32, 64, 48, (0, 0, 0), M.KERNEL_AUTO)
        a.close()
        with torch.cuda.stream(stream):
            a = make(M, M.CG, M.FP32, 64, 48, (0, 0, 0), M.KERNEL_AUTO)
        b = make(M, M.CG, M.FP32, 64, 48, (0, 0, 0), M.KERNEL_TWO_PASS)
        with torch.cuda.stream(stream):
            a.step(4)
        stream.synchronize()
        b.step(4)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            a.step(k)
        for _ in range(3):
            g.replay()
            torch.cuda.synchronize()
            b.step(k)
            assert np.array_equal(a.export_f().cpu().numpy(), b.export_f().cpu().numpy())
        a.close()
        b.close()


THIN = [(2, 37184, 2, (0, 0, 0)), (4, 44370, 0, (0, 1, 0)), (6, 60668, 3, (1, 2, 0)), (8, 53035, 2, (0, 0, 0)),
        (15, 6380, 2, (0, 1, 0)), (16, 25965, 0, (0, 1, 0)), (20, 16135, 2, (0, 1, 0))]
NOT_THIN = [(28, 1759, 1, (0, 1, 0)), (40, 8856, 0, (0, 1, 0)), (38709, 2, 2, (0, 1, 0)), (6, 11636, 3, (0, 0, 0))]


@pytest.mark.parametrize("nx,ny,prec,bc", THIN + NOT_THIN)
def test_thin_boxes(M, nx, ny, prec, bc):
    """Boxes a few nodes wide leave a tile's lanes idle: the two-pass launches'
    results bit for bit, at no more than 1.25 times their time (tiles whatever
    the width took 1.3-9 times as long on the first list)."""
    import torch
    a = make(M, M.CG, prec, nx, ny, bc, M.KERNEL_AUTO)
    b = make(M, M.CG, prec, nx, ny, bc, M.KERNEL_TWO_PASS)
    for n in (1, 6):
        a.step(n)
        b.step(n)
        assert np.array_equal(a.export_f().cpu().numpy(), b.export_f().cpu().numpy())
    us = ([], [])
    for _ in range(7):
        for s, t in zip((a, b), us):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            s.step(80)
            e[1].record()
            e[1].synchronize()
            t.append(e[0].elapsed_time(e[1]) / 80 * 1e3)
    print(f"[thin] {nx}x{ny} prec={prec} auto {min(us[0]):.1f} two-pass {min(us[1]):.1f} us", flush=True)
    assert min(us[0]) <= 1.25 * min(us[1])
    a.close()
    b.close()
