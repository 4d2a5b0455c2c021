"""The automatic kernel choice on D3Q19: one-pass columns with edge columns in
y where 4 does not divide ny, two-pass kernels where the columns would idle;
both bitwise equal to the pinned two-pass kernels."""
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


def fields(M, model, shape):
    rR, rB = inputs.droplet(shape, min(shape) / 3.0, 1.0, 1.0)
    return (0.12 + 1.78 * rR, None) if model == "SC_MP" else (rR + 0.02, rB + 0.02)


@pytest.mark.parametrize("model", ["CG", "SC_MP", "SC_MC"])
@pytest.mark.parametrize("precision", ["FP64", "FP32", "MIXED", "FP16"])
def test_odd_rows_step_in_one_pass(M, model, precision):
    import torch
    for box, bc in (((128, 126, 128), (0, 0, 0)), ((187, 131, 190), (1, 1, 2)), ((128, 121, 150), (0, 2, 1))):
        nx, ny, nz = box
        kw = dict(lattice=M.D3Q19, model=getattr(M, model), precision=getattr(M, precision), nx=nx, ny=ny, nz=nz, bc=bc)
        kw.update(dict(G=-5.0, rho0_R=1.9, rho0_B=0.12) if model == "SC_MP" else
                  dict(A=0.02, tau_R=0.8) if model == "CG" else dict(G_RB=1.2))
        ini = fields(M, model, (nz, ny, nx))
        out = []
        for kernel in (M.KERNEL_AUTO, M.KERNEL_TWO_PASS):
            print(f"[odd rows] {model} {precision} {box} {bc} kernel={kernel}", flush=True)
            s = M.Sim(M.make_params(kernel=kernel, **kw))
            assert s.kernel_used() == (M.KERNEL_TWO_PASS if kernel else M.KERNEL_FUSED)
            s.init_equilibrium(*ini)
            assert s.step(5)[0] == M.OK
            out.append(s.export_f())
            s.close()
        assert torch.equal(*out)
        del out
        torch.cuda.empty_cache()


@pytest.mark.parametrize("box,precision,kernel", [
    ((80, 40, 152), "FP32", "TWO_PASS"), ((72, 72, 72), "FP64", "TWO_PASS"), ((100, 100, 100), "FP16", "TWO_PASS"),
    ((64, 32, 200), "MIXED", "TWO_PASS"), ((128, 128, 128), "FP32", "FUSED"), ((128, 128, 128), "MIXED", "FUSED"),
    ((176, 176, 176), "FP64", "FUSED"), ((40, 16, 8), "FP32", "FUSED"), ((128, 126, 128), "FP64", "FUSED"),
    ((150, 101, 90), "FP64", "TWO_PASS")])
def test_automatic_choice(M, box, precision, kernel):
    p = M.make_params(lattice=M.D3Q19, precision=getattr(M, precision), nx=box[0], ny=box[1], nz=box[2])
    s = M.Sim(p)
    assert s.kernel_used() == getattr(M, "KERNEL_" + kernel)
    if kernel == "FUSED":
        tx, ty, tz = s.fused_tile()
        blocks = -(-box[0] // tx) * -(-box[1] // ty) * -(-box[2] // tz)
        assert tz >= 1 and blocks >= min(128, box[2])
    s.close()
    if box[1] % 4 == 0:   # asked for, the one-pass kernel is there
        s = M.Sim(dict(p, kernel=M.KERNEL_FUSED))
        assert s.kernel_used() == M.KERNEL_FUSED
        s.close()


@pytest.mark.parametrize("lattice,precision,box,answers", [
    ("D3Q19", "FP32", (64, 64, 64), True), ("D3Q19", "FP64", (72, 72, 72), True), ("D3Q19", "MIXED", (32, 244, 53), True),
    ("D2Q9", "FP32", (17, 40000, 1), True), ("D3Q19", "FP64", (150, 101, 90), False), ("D2Q9", "FP32", (512, 512, 1), False)])
def test_columns_of_a_box_left_to_the_automatic_choice(M, lattice, precision, box, answers):
    """mclbm_fused_tile answers for every box whose one-pass kernel was there to
    choose, as for the one-pass kernel asked for, also where two passes are
    taken; pinned to the two-pass kernels it refuses."""
    nx, ny, nz = box
    kw = dict(lattice=getattr(M, lattice), precision=getattr(M, precision), nx=nx, ny=ny, nz=nz)
    s = M.Sim(M.make_params(**kw))
    assert s.kernel_used() == M.KERNEL_TWO_PASS
    if answers:
        one = M.Sim(M.make_params(kernel=M.KERNEL_FUSED, **kw))
        assert s.fused_tile() == one.fused_tile()
        one.close()
        two = M.Sim(M.make_params(kernel=M.KERNEL_TWO_PASS, **kw))
        with pytest.raises(M.MclbmError):
            two.fused_tile()
        two.close()
    else:
        with pytest.raises(M.MclbmError):
            s.fused_tile()
    s.close()


@pytest.mark.parametrize("model,precision,box,bc,kernel", [
    ("SC_MP", "FP16", (128, 88, 41), (0, 0, 0), "TWO_PASS"), ("SC_MP", "MIXED", (128, 72, 88), (1, 1, 2), "TWO_PASS"),
    ("CG", "MIXED", (96, 72, 33), (0, 0, 0), "TWO_PASS"), ("SC_MC", "FP16", (48, 64, 110), (0, 0, 0), "TWO_PASS"),
    ("CG", "FP64", (96, 48, 72), (1, 1, 2), "TWO_PASS"), ("SC_MP", "FP32", (96, 80, 44), (1, 1, 2), "TWO_PASS"),
    ("CG", "FP32", (96, 64, 56), (0, 0, 0), "FUSED"), ("SC_MC", "MIXED", (96, 72, 127), (0, 0, 0), "FUSED"),
    ("CG", "FP64", (64, 64, 66), (0, 0, 0), "FUSED"), ("SC_MP", "FP32", (64, 136, 40), (0, 0, 0), "FUSED"),
    ("SC_MP", "MIXED", (288, 56, 98), (0, 0, 0), "FUSED"), ("SC_MP", "MIXED", (288, 48, 72), (0, 0, 0), "TWO_PASS"),
    ("CG", "FP16", (96, 48, 44), (0, 0, 0), "FUSED"), ("SC_MP", "FP32", (112, 40, 44), (0, 0, 0), "FUSED"),
    ("CG", "MIXED", (128, 16, 16), (0, 0, 0), "FUSED")])
def test_batched_kernel_left_to_the_automatic_choice(M, model, precision, box, bc, kernel):
    """Batches of the classes that the batched two-pass launches step faster take
    them (128 x 88 x 41 FP16 multiphase, four of them, 47 us against 78), bitwise as
    with the one-pass kernel asked for."""
    import torch
    nx, ny, nz = box
    kw = dict(lattice=M.D3Q19, model=getattr(M, model), precision=getattr(M, precision), nx=nx, ny=ny, nz=nz, bc=bc)
    kw.update(dict(G=-5.0, rho0_R=1.9, rho0_B=0.12) if model == "SC_MP" else
              dict(A=0.02, tau_R=0.8) if model == "CG" else dict(G_RB=1.2))
    ini = fields(M, model, (nz, ny, nx))
    out = []
    for asked in ("AUTO", "FUSED"):
        s = M.Sim(M.make_params(kernel=getattr(M, "KERNEL_" + asked), **kw))
        s.init_equilibrium(*ini)
        b = M.Batch([s], [5])
        assert b.kernels() == [getattr(M, "KERNEL_" + (kernel if asked == "AUTO" else "FUSED"))]
        b.step(5)
        assert b.status()[0] == [M.DONE]
        b.close()
        out.append(s.export_f())
        s.close()
    assert torch.equal(*out)


@pytest.mark.parametrize("lattice,box", [("D3Q19", (128, 112, 96)), ("D2Q9", (700, 700, 1))])
def test_diverged_states_step_in_the_same_time(M, lattice, box):
    """A state that is bad at every node flags it once, not once per wavefront:
    two-pass steps take no more than 1.5 times those of a sound state (3 times
    with an atomic from every wavefront), and the flag is set."""
    import torch
    nx, ny, nz = box
    p = M.make_params(lattice=getattr(M, lattice), model=M.SC_MP, precision=M.FP32, nx=nx, ny=ny, nz=nz, G=-5.0,
                      rho0_R=1.9, rho0_B=0.12, kernel=M.KERNEL_TWO_PASS)
    us = []
    for bad in (False, True):
        s = M.Sim(p)
        s.init_equilibrium(*fields(M, "SC_MP", (nz, ny, nx)))
        if bad:
            s.import_f(torch.full_like(s.export_f(), float("nan")))
        s.step(4)
        t = []
        for _ in range(7):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            s.step(20)
            e[1].record()
            e[1].synchronize()
            t.append(e[0].elapsed_time(e[1]) / 20 * 1e3)
        us.append(min(t))
        assert s.diverged() == bad
        s.close()
    print(f"[diverged] {lattice} {box} sound {us[0]:.1f} diverged {us[1]:.1f} us", flush=True)
    assert us[1] <= 1.5 * us[0]
