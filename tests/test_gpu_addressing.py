"""Lattices on both sides of the line where the arrays of one colour span
4 GB: below it the step kernels address populations through buffer resources
with 32-bit byte offsets, from there on through 64-bit pointers.  A droplet
block at the highest node offsets must evolve bit for bit as the same block in
a 64^3 (64^2) box: after 5 steps no node of it depends on anything beyond 10
nodes from it."""
import gc

import numpy as np
import pytest

from paper_2110_05197_amd import inputs

pytestmark = pytest.mark.gpu
B, STEPS = 32, 5
ONE, TWO = 2, 1   # one-pass and two-pass kernels


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_05197_amd as M
    M.lib()
    return M


def run(M, kw, box, at, via):
    import torch
    nz, ny, nx = box
    z0, y0, x0 = at
    two_d = nz == 1
    p = M.make_params(nx=nx, ny=ny, nz=nz, **kw)
    one = p["model"] == M.SC_MP
    rR, rB = inputs.droplet((1, B, B) if two_d else (B, B, B), 6.0, *((1.9, 0.15) if one else (1.0, 1.0)))
    blocks = [rR + rB] if one else [rR, rB]
    fields = []
    for blk, amb in zip(blocks, (0.15,) if one else (0.0, 1.0)):
        f = torch.full(box, amb, dtype=torch.float64, device="cuda")
        f[z0:z0 + (1 if two_d else B), y0:y0 + B, x0:x0 + B] = torch.from_numpy(blk).cuda()
        fields.append(f)
    s = M.Sim(p)
    s.init_equilibrium(*fields)
    del fields
    if via == "batch":
        b = M.Batch([s], [STEPS])
        b.step(STEPS, use_graph=False)
        b.status()
        kernel = b.kernels()[0]
        b.close()
    else:
        s.step(STEPS)
        kernel = s.kernel_used()
    words, word_bytes, _ = M.population_stride(p)
    far = (9 if two_d else 19) * words * word_bytes >= 2 ** 32
    rho = s.moments()[0]
    out = rho[z0:z0 + (1 if two_d else B), y0:y0 + B, x0:x0 + B].cpu().numpy()
    s.close()
    del rho, s
    gc.collect()
    torch.cuda.empty_cache()
    return out, kernel, far


CASES = [  # lattice, model, precision, box (nz, ny, nx), far, kernel, boundaries, via
    ("D3Q19", "CG", "FP64", (296, 296, 320), False, ONE, (0, 0, 0), "solo"),
    ("D3Q19", "CG", "FP64", (296, 296, 320), False, TWO, (0, 0, 0), "solo"),
    ("D3Q19", "CG", "FP64", (296, 304, 320), True, ONE, (0, 0, 0), "solo"),
    ("D3Q19", "CG", "FP64", (296, 304, 320), True, TWO, (1, 1, 0), "solo"),
    ("D3Q19", "CG", "FP64", (296, 304, 320), True, ONE, (0, 0, 0), "batch"),
    ("D3Q19", "CG", "FP64", (296, 304, 320), True, TWO, (0, 0, 0), "batch"),
    ("D3Q19", "SC_MP", "FP32", (376, 384, 384), False, ONE, (1, 1, 0), "solo"),
    ("D3Q19", "SC_MP", "FP32", (388, 384, 384), True, ONE, (1, 1, 0), "solo"),
    ("D3Q19", "SC_MP", "FP32", (388, 384, 384), True, TWO, (0, 0, 0), "solo"),
    ("D2Q9", "CG", "FP64", (1, 7700, 7600), False, ONE, (0, 0, 0), "solo"),
    ("D2Q9", "CG", "FP64", (1, 7700, 7900), True, ONE, (0, 0, 0), "solo"),
    ("D2Q9", "CG", "FP64", (1, 7700, 7900), True, TWO, (0, 0, 0), "batch"),
]


@pytest.mark.parametrize("lattice,model,precision,box,far,kernel,bc,via", CASES)
def test_block_at_the_top_of_the_address_range(M, lattice, model, precision, box, far, kernel, bc, via):
    print(f"[addressing] {lattice} {model} {precision} {box} kernel {kernel} bc {bc} {via}", flush=True)
    kw = dict(lattice=getattr(M, lattice), model=getattr(M, model), precision=getattr(M, precision), bc=bc,
              kernel=kernel)
    kw.update(dict(G=-5.0, rho0_R=1.9, rho0_B=0.15) if model == "SC_MP" else dict(A=0.02))
    flat = box[0] == 1
    small, _, _ = run(M, kw, (1, 64, 64) if flat else (64, 64, 64), (0 if flat else 16, 16, 16), "solo")
    at = (0 if flat else box[0] - B - 1, box[1] - B - (1 if flat else 12), box[2] - B - 12)
    big, used, is_far = run(M, kw, box, at, via)
    assert is_far == far and used == kernel
    assert np.array_equal(big, small)
    assert small.max() - small.min() > 0.5   # the droplet is there


# The forces that reach beyond a node's neighbours: the repulsion (normals at the
# neighbours, three nodes a step with the streaming) and the multirange ones (two
# nodes out, three a step), and the storages without a case above.
BENZI = dict(G_RB=0.405, Ga_R=-9.0, Ga_B=-8.0, Gr_R=8.1, Gr_B=7.1, psi_rho0=0.83, rho0_X=0.83, rho0_R=1.18, rho0_B=0.18)
REACH = 3 * STEPS + 1
FAR_REACHING = [  # force, precision, box, far, kernel, boundaries, via
    ("repulsion", "FP64", (296, 296, 320), False, TWO, (0, 0, 0), "solo"),
    ("repulsion", "FP64", (296, 304, 320), True, TWO, (0, 0, 0), "solo"),
    ("repulsion", "FP64", (296, 304, 320), True, TWO, (1, 1, 0), "batch"),
    ("repulsion", "FP32", (376, 384, 384), False, TWO, (1, 1, 0), "batch"),
    ("repulsion", "FP16", (388, 384, 384), True, TWO, (0, 0, 0), "solo"),
    ("multirange", "FP64", (296, 296, 320), False, TWO, (0, 0, 0), "solo"),
    ("multirange", "FP64", (296, 304, 320), True, TWO, (1, 1, 0), "solo"),
    ("multirange", "FP32", (376, 384, 384), False, TWO, (1, 1, 0), "solo"),
    ("multirange", "FP32", (388, 384, 384), True, TWO, (0, 0, 0), "solo"),
    ("multirange", "FP32", (388, 384, 384), True, TWO, (0, 0, 0), "batch"),
    ("multirange", "MIXED", (388, 384, 384), True, TWO, (1, 1, 0), "solo"),
    ("none", "MIXED", (376, 384, 384), False, ONE, (0, 0, 0), "solo"),
    ("none", "MIXED", (388, 384, 384), True, ONE, (1, 1, 0), "batch"),
    ("none", "FP16", (376, 384, 384), False, ONE, (0, 0, 0), "solo"),
    ("none", "FP16", (376, 384, 384), False, TWO, (1, 1, 0), "batch"),
]


def evolve(M, kw, box, at, via):
    """run() of two-component boxes with some of both colours everywhere."""
    import torch
    nz, ny, nx = box
    z0, y0, x0 = at
    p = M.make_params(nx=nx, ny=ny, nz=nz, **kw)
    fields = []
    for blk, amb in zip(inputs.droplet((B, B, B), 6.0, 1.0, 1.0), (0.0, 1.0)):
        f = torch.full(box, amb + 0.18, dtype=torch.float64, device="cuda")
        f[z0:z0 + B, y0:y0 + B, x0:x0 + B] = torch.from_numpy(blk).cuda() + 0.18
        fields.append(f)
    s = M.Sim(p)
    s.init_equilibrium(*fields)
    del fields
    if via == "batch":
        b = M.Batch([s], [STEPS])
        b.step(STEPS, use_graph=False)
        b.status()
        kernel = b.kernels()[0]
        b.close()
    else:
        s.step(STEPS)
        kernel = s.kernel_used()
    words, word_bytes, _ = M.population_stride(p)
    rho = s.moments()[0]
    out = rho[z0:z0 + B, y0:y0 + B, x0:x0 + B].cpu().numpy()
    s.close()
    del rho, s
    gc.collect()
    torch.cuda.empty_cache()
    return out, kernel, 19 * words * word_bytes >= 2 ** 32


@pytest.mark.parametrize("force,precision,box,far,kernel,bc,via", FAR_REACHING)
def test_far_reaching_forces_at_the_top_of_the_address_range(M, force, precision, box, far, kernel, bc, via):
    print(f"[addressing] {force} {precision} {box} kernel {kernel} bc {bc} {via}", flush=True)
    kw = dict(lattice=M.D3Q19, precision=getattr(M, precision), bc=bc, kernel=kernel)
    kw.update(dict(model=M.SC_MC, **BENZI) if force == "multirange" else
              dict(A=0.02, Pi=0.01 if force == "repulsion" else 0.0))
    small, _, _ = evolve(M, kw, (64, 64, 64), (16, 16, 16), "solo")
    at = (box[0] - B - 1, box[1] - B - REACH, box[2] - B - REACH)
    big, used, is_far = evolve(M, kw, box, at, via)
    assert is_far == far and used == kernel
    assert np.isfinite(small).all() and np.array_equal(big, small)
    assert small.max() - small.min() > 0.5   # the droplet is there
