"""Droplet labelling on random porous fields (near the percolation threshold:
winding components of every size, wrapping through periodic faces) against the
oracle's labelling, on rows around the wavefront's 64 lanes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_05197_amd as M
    M.lib()
    return M


@pytest.mark.parametrize("shape,bc,fill", [
    ((5, 6, 63), (0, 0, 0), 0.35), ((4, 7, 64), (0, 1, 2), 0.35), ((7, 5, 65), (0, 0, 1), 0.3),
    ((2, 3, 130), (0, 0, 0), 0.5), ((9, 2, 2), (0, 0, 0), 0.4), ((40, 41, 43), (0, 0, 0), 0.32),
    ((40, 41, 43), (1, 0, 2), 0.95), ((1, 66, 129), (0, 0, 0), 0.58), ((1, 50, 257), (1, 1, 0), 0.62)])
def test_droplets_on_porous_fields(M, orc, shape, bc, fill):
    nz, ny, nx = shape
    rhoN = np.where(np.random.default_rng(nx + ny).random(shape) < fill, 0.8, -0.8)
    p = M.make_params(lattice=M.D2Q9 if nz == 1 else M.D3Q19, precision=M.FP64, nx=nx, ny=ny, nz=nz, bc=bc)
    s = M.Sim(p)
    s.init_equilibrium(0.5 * (1 + rhoN), 0.5 * (1 - rhoN))
    print(f"[porous] {shape} bc={bc}", flush=True)
    po = orc.make_params(**{k: p[k] for k in orc.DEFAULTS if k in p})
    n_o, lab = orc.label_components(po, s.export_f().cpu().numpy())
    sizes_o = sorted(np.unique(lab[lab >= 0], return_counts=True)[1].tolist(), reverse=True)
    for _ in range(3):
        n, sizes = s.droplets(rhoN.size)
        assert n == n_o and sizes == sizes_o
    s.close()


def test_more_crossings_than_one_copy_holds(M, orc):
    """A striped line of 1300 nodes: 1300 crossings, more than the first copy
    brings back, equal through both entry points and to the oracle's."""
    nx = 1300
    stripes = np.broadcast_to(np.where(np.arange(nx) % 2 == 0, 0.8, -0.8), (2, 4, nx))
    p = M.make_params(lattice=M.D3Q19, precision=M.FP64, nx=nx, ny=4, nz=2)
    s = M.Sim(p)
    s.init_equilibrium(0.5 * (1 + stripes), 0.5 * (1 - stripes))
    po = orc.make_params(**{k: p[k] for k in orc.DEFAULTS if k in p})
    ref, nref = orc.interface_crossings(po, s.export_f().cpu().numpy(), 0, 1, 1, nx)
    for noalloc in (False, True):
        for room in (nx, 600, 511, 3):
            got, n = s.interface_crossings(0, 1, 1, max_out=room, noalloc=noalloc)
            assert n == nref == nx
            assert np.allclose(got, ref[:room], rtol=0, atol=1e-9)
    s.close()
