"""The cubic-tile gridding kernels of general frames (tune = 2), whole volumes against the FP64 oracle:
both fetches (rows of whole 16-byte chunks or of any length), one, two and four view groups per tile, view
counts around the groups and past the 64 box origins formed at once, boxes across every face of the stack.

Tolerances: the FP32 bar of the whole-volume checks (1e-5); 16-bit planes three roundings of the type."""
import numpy as np
import pytest

import _oracle_par
import _problems
from synth import scan
from test_gpu_parity import assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BOUND = {1: 3 * 2.0 ** -9, 2: 3 * 2.0 ** -11}


# n_vox: at most 256 tiles (four groups), 7^3 and 8^3 tiles (two), 9^3 tiles (one)
@pytest.mark.parametrize("n_vox,m,k,n", [
    (8, 16, 8, 3), (30, 30, 30, 5), (45, 45, 40, 8), (24, 25, 24, 261), (20, 54, 40, 1), (40, 27, 33, 6), (20, 16, 20, 70),
    (50, 50, 50, 3), (64, 64, 64, 5), (56, 75, 56, 2), (60, 45, 60, 131), (50, 48, 50, 1),
    (65, 75, 65, 3), (72, 72, 72, 2), (66, 50, 60, 66)])
@pytest.mark.parametrize("ewald", [1, 0], ids=["curved", "flat"])
def test_cubic_tiles_match_oracle(n_vox, m, k, n, ewald):
    pb = _general(n_vox, m, k if ewald else 1, n)
    pb.ewald = ewald
    got = _run(pb, tune=2)
    ref = _reference(pb)
    assert_close(got, ref, 1e-5, (n_vox, m, n, ewald))


def _general(n_vox, m, k, n):
    dx = 1e-10
    dirs = scan.uniform_sphere(900 + n_vox + m, n)
    dist = np.linspace(30e-10, 40e-10, n)
    lam, sig = 0.1e-10, 0.05
    imgs = _problems._born(800 + m, n_vox, m, dx, lam, dirs, dist, sig, count=12)
    return _problems.Problem(f"cube{n_vox}_{m}", n_vox, m, k, dx, lam, sig, 1e-3, 1, "ramp_iso", dirs, dist, imgs)


def _run(pb, **kw):
    from paper_2206_09151_amd import tomo
    plan = tomo.Plan(pb.params(**kw), pb.dirs, pb.dist)
    vol = torch.full((pb.n_vox,) * 3, float("nan"), dtype=torch.float32, device="cuda:0")
    plan.reconstruct(torch.from_numpy(pb.images).to("cuda:0"), vol)
    assert plan.grid_rows == 0
    plan.destroy()
    return vol.cpu().numpy()


def _reference(pb):
    return _oracle_par.reconstruct_views(pb.images.astype(np.float64), pb.dirs, pb.dist, pb.oracle_geometry())


@pytest.mark.parametrize("n_vox,m", [(45, 48), (30, 30), (33, 45), (64, 64), (20, 16), (56, 50), (65, 72), (66, 54)])
@pytest.mark.parametrize("dtype", [1, 2], ids=["bf16", "fp16"])
def test_cubic_tiles_of_16_bit_planes(n_vox, m, dtype):
    pb = _general(n_vox, m, n_vox, 5)
    got, ref = _run(pb, tune=2, plane_dtype=dtype), _reference(pb)
    assert np.linalg.norm(got - ref) <= BOUND[dtype] * np.linalg.norm(ref), (n_vox, m, dtype)
