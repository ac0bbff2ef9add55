"""Whole single-axis reconstructions by slices (automatic angle batch): every detector size of the
slice kernels against the FP64 oracle over the whole volume, with square and narrower slices
(K = M and K < M, N = M and N < M, both parities of N), and the plans that stay on plane stacks.

Tolerance: the FP32 bar of the whole-volume checks, rel-L2 and max|d| / max|ref| <= 1e-5."""
import numpy as np
import pytest

import _oracle_par
import _problems
from synth import scan
from test_gpu_parity import assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [m for m in _problems.smooth_sizes() if m <= 192]


def _problem(m, n_vox, k, n):
    dx = 1e-10
    dirs = scan.single_axis(n, 180.0, offset_deg=3.0 + m % 11)
    dist = np.linspace(50e-10, 60e-10, n)
    lam, sig = 0.05e-10, 0.1
    imgs = _problems._born(700 + m, n_vox, m, dx, lam, dirs, dist, sig, count=24)
    return _problems.Problem(f"slices{m}", n_vox, m, k, dx, lam, sig, 1e-3, 1, "ramp_iso" if m % 2 else "ramp_axis",
                             dirs, dist, imgs)


def _run(pb, **kw):
    from paper_2206_09151_amd import tomo
    plan = tomo.Plan(pb.params(**kw), pb.dirs, pb.dist)
    vol = torch.full((pb.n_vox,) * 3, float("nan"), dtype=torch.float32, device="cuda:0")
    plan.timing(True)
    plan.reconstruct(torch.from_numpy(pb.images).to("cuda:0"), vol)
    launches = plan.timing_read()["planes"][1]
    plan.destroy()
    return vol.cpu().numpy(), launches


@pytest.mark.parametrize("m", SIZES)
@pytest.mark.parametrize("square", [True, False], ids=["square", "narrow"])
def test_slices_match_oracle(m, square):
    """Blocks of three views and a ragged last one (n = 7: two blocks of 3 and 4 views)."""
    pb = _problem(m, m if square else m - 4, m if square else m - 2, 7)
    print(f"M={m} N={pb.n_vox} K={pb.n_planes}", flush=True)
    got, launches = _run(pb)
    assert launches == 1
    ref = _oracle_par.reconstruct_views(pb.images.astype(np.float64), pb.dirs, pb.dist, pb.oracle_geometry())
    assert np.isfinite(got).all()
    assert_close(got, ref, 1e-5, (m, square))


@pytest.mark.parametrize("dtype", [0, 1, 2], ids=["f32", "bf16", "fp16"])
@pytest.mark.parametrize("n", [1, 2, 24])
def test_slices_of_few_views_and_16_bit_plans(n, dtype):
    """One and two views (one block); 16-bit plans keep the stack path, with its 16-bit rounding: the
    volume is bitwise that of a plan with an explicit angle batch."""
    pb = _problem(32, 32, 32, n)
    got, _ = _run(pb, plane_dtype=dtype)
    if dtype != 0:
        assert np.array_equal(got, _run(pb, plane_dtype=dtype, angle_batch=n)[0])
    ref = _oracle_par.reconstruct_views(pb.images.astype(np.float64), pb.dirs, pb.dist, pb.oracle_geometry())
    assert_close(got, ref, {0: 1e-5, 1: 3 * 2.0 ** -9, 2: 3 * 2.0 ** -11}[dtype], (n, dtype))


@pytest.mark.parametrize("n_vox,m,k", [(48, 32, 48), (32, 32, 64), (32, 32, 31), (44, 45, 44)])
def test_other_shapes_stay_on_the_general_path(n_vox, m, k):
    """N > M, K > M, M - K odd and M - N odd: general or stack kernels, same results."""
    pb = _problem(m, n_vox, k, 6)
    got, _ = _run(pb)
    ref = _oracle_par.reconstruct_views(pb.images.astype(np.float64), pb.dirs, pb.dist, pb.oracle_geometry())
    assert_close(got, ref, 1e-5, (n_vox, m, k))


BOUND = {0: 1e-5, 1: 3 * 2.0 ** -9, 2: 3 * 2.0 ** -11}


@pytest.mark.parametrize("m,n_vox", [(25, 25), (27, 21), (45, 45), (50, 46), (54, 54), (100, 96)])
@pytest.mark.parametrize("dtype", [0, 1, 2], ids=["f32", "bf16", "fp16"])
def test_stack_gridding_of_rows_that_are_not_whole_chunks(m, n_vox, dtype):
    """Plane stacks whose rows are not whole 16-byte chunks (fetched dword by dword; 16-bit rows of
    odd M stay on the general kernels): batches of three views."""
    pb = _problem(m, n_vox, min(n_vox, 40), 7)
    got, _ = _run(pb, angle_batch=3, plane_dtype=dtype)
    ref = _oracle_par.reconstruct_views(pb.images.astype(np.float64), pb.dirs, pb.dist, pb.oracle_geometry())
    if dtype == 0:
        assert_close(got, ref, 1e-5, (m, dtype))
    else:
        assert np.linalg.norm(got - ref) <= BOUND[dtype] * np.linalg.norm(ref), (m, dtype)


@pytest.mark.parametrize("m,n_vox,n", [(16, 16, 5), (25, 25, 70), (32, 30, 9), (64, 64, 4), (45, 45, 1), (32, 48, 6)])
@pytest.mark.parametrize("dtype", [0, 1, 2], ids=["f32", "bf16", "fp16"])
def test_flat_gridding_matches_oracle(m, n_vox, n, dtype):
    """Without curvature (one plane per view): ragged tiles and row blocks, odd detectors, a volume
    wider than the detector, view counts around the rounds of four and more than the 64 window
    origins formed at once."""
    pb = _problem(m, n_vox, 1, n)
    pb.ewald = 0
    got, _ = _run(pb, plane_dtype=dtype)
    ref = _oracle_par.reconstruct_views(pb.images.astype(np.float64), pb.dirs, pb.dist, pb.oracle_geometry())
    if dtype == 0:
        assert_close(got, ref, 1e-5, (m, n, dtype))
    else:
        assert np.linalg.norm(got - ref) <= BOUND[dtype] * np.linalg.norm(ref), (m, n, dtype)
