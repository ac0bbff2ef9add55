"""The split of a sliced single-axis scan into blocks of views: single-view blocks of short scans, ragged
blocks, and blocks of many views, against the FP64 oracle over the whole volume (the FP32 bar, 1e-5)."""
import numpy as np
import pytest

import _oracle_par
from test_gpu_axis import _problem, _run
from test_gpu_parity import assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n_vox,k,n", [
    (36, 36, 36, 4), (36, 34, 30, 8), (45, 45, 45, 10), (64, 64, 64, 7), (64, 62, 64, 13), (72, 72, 72, 3),
    (96, 94, 96, 4), (128, 128, 128, 3), (192, 192, 192, 2),           # blocks of one view and a few more
    (25, 25, 25, 100), (36, 36, 36, 61), (64, 64, 64, 50), (81, 81, 79, 31), (125, 125, 125, 13), (160, 158, 160, 9)])
def test_view_blocks_match_oracle(m, n_vox, k, n):
    pb = _problem(m, n_vox, k, n)
    print(f"M={m} N={n_vox} K={k} n={n}", flush=True)
    got, launches = _run(pb)
    assert launches == 1
    ref = _oracle_par.reconstruct_views(pb.images.astype(np.float64), pb.dirs, pb.dist, pb.oracle_geometry())
    assert_close(got, ref, 1e-5, (m, n))


@pytest.mark.parametrize("m,n_vox,k,n,slices", [
    (16, 16, 16, 6, False), (16, 16, 16, 7, True), (36, 36, 36, 3, False), (36, 36, 36, 4, True),
    (50, 50, 50, 1, False), (54, 54, 54, 1, True),                                         # the shortest scans
    (32, 32, 2, 30, False), (32, 32, 4, 30, True), (90, 90, 10, 30, True),                 # room for few blocks
    (160, 20, 20, 6, False), (160, 80, 80, 6, True), (192, 192, 24, 5, False), (192, 144, 144, 5, True)])
def test_route_of_small_scans_and_volumes(m, n_vox, k, n, slices):
    """Scans that plane stacks reconstruct faster take them: the volume is then bit for bit that of an
    explicit batch of the same size; either route matches the oracle."""
    from paper_2206_09151_amd import tomo
    pb = _problem(m, n_vox, k, n)
    plan = tomo.Plan(pb.params(), pb.dirs, pb.dist)
    batch = plan.batch
    plan.destroy()
    got, stacks = _run(pb)[0], _run(pb, angle_batch=batch)[0]
    assert np.array_equal(got, stacks) == (not slices)
    ref = _oracle_par.reconstruct_views(pb.images.astype(np.float64), pb.dirs, pb.dist, pb.oracle_geometry())
    assert_close(got, ref, 1e-5, (m, n))
    assert_close(stacks, ref, 1e-5, (m, n))
