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
