"""The single-axis gridding kernels of plane stacks (2, 4 and 8 voxel rows per thread), through explicit
batches, which plans with an automatic batch no longer run at these sizes: bitwise the same volume
whatever the rows, and the FP64 oracle's to the FP32 bar.  And the slice path's asynchronous form and
domain errors."""
import numpy as np
import pytest

import _oracle_par
import _problems
from test_gpu_axis import _problem
from test_gpu_parity import assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _run(pb, batch, tune, **kw):
    from paper_2206_09151_amd import tomo
    plan = tomo.Plan(pb.params(angle_batch=batch, tune=tune, **kw), pb.dirs, pb.dist)
    vol = torch.full((pb.n_vox,) * 3, float("nan"), dtype=torch.float32, device="cuda:0")
    plan.timing(True)
    plan.reconstruct(torch.from_numpy(pb.images).to("cuda:0"), vol)
    launches = plan.timing_read()
    rows = plan.grid_rows
    plan.destroy()
    n_batches = -(-pb.n // batch)
    assert launches["planes"][1] == launches["grid"][1] == n_batches > 1       # plane stacks, batch by batch
    return vol.cpu().numpy(), rows


@pytest.mark.parametrize("name", ["axis32", "ragged44", "oddk16", "m128", "m160"])
def test_stack_gridding_rows_are_bitwise_equal(name):
    pb = _problems.make(name)
    batch = max(1, pb.n // 2 - 1)
    (v8, r8), (v2, r2) = _run(pb, batch, 0), _run(pb, batch, 5)
    auto, rows = _run(pb, batch, 1)
    print(f"{name}: batches of {batch}, autotuned to {rows} rows", flush=True)
    assert (r8, r2) == (8, 2) and rows in (2, 4, 8)
    assert np.array_equal(v8, v2) and np.array_equal(v8, auto)
    ref = _oracle_par.reconstruct_views(pb.images.astype(np.float64), pb.dirs, pb.dist, pb.oracle_geometry())
    assert_close(v8, ref, 1e-5, name)


@pytest.mark.parametrize("dtype", [0, 1, 2], ids=["f32", "bf16", "fp16"])
@pytest.mark.parametrize("m,n_vox,k", [(128, 128, 128), (128, 114, 128), (96, 90, 50)])
def test_large_and_ragged_stacks(m, n_vox, k, dtype):
    """A volume of whole tiles, one whose last tiles are 2 voxels wide and one cut in columns and rows."""
    pb = _problem(m, n_vox, k, 9)
    v8, _ = _run(pb, 4, 0, plane_dtype=dtype)
    v2, _ = _run(pb, 4, 5, plane_dtype=dtype)
    assert np.array_equal(v8, v2)
    ref = _oracle_par.reconstruct_views(pb.images.astype(np.float64), pb.dirs, pb.dist, pb.oracle_geometry())
    if dtype == 0:
        assert_close(v8, ref, 1e-5, (m, n_vox))
    else:
        assert np.linalg.norm(v8 - ref) <= 3 * 2.0 ** {1: -9, 2: -11}[dtype] * np.linalg.norm(ref), (m, n_vox)


@pytest.mark.parametrize("m,n", [(32, 24), (64, 20), (96, 9)])
def test_slices_asynchronously_and_with_invalid_images(m, n):
    """By slices: the asynchronous form gives the bits of the waiting one, an invalid image value is
    reported once by the call that waits next, and the plan then works as before."""
    from paper_2206_09151_amd import tomo
    pb = _problem(m, m, m, n)
    plan = tomo.Plan(pb.params(), pb.dirs, pb.dist)
    img = torch.from_numpy(pb.images).to("cuda:0")
    a, b = (torch.empty((m,) * 3, dtype=torch.float32, device="cuda:0") for _ in range(2))
    plan.reconstruct(img, a)
    plan.reconstruct_async(img, b)
    plan.sync()
    assert torch.equal(a, b)
    stacks = tomo.Plan(pb.params(angle_batch=n), pb.dirs, pb.dist)
    stacks.reconstruct(img, b)
    stacks.destroy()
    assert not torch.equal(a, b)                                     # the plan above ran by slices
    for value, where in ((0.0, (0, 0, 0)), (-1.0, (n // 2, m // 2, m - 1)), (float("nan"), (n - 1, m - 1, m - 1)),
                         (float("inf"), (n - 1, m - 1, 0))):
        bad = img.clone()
        bad[where] = value
        plan.reconstruct_async(bad, b)
        with pytest.raises(tomo.TomoError) as e:
            plan.sync()
        assert e.value.status == tomo.EDOMAIN
        plan.sync()                                                  # reported once
        with pytest.raises(tomo.TomoError) as e:
            plan.reconstruct(bad, b)
        assert e.value.status == tomo.EDOMAIN
    plan.reconstruct(img, b)
    assert torch.equal(a, b)
    plan.destroy()
