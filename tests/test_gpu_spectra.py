"""The two-kernel spectra (FP32 planes, slices, Fourier form) at the edges of their ranges."""
from dataclasses import replace

import numpy as np
import pytest

import _problems
from synth import scan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _plan(m, n, **kw):
    from paper_2206_09151_amd import tomo
    dirs, dist = scan.single_axis(n, 180.0, offset_deg=2.0), np.full(n, 50e-10)
    base = dict(n_vox=m, n_angles=n, voxel_size=1e-10, wavelength=0.05e-10, sigma=0.1, epsilon=1e-3)
    base.update(kw)
    return tomo.Plan(tomo.Params(**base), dirs, dist)


@pytest.mark.parametrize("value,i_in", [(1e-30, 1e300), (1e30, 1e-300)], ids=["underflow", "overflow"])
@pytest.mark.parametrize("m,kw", [(64, {}), (64, {"angle_batch": 2}), (64, {"ewald": 0}), (32, {"angle_batch": 2}),
                                  (64, {"plane_dtype": 1})], ids=["slices", "stacks", "flat", "small", "bf16"])
def test_contrast_beyond_fp64_shows_in_the_volume(m, kw, value, i_in):
    """I / I_in that FP64 holds only as 0 or infinity has no finite logarithm: every path shows it as a
    volume that is not finite inside every view's support (the inscribed ball), not as a plausible one."""
    plan = _plan(m, 6, i_in=i_in, **kw)
    img = torch.full((6, m, m), value, dtype=torch.float32, device="cuda:0")
    vol = torch.zeros((m,) * 3, dtype=torch.float32, device="cuda:0")
    plan.reconstruct(img, vol)
    r = np.arange(m) - (m - 1) / 2
    ball = torch.from_numpy(r[:, None, None] ** 2 + r[:, None] ** 2 + r ** 2 < (m / 2 - 2) ** 2)
    assert not torch.isfinite(vol.cpu()[ball]).any()
    plan.destroy()


@pytest.mark.parametrize("m,kw", [(75, {"ewald": 0}), (125, {"ewald": 0}), (128, {"ewald": 0}), (48, {"n_planes": 4}),
                                  (256, {"n_planes": 2}), (45, {"fourier": 1}), (36, {"fourier": 2})])
def test_row_spectra_in_several_rounds_are_bitwise_those_of_one(m, kw):
    """A workspace limit with room for one, two or four of nine views' row spectra (one plane of odd M
    has room for less than one view in its stack): ragged rounds, the same bits."""
    from paper_2206_09151_amd import tomo
    base = dict(angle_batch=1, **kw)
    img = torch.rand((9, m, m), generator=torch.Generator().manual_seed(m)).to("cuda:0") + 0.5
    row = 8 * m * ((m + 1) // 2)
    plan = _plan(m, 9, **base)
    full = tomo.workspace_bytes(plan.params)
    least = tomo.workspace_bytes(replace(plan.params, max_workspace_bytes=1))
    vols = []
    for rounds_of in (9, 4, 2, 1):
        if rounds_of < 9:
            plan = _plan(m, 9, max_workspace_bytes=max(full - (9 - rounds_of) * row, least), **base)
        vol = torch.zeros((m,) * 3, dtype=torch.float32, device="cuda:0")
        if "fourier" in kw:
            plan.fourier_reconstruct(img, vol)
        else:
            plan.reconstruct(img, vol)
        vols.append(vol.cpu())
        plan.destroy()
    assert torch.isfinite(vols[0]).all() and vols[0].abs().max() > 0
    for v in vols[1:]:
        assert torch.equal(v, vols[0])


@pytest.mark.parametrize("n", [1, 255, 256, 300])
def test_splat_bound_over_many_views(n):
    """The splat's fixed-point unit comes from the views' bounds, 256 at a time: the volume of the atomic
    splat against that of the operator gather (FP32 bar, 1e-5), with one view a thousand times brighter
    last, so that a bound that left it out would overflow the accumulator."""
    img = torch.rand((n, 16, 16), generator=torch.Generator().manual_seed(n)) + 0.5
    img[-1] = torch.exp(1000.0 * torch.log(img[-1]).clamp(-0.08, 0.08))
    img = img.to("cuda:0")
    vols = []
    for mode in (1, 2):
        plan = _plan(16, n, fourier=mode)
        vol = torch.zeros((16,) * 3, dtype=torch.float32, device="cuda:0")
        plan.fourier_reconstruct(img, vol)
        vols.append(vol.double().cpu())
        plan.destroy()
    assert torch.linalg.norm(vols[1] - vols[0]) <= 1e-5 * torch.linalg.norm(vols[0])


@pytest.mark.parametrize("m,k,nb", [(64, 64, 5), (125, 1, 1), (125, 1, 134), (135, 1, 115), (128, 1, 128), (256, 4, 32),
                                    (75, 3, 372)])
def test_noalloc_row_spectra_find_room(m, k, nb):
    """tomo_backpropagate_noalloc's row spectra behind the spectra in the static workspace, or (calls that
    fill the workspace) in the planes: bit for bit tomo_backpropagate's planes, and nothing written past them."""
    plan = _plan(m, nb, angle_batch=8, **({"n_planes": k} if k > 1 else {"ewald": 0}))
    img = torch.rand((nb, m, m), generator=torch.Generator().manual_seed(m)).to("cuda:0") + 0.5
    want = torch.full(plan.stack_shape(nb), float("nan"), device="cuda:0")
    got = torch.full(plan.stack_shape(nb + 1), float("nan"), device="cuda:0")
    plan.backpropagate(img, 0, nb, want)
    plan.backpropagate_noalloc(img, 0, nb, got)
    torch.cuda.synchronize()
    assert torch.equal(got[:nb], want) and torch.isnan(got[nb]).all()
    plan.destroy()


def test_noalloc_leaves_the_plans_workspace_alone():
    """Reconstructions on one stream while tomo_backpropagate_noalloc runs on another (FP32 planes: it only
    reads the plan's tables): both give the bits that they give alone."""
    for kw in ({}, {"angle_batch": 8}):
        plan = _plan(96, 24, **kw)
        img = torch.rand((24, 96, 96), generator=torch.Generator().manual_seed(3)).to("cuda:0") + 0.5
        vol, alone = (torch.empty((96,) * 3, device="cuda:0") for _ in range(2))
        st, st_alone = (torch.empty(plan.stack_shape(6), device="cuda:0") for _ in range(2))
        plan.reconstruct(img, alone)
        plan.backpropagate(img[4:10].contiguous(), 4, 6, st_alone)
        part = img[4:10].contiguous()
        torch.cuda.synchronize()
        a, b = torch.cuda.Stream(), torch.cuda.Stream()
        for _ in range(40):
            plan.reconstruct_async(img, vol, stream=a)
            plan.backpropagate_noalloc(part, 4, 6, st, stream=b)
            plan.backpropagate_noalloc(part, 4, 6, st, stream=b)
        torch.cuda.synchronize()
        assert torch.equal(vol, alone) and torch.equal(st, st_alone)
        plan.destroy()
