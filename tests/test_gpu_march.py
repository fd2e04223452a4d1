"""Where the march along a ray begins and what decides its samples: a tile's
first samples are skipped from the free-space bits of the map, 128 samples per
wavefront and at most 512, the rest is marched; thresholds other than 0 and
grids whose bits do not fit beside a workgroup are marched without bits."""
import numpy as np
import pytest
import torch

import oracle as orc
import synth
from gpu_util import DEV, P, banner, cam_of, depth_close, gpu_map, grid_of, neq_check, oracle_map_values, t
from test_gpu_parity import _gd_inputs, _shell_field

pytestmark = pytest.mark.gpu


def _pose(at, yaw, pitch=0.0):
    return synth.pose7(np.asarray(at, float), orc.rot_to_quat(synth.camera_rotation(yaw, pitch)))


@pytest.mark.parametrize("k", [129, 256, 257, 511, 513, 1100])
@pytest.mark.parametrize("dtype", [0, 1])
def test_surface_late_on_the_ray(k, dtype):
    """More samples than one wavefront, and than the tile's start, covers; a
    closed shell seen from outside (near and far) and from inside, first
    crossings from early in the ray to near its end: hit samples bit for bit
    against the oracle, depth to tolerance."""
    banner(f"late surface K={k} dtype={dtype}")
    n, vox = 40, 0.05
    mid = 0.5 * n * vox
    field = _shell_field(n)
    g = P().Grid.make(n, vox, (0.0, 0.0, 0.0), dtype)
    vm = gpu_map(g, field, np.ones_like(field))
    og = orc.Grid(n, vox, (0.0, 0.0, 0.0))
    late = []
    for at, yaw, pitch, far in [((-2.6, mid, mid), 0.0, 0.0, 3.2), ((-0.4, mid, mid), 0.1, 0.1, 4.0),
                                ((-1.4, -1.4, 0.4), 0.75, -0.2, 3.4), ((mid, mid, mid), 1.0, 0.3, 1.8),
                                ((0.1, 0.1, 0.1), 0.7, -0.5, 4.2)]:
        cm = synth.Camera(37, 29, 45.0, 45.0, 18.5, 14.0, 0.05, far, k)
        out = P().render(g, vm, cam_of(cm), P().poses_tensor(_pose(at, yaw, pitch)), hit_k=True)
        ref = orc.render(og, oracle_map_values(field, dtype), orc.cam_from(cm), _pose(at, yaw, pitch))
        np.testing.assert_array_equal(out["hit_k"][0].cpu().numpy(), ref["hit_k"])
        v = ref["mask"] == 1
        assert np.all(depth_close(out["depth"][0].cpu().numpy()[v], ref["depth"][v]))
        late.append(int((ref["hit_k"] > 0.7 * k).sum()))
    print(f"[march] crossings past 0.7 K per view: {late}", flush=True)
    assert sum(late) > 500


def test_threshold_other_than_zero():
    """tau != 0 is marched without bits: render, render Jacobian and a descent
    step against the oracle with the same threshold."""
    banner("tau = 0.01")
    c, m0, v0, pose = _gd_inputs()
    c["cam"].tau = 0.01
    g, cam = grid_of(c["scene"], 0), cam_of(c["cam"])
    og, oc = orc.grid_from_scene(c["scene"]), orc.cam_from(c["cam"])
    assert cam.tau == oc.tau == 0.01
    p = orc.Params()
    w = P().Weights.make(p.b_geo, p.b_rgb, p.gate_geo, p.gate_rgb)
    vm, pt = gpu_map(g, m0, v0), P().poses_tensor(pose)
    D, C = t(c["depth"][0]), t(c["rgb"][0])
    out = P().render(g, vm, cam, pt, hit_k=True)
    ref = orc.render(og, m0.astype(np.float64), oc, pose)
    np.testing.assert_array_equal(out["hit_k"][0].cpu().numpy(), ref["hit_k"])
    v = ref["mask"] == 1
    assert v.sum() > 1000 and np.all(depth_close(out["depth"][0].cpu().numpy()[v], ref["depth"][v]))
    j = P().render_jacobian(g, vm, cam, pt, D[None].contiguous(), C[None].contiguous(), w)
    neq_check(j["neq"][0].cpu().numpy(), orc.render_jacobian(og, m0.astype(np.float64), oc, pose, c["depth"][0],
                                                             c["rgb"][0], p)["neq"], "tau")
    cost = torch.zeros(1, dtype=torch.float64, device=DEV)
    P().map_gd(g, vm, cam, pt, D, C, w, 3e-6, 3e-3, 1, P().map_gd_workspace(g, cam), cost)
    want, wcost = orc.map_gd(og, m0.astype(np.float64), v0.astype(np.float64), oc, pose, c["depth"][0], c["rgb"][0],
                             p, 3e-6, 3e-3, 1)
    np.testing.assert_allclose(cost.cpu().numpy(), wcost, rtol=1e-5)
    got = vm.to_dense()[0].cpu().numpy()
    assert np.count_nonzero(want != m0) > 10000
    assert np.all(np.abs(got - want) <= 1e-6 * np.maximum(np.abs(want), 1e-2))


@pytest.mark.parametrize("n", [464, 472, 584, 592])
def test_grids_around_the_bits_limit(n):
    """The dilated bits of a grid fit a workgroup to n = 584, both bitmaps
    would to 464: the march with whatever bits there are finds the samples
    that the march without any finds.  (A threshold of 1e-30 turns the bits
    off; no interpolated value of this map lies between it and 0.)"""
    banner(f"bits limit n={n}")
    vox = 6.4 / n
    g = P().Grid.make(n, vox, (0.0, 0.0, 0.0))
    mean = torch.full((4, n, n, n), -0.5, device=DEV)
    occ = mean[0]
    for a in range(3):
        for e in (slice(0, 5), slice(n - 5, n)):
            occ.transpose(0, a)[e].fill_(0.5)
    occ[:, n // 2:n // 2 + 9, n // 4:n // 4 + 7] = 0.25
    occ[n // 3:n // 3 + 3, : n // 3, n // 2:] = 0.75
    vm = P().VoxelMap(g).init()
    vm.from_dense(mean, None)
    del mean, occ
    hits = []
    for at, yaw, pitch in [((3.2, 3.2, 3.0), 0.3, 0.1), ((-1.0, 2.0, 3.0), 0.1, 0.0), ((5.9, 0.6, 5.8), 2.3, -0.5)]:
        got = []
        for tau in (0.0, 1e-30):
            cam = P().Camera.make(203, 151, 150.0, 150.0, 101.0, 75.0, 0.05, 9.0, 640, tau)
            got.append(P().render(g, vm, cam, P().poses_tensor(_pose(at, yaw, pitch)), hit_k=True))
        for key in ("hit_k", "mask", "depth", "rgb"):
            assert torch.equal(got[0][key], got[1][key]), key
        hits.append(int((got[0]["hit_k"] > 0).sum()))
    print(f"[march] hits {hits}", flush=True)
    assert min(hits) > 5000
