"""HIP library (through the C ABI) against the FP64 oracle, element by element
on the same seeded inputs.

Integer decisions (hit sample, interpolation cell, updated-voxel set, pixel
association) are compared bit for bit; the oracle takes them with the same
single-precision recipe as the kernels.  Values are compared with the
tolerances in gpu_util.
"""
import ctypes
from fractions import Fraction

import numpy as np
import pytest
import torch

import oracle as orc
import synth
from gpu_util import (DEV, banner, cam_of, depth_close, gpu_map, grid_of, oracle_map_values, rgb_close,
                      rot_angle, t, P)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    P().lib()
    yield


@pytest.fixture(scope="module")
def case1():
    c = synth.single_frame_case(0)
    mean, var = synth.gt_map(c["scene"])
    return c, mean, var


@pytest.fixture(scope="module")
def case2():
    """One frame of the 256^3 / 320x240 / 128-sample trajectory workload."""
    c = synth.trajectory_case(seed=1, n=256, width=320, height=240, n_samples=128, n_frames=6)
    mean, var = synth.gt_map(c["scene"], dtype=np.float32)
    return c, mean, var


# ---------------------------------------------------------------------------
def test_map_roundtrip(case1):
    banner("map roundtrip")
    c, mean, var = case1
    for dtype in (0, 1):
        g = grid_of(c["scene"], dtype)
        vm = gpu_map(g, mean, var)
        m2, v2 = vm.to_dense()
        exp_m = oracle_map_values(mean, dtype).astype(np.float32)
        exp_v = oracle_map_values(var, dtype).astype(np.float32)
        np.testing.assert_array_equal(m2.cpu().numpy(), exp_m)
        np.testing.assert_array_equal(v2.cpu().numpy(), exp_v)
    # planes helpers
    n = 16
    x = torch.randn(3, n, n, n, device=DEV)
    b = P().dense_to_bricks(n, x)
    np.testing.assert_array_equal(P().bricks_to_dense(n, b).cpu().numpy(), x.cpu().numpy())


def _render_compare(c, mean, var, pose, dtype, normals=True, label=""):
    g = grid_of(c["scene"], dtype)
    cam = cam_of(c["cam"])
    vm = gpu_map(g, mean, var)
    out = P().render(g, vm, cam, P().poses_tensor(pose), normals=normals, hit_k=True)
    torch.cuda.synchronize()
    og = orc.grid_from_scene(c["scene"])
    oc = orc.cam_from(c["cam"])
    ref = orc.render(og, oracle_map_values(mean, dtype), oc, pose, decide32=True, normals=normals)
    hk = out["hit_k"][0].cpu().numpy()
    np.testing.assert_array_equal(hk, ref["hit_k"], err_msg=f"hit sample {label}")
    mk = out["mask"][0].cpu().numpy()
    np.testing.assert_array_equal(mk, ref["mask"])
    v = mk == 1
    d = out["depth"][0].cpu().numpy()
    assert np.all(depth_close(d[v], ref["depth"][v])), np.max(np.abs(d[v] - ref["depth"][v]))
    assert np.all(d[~v] == 0)
    rgb = out["rgb"][0].cpu().numpy()
    assert np.all(rgb_close(rgb[v], ref["rgb"][v])), np.max(np.abs(rgb[v] - ref["rgb"][v]))
    if normals:
        # the normals kernel against the oracle's normals of the same image
        n_ref, m_ref = orc.normals_of(oc, d.astype(np.float64), mk, 0.1)
        nm = out["nmask"][0].cpu().numpy()
        np.testing.assert_array_equal(nm, m_ref, err_msg=f"normal mask {label}")
        both = nm == 1
        nrm = out["normals"][0].cpu().numpy()
        assert np.max(np.abs(nrm[both] - n_ref[both])) <= 1e-4
    return out, ref


@pytest.mark.parametrize("dtype", [0, 1])
def test_render_small(case1, dtype):
    banner(f"render 64^3 80x60 dtype={dtype}")
    c, mean, var = case1
    for pose in (synth.pose7(c["t_gt"], c["q_gt"]), synth.pose7(c["t_init"], c["q_init"])):
        _render_compare(c, mean, var, pose, dtype)


def test_render_edge_cases(case1):
    """Camera outside the grid looking away (no hits), camera inside a solid
    (k* = 0 everywhere: invalid), ragged image (not a multiple of the 8x8
    tile), minimal sample count."""
    banner("render edge cases")
    c, mean, var = case1
    g = grid_of(c["scene"])
    vm = gpu_map(g, mean, var)
    og = orc.grid_from_scene(c["scene"])
    cases = [
        (synth.Camera(37, 23, 30.0, 30.0, 18.5, 11.5, 0.1, 3.0, 32), np.array([-5.0, -5.0, -5.0, 1.0, 0, 0, 0])),
        (synth.Camera(17, 9, 12.0, 12.0, 8.0, 4.0, 0.1, 3.0, 2), synth.pose7(c["t_gt"], c["q_gt"])),
        (synth.Camera(33, 17, 25.0, 25.0, 16.0, 8.5, 0.0, 1.0, 7), np.array([0.05, 0.05, 0.05, 1.0, 0, 0, 0])),
    ]
    for cm, pose in cases:
        cam = cam_of(cm)
        out = P().render(g, vm, cam, P().poses_tensor(pose), hit_k=True)
        ref = orc.render(og, oracle_map_values(mean, 0), orc.cam_from(cm), pose)
        np.testing.assert_array_equal(out["hit_k"][0].cpu().numpy(), ref["hit_k"])
        np.testing.assert_array_equal(out["mask"][0].cpu().numpy(), ref["mask"])
        v = ref["mask"] == 1
        assert np.all(depth_close(out["depth"][0].cpu().numpy()[v], ref["depth"][v]))


def _shell_field(n, open_face=False):
    """Occupancy 0.5 in the outermost voxel layer of the grid and -0.5 inside
    (colour a ramp along x); with open_face the x = n-1 face is left empty,
    so rays can leave the grid there."""
    mean = np.zeros((4, n, n, n))
    mean[0] = -0.5
    z, y, x = np.meshgrid(np.arange(n), np.arange(n), np.arange(n), indexing="ij")
    shell = (x == 0) | (y == 0) | (z == 0) | (y == n - 1) | (z == n - 1)
    if not open_face:
        shell |= x == n - 1
    mean[0][shell] = 0.5
    for ch in (1, 2, 3):
        mean[ch] = 0.2 * ch + 0.5 * x / n
    return mean


@pytest.mark.parametrize("dtype", [0, 1])
def test_render_crossings_at_the_grid_boundary(dtype):
    """Crossings in the cells that straddle the grid's boundary, where some
    trilinear corners are the outside value: a closed shell of occupied
    voxels seen from outside (entry through the partial cells) and from
    inside; an open shell whose outside value is positive (the crossing lies
    beyond the last voxel, so the march may not stop where it leaves the
    grid); and the same open shell with the negative default (rays leave the
    grid and never hit).  hit_k and mask bit-exact, depth to tolerance."""
    banner(f"render at the grid boundary dtype={dtype}")
    n, vox = 32, 0.05
    mid = 0.5 * n * vox           # voxel centres sit at (i + 1/2) voxel
    cm = synth.Camera(40, 30, 30.0, 30.0, 19.5, 14.5, 0.05, 4.0, 96)
    cam = cam_of(cm)

    def pose_at(t, yaw, pitch=0.0):
        return synth.pose7(np.asarray(t, float), orc.rot_to_quat(synth.camera_rotation(yaw, pitch)))

    closed, opened = _shell_field(n), _shell_field(n, open_face=True)
    cases = [
        # closed shell, default outside value
        (closed, -0.001, pose_at((-1.0, mid, mid), 0.0)),
        (closed, -0.001, pose_at((-0.6, -0.6, -0.3), 0.75, -0.3)),
        (closed, -0.001, pose_at((mid, mid, mid), 1.0, 0.4)),
        (closed, -0.001, pose_at((0.1, 0.1, 0.1), 0.7, -0.5)),
        # open x = n-1 face, positive outside value
        (opened, 0.5, pose_at((mid, mid, mid), 0.0)),
        (opened, 0.5, pose_at((mid, mid + 0.2, mid - 0.1), 0.3, -0.2)),
        (opened, 0.5, pose_at((2.5, mid, mid), np.pi)),
        # open face, default outside value
        (opened, -0.001, pose_at((mid, mid, mid), 0.0)),
        (opened, -0.001, pose_at((2.5, mid, mid), np.pi)),
    ]
    n_valid = n_invalid = 0
    for field, occ_out, pose in cases:
        g = P().Grid.make(n, vox, (0.0, 0.0, 0.0), dtype, occ_out=occ_out)
        vm = gpu_map(g, field, np.ones_like(field))
        og = orc.Grid(n, vox, (0.0, 0.0, 0.0), occ_out=occ_out)
        out = P().render(g, vm, cam, P().poses_tensor(pose), hit_k=True)
        ref = orc.render(og, oracle_map_values(field, dtype), orc.cam_from(cm), pose)
        np.testing.assert_array_equal(out["hit_k"][0].cpu().numpy(), ref["hit_k"])
        np.testing.assert_array_equal(out["mask"][0].cpu().numpy(), ref["mask"])
        v = ref["mask"] == 1
        n_valid += int(v.sum())
        n_invalid += int((~v).sum())
        assert np.all(depth_close(out["depth"][0].cpu().numpy()[v], ref["depth"][v]))
        assert np.all(rgb_close(out["rgb"][0].cpu().numpy()[v], ref["rgb"][v]))
    print(f"[boundary] {n_valid} hits, {n_invalid} misses over {len(cases)} views", flush=True)
    assert n_valid > 4000 and n_invalid > 1000


@pytest.mark.parametrize("dtype", [0, 1])
def test_render_with_the_papers_sampling(case1, dtype):
    """The paper's ray samples (offsets eps, 2 eps, ... up to the maximum
    depth, eps = 0.4 voxel) through the library's sampling helper: hit
    samples bit-exact against the oracle's camera for the same sampling."""
    banner(f"render with the paper's sampling dtype={dtype}")
    c, mean, var = case1
    sc, cm = c["scene"], c["cam"]
    g = grid_of(sc, dtype)
    vm = gpu_map(g, mean, var)
    cam = P().Camera.paper_sampling(cm.width, cm.height, cm.fx, cm.fy, cm.cx, cm.cy, sc.voxel, 3.0)
    ocam = orc.paper_sample_camera(cm.width, cm.height, cm.fx, cm.fy, cm.cx, cm.cy, sc.voxel, 3.0)
    assert (cam.d_near, cam.d_far, cam.n_samples) == (ocam.d_near, ocam.d_far, ocam.n_samples)
    pose = synth.pose7(c["t_gt"], c["q_gt"])
    out = P().render(g, vm, cam, P().poses_tensor(pose), hit_k=True)
    ref = orc.render(orc.grid_from_scene(sc), oracle_map_values(mean, dtype), ocam, pose)
    np.testing.assert_array_equal(out["hit_k"][0].cpu().numpy(), ref["hit_k"])
    np.testing.assert_array_equal(out["mask"][0].cpu().numpy(), ref["mask"])
    v = ref["mask"] == 1
    print(f"[paper sampling] K={cam.n_samples} eps={cam.d_near:.4f} m, {int(v.sum())} hits", flush=True)
    assert v.sum() > 0.5 * v.size
    assert np.all(depth_close(out["depth"][0].cpu().numpy()[v], ref["depth"][v]))
    assert np.all(rgb_close(out["rgb"][0].cpu().numpy()[v], ref["rgb"][v]))


def test_render_batched_frames(case1):
    """n_frames > 1 in one launch equals the frames rendered one by one."""
    banner("render batched")
    c, mean, var = case1
    g = grid_of(c["scene"])
    cam = cam_of(c["cam"])
    vm = gpu_map(g, mean, var)
    rng = np.random.default_rng(0)
    poses = np.stack([synth.pose7(*synth.perturb_pose(rng, c["t_gt"], c["q_gt"], 0.1, 0.2)) for _ in range(5)])
    allb = P().render(g, vm, cam, P().poses_tensor(poses), normals=True, hit_k=True)
    for i in range(5):
        one = P().render(g, vm, cam, P().poses_tensor(poses[i]), normals=True, hit_k=True)
        for k in one:
            assert torch.equal(one[k][0], allb[k][i]), k


@pytest.mark.parametrize("dtype", [0, 1])
def test_render_full_size_frame(case2, dtype):
    banner(f"render 256^3 320x240x128 dtype={dtype}")
    c, mean, var = case2
    tr = c["traj"]
    for i in (0, 3):
        _render_compare(c, mean, var, synth.pose7(tr.t[i], tr.q[i]), dtype, label=f"frame {i}")


# ---------------------------------------------------------------------------
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("warm", [False, True, "mixed"])
def test_map_update(case1, dtype, warm):
    """cold: prior map; warm: ground-truth means, variance 0.25; mixed:
    random means and a different random variance per channel and voxel (the
    per-channel precision path of the kernel)."""
    banner(f"map_update 64^3 dtype={dtype} warm={warm}")
    c, mean_gt, _ = case1
    n = c["scene"].n
    if warm == "mixed":
        r = np.random.default_rng(11)
        mean = r.normal(0.0, 0.05, size=(4, n, n, n))
        var = r.uniform(0.05, 3.0, size=(4, n, n, n))
    elif warm:
        mean = mean_gt.copy()
        var = np.full_like(mean, 0.25)
    else:
        mean = np.zeros((4, n, n, n)); mean[0] = -0.001
        var = np.full_like(mean, 1e4)
    g = grid_of(c["scene"], dtype)
    cam = cam_of(c["cam"])
    vm = gpu_map(g, mean, var)
    rng = np.random.default_rng(5)
    od, oc = synth.raycast(c["scene"], c["cam"], c["t_gt"], c["q_gt"], rng, 0.01, 0.02)
    od = od.astype(np.float32); oc = oc.astype(np.float32)
    od[3, 5] = np.nan; od[10, 10] = -1.0; od[20, 7] = np.inf   # invalid observations
    pose = synth.pose7(c["t_init"], c["q_init"])
    p = orc.Params()
    nupd = P().map_update(g, vm, cam, P().poses_tensor(pose), t(od), t(oc), p.trunc_voxels * g.voxel, 1.0)
    m2, v2 = vm.to_dense()
    torch.cuda.synchronize()
    om = oracle_map_values(mean, dtype)
    ov = oracle_map_values(var, dtype)
    m0, v0 = om.copy(), ov.copy()
    cnt, upd = orc.map_update(orc.grid_from_scene(c["scene"]), om, ov, orc.cam_from(c["cam"]), pose, od, oc, p,
                              decide32=True, want_mask=True)
    assert int(nupd.item()) == cnt > 1000
    m2 = m2.cpu().numpy().astype(np.float64)
    v2 = v2.cpu().numpy().astype(np.float64)
    u = upd.astype(bool)
    # unchanged voxels are bitwise unchanged
    np.testing.assert_array_equal(m2[:, ~u], m0[:, ~u])
    np.testing.assert_array_equal(v2[:, ~u], v0[:, ~u])
    # the value path is the definition in double precision, rounded once on
    # store: the stored map equals the oracle's result rounded the same way
    if dtype == 0:
        np.testing.assert_array_equal(m2[:, u], om[:, u].astype(np.float32).astype(np.float64))
        np.testing.assert_array_equal(v2[:, u], ov[:, u].astype(np.float32).astype(np.float64))
    else:
        np.testing.assert_array_equal(m2[:, u], synth.bf16_round(om[:, u]).astype(np.float64))
        np.testing.assert_array_equal(v2[:, u], synth.bf16_round(ov[:, u]).astype(np.float64))


def test_map_update_full_size(case2):
    """256^3 map, 320x240 frame: the updated set is identical voxel for voxel."""
    banner("map_update 256^3 320x240")
    c, _, _ = case2
    n = c["scene"].n
    g = grid_of(c["scene"])
    cam = cam_of(c["cam"])
    vm = P().VoxelMap(g).init()
    tr = c["traj"]
    pose = synth.pose7(tr.t[2], tr.q[2])
    od = c["depth"][2]; oc = c["rgb"][2]
    p = orc.Params()
    nupd = P().map_update(g, vm, cam, P().poses_tensor(pose), t(od), t(oc), p.trunc_voxels * g.voxel, 1.0)
    m2, v2 = vm.to_dense()
    om = np.zeros((4, n, n, n)); om[0] = np.float32(-0.001)
    ov = np.full_like(om, 1e4)
    cnt, upd = orc.map_update(orc.grid_from_scene(c["scene"]), om, ov, orc.cam_from(c["cam"]), pose, od, oc, p,
                              want_mask=True)
    assert int(nupd.item()) == cnt > 100000
    changed = (v2[0].cpu().numpy() != np.float32(1e4))
    np.testing.assert_array_equal(changed, upd.astype(bool))
    u = upd.astype(bool)
    m2 = m2.cpu().numpy()
    np.testing.assert_array_equal(m2[:, u], om[:, u].astype(np.float32))


@pytest.mark.parametrize("dtype", [0, 1])
def test_free_space_bits_follow_updates(case2, dtype):
    """The map update keeps each brick's free-space bit equal to (maximum
    occupancy <= 0) incrementally: after several updates, renders with the
    maintained bits equal renders after the bits are rebuilt from scratch,
    and the hit samples equal the oracle's (which marches every sample)."""
    banner(f"free-space bits after map updates, dtype {dtype}")
    c, _, _ = case2
    g = grid_of(c["scene"], dtype)
    cam = cam_of(c["cam"])
    vm = P().VoxelMap(g).init()
    tr = c["traj"]
    p = orc.Params()
    for i in range(0, 6, 2):
        P().map_update(g, vm, cam, P().poses_tensor(synth.pose7(tr.t[i], tr.q[i])), t(c["depth"][i]),
                       t(c["rgb"][i]), p.trunc_voxels * g.voxel, 1.0)
    poses = P().poses_tensor(np.stack([synth.pose7(tr.t[i], tr.q[i]) for i in (1, 3, 5)]))
    a = P().render(g, vm, cam, poses, hit_k=True)
    a = {k: v.clone() for k, v in a.items()}
    vm.refresh()
    b = P().render(g, vm, cam, poses, hit_k=True)
    for k in ("hit_k", "depth", "rgb", "mask"):
        assert torch.equal(a[k], b[k]), k
    m, _ = vm.to_dense()
    mv = m.cpu().numpy().astype(np.float64)
    ref = orc.render(orc.grid_from_scene(c["scene"]), mv, orc.cam_from(c["cam"]), synth.pose7(tr.t[3], tr.q[3]))
    np.testing.assert_array_equal(a["hit_k"][1].cpu().numpy(), ref["hit_k"])


# ---------------------------------------------------------------------------
def _filter_run(n, width, n_frames, objective, dtype=0, modes=0):
    c = synth.trajectory_case(seed=2, n=n, width=width, height=width * 3 // 4, n_samples=n // 2,
                              n_frames=n_frames)
    tr = c["traj"]
    g = grid_of(c["scene"], dtype)
    cam = cam_of(c["cam"])
    fp = P().FilterParams(objective=objective, modes=modes)
    f = P().Filter(g, cam, fp)
    f.map.init()
    x0 = np.concatenate([tr.t[0], tr.q[0], tr.v[0], tr.w[0]])
    P0 = np.diag([1e-6] * 6 + [1e-4] * 6)
    f.reset(x0, P0)
    og = orc.grid_from_scene(c["scene"])
    mean = np.zeros((4, n, n, n)); mean[0] = np.float32(-0.001)
    var = np.full_like(mean, 1e4)
    of = orc.Filter(og, orc.cam_from(c["cam"]), _oracle_params(objective, modes, fp.irls_floor),
                    dict(t=tr.t[0], q=tr.q[0], v=tr.v[0], w=tr.w[0]), P0, mean, var)
    D = t(c["depth"]); C = t(c["rgb"]); U = t(tr.u, torch.float64)
    res = []
    for i in range(n_frames):
        f.step(D[i], C[i], U[i - 1] if i else None)
        of.step(c["depth"][i].astype(np.float64), c["rgb"][i].astype(np.float64), tr.u[i - 1] if i else None)
        s = f.state()
        res.append((np.array(s.pose.t), np.array(s.pose.q), np.array(s.v), np.array(s.w),
                    np.array(s.P).reshape(12, 12), s.flags, of.s.t.copy(), of.s.q.copy(), of.s.v.copy(),
                    of.s.w.copy(), of.s.P.copy(), int(s.n_updated), of.s.last["n_updated"]))
    return res


@pytest.mark.parametrize("objective", [0, 1])
def test_filter_steps_match_oracle(objective):
    """Filter state after each step against the oracle filter run on the same
    frames.  The closed loop (pose -> map update -> render -> next pose) feeds
    any difference back; with the render-through objective it grows by one to
    two orders of magnitude per step (the oracle run with double- instead of
    single-precision decisions diverges from itself the same way), so that
    objective is compared over a shorter horizon."""
    n_frames = 6 if objective == 0 else 4
    banner(f"filter 128^3 160x120 objective={objective} frames={n_frames}")
    res = _filter_run(128, 160, n_frames, objective)
    for i, (tg, qg, vg, wg, Pg, flags, to, qo, vo, wo, Po, nu_g, nu_o) in enumerate(res):
        print(f"step {i}: |dt| {np.linalg.norm(tg - to):.3e} m, dR {rot_angle(qg, qo):.3e} rad", flush=True)
        assert flags == 0
        assert np.linalg.norm(tg - to) <= 1e-5, (i, np.linalg.norm(tg - to))
        assert rot_angle(qg, qo) <= 1e-5, (i, rot_angle(qg, qo))
        assert np.linalg.norm(vg - vo) <= 1e-4, i
        assert np.linalg.norm(Pg - Po) <= 1e-4 * np.linalg.norm(Po), (i, np.linalg.norm(Pg - Po) / np.linalg.norm(Po))
        assert abs(nu_g - nu_o) <= max(10, 1e-4 * nu_o), (i, nu_g, nu_o)


def _oracle_params(objective, modes, irls_floor):
    return orc.Params(objective="p1" if objective else "p2",
                      transition_dt2=bool(modes & P().MODE_TRANSITION_DT2),
                      laplace_factor=1.0 if modes & P().MODE_LAPLACE_FACTOR1 else 2.0,
                      irls=bool(modes & P().MODE_IRLS_L1), irls_floor=irls_floor)


@pytest.mark.parametrize("objective", [0, 1])
def test_filter_paper_modes_match_oracle(objective):
    """The paper's literal forms together (u dt^2 transition, Laplace factor
    1, L1 objective by IRLS in the Gauss-Newton iterations), 128^3 / 160x120,
    six frames.  With the printed transition the acceleration controls are
    under-integrated and tracking drifts by centimetres, which makes the
    closed loop ill-conditioned (the oracle with FP64 decisions parts from
    its FP32-decision run by 5e-5 m at the sixth frame), so every step is
    compared from the same start: before step i the oracle takes the GPU
    filter's state and map and renders its anchor from them.

    The render-through objective under IRLS is itself sensitive at the
    1e-5 level within one step: a pixel whose hit sample flips between
    iterates changes its residual, and its IRLS weight grows as 1/|r| (up to
    50 times 1/b^2 at the default floor).  In the oracle, moving the start
    pose of one step by 1e-9 m moves that step's result by up to 1.7e-5 m on
    this trajectory (2e-7 m with the default squared objective), so for P1
    the pose bar here is 1e-4 m / rad; P2 keeps the 1e-5 bar."""
    n, width, n_frames = 128, 160, 6
    pose_bar = 1e-5 if objective == 0 else 1e-4
    modes = P().MODE_TRANSITION_DT2 | P().MODE_LAPLACE_FACTOR1 | P().MODE_IRLS_L1
    banner(f"filter 128^3 160x120 objective={objective} modes={modes}, one step at a time from the GPU state")
    c = synth.trajectory_case(seed=2, n=n, width=width, height=width * 3 // 4, n_samples=n // 2, n_frames=n_frames)
    tr = c["traj"]
    fp = P().FilterParams(objective=objective, modes=modes)
    f = P().Filter(grid_of(c["scene"]), cam_of(c["cam"]), fp)
    f.map.init()
    P0 = np.diag([1e-6] * 6 + [1e-4] * 6)
    f.reset(np.concatenate([tr.t[0], tr.q[0], tr.v[0], tr.w[0]]), P0)
    og, ocm = orc.grid_from_scene(c["scene"]), orc.cam_from(c["cam"])
    op = _oracle_params(objective, modes, fp.irls_floor)
    D = t(c["depth"]); C = t(c["rgb"]); U = t(tr.u, torch.float64)
    for i in range(n_frames):
        s0 = f.state()
        m0, v0 = f.map.to_dense()
        pose0 = np.concatenate([np.array(s0.pose.t), np.array(s0.pose.q)])
        of = orc.Filter(og, ocm, op, dict(t=pose0[:3], q=pose0[3:], v=np.array(s0.v), w=np.array(s0.w)),
                        np.array(s0.P).reshape(12, 12), m0.cpu().numpy().astype(np.float64),
                        v0.cpu().numpy().astype(np.float64))
        if i:
            of.s.step = i
            of.s.Sbar = np.array(s0.Sbar).reshape(6, 6) if s0.has_sbar else None
            of.s.anchor = orc.render(og, of.mean, ocm, pose0, normals=True)
            of.s.anchor_pose = pose0.copy()
        f.step(D[i], C[i], U[i - 1] if i else None)
        of.step(c["depth"][i].astype(np.float64), c["rgb"][i].astype(np.float64), tr.u[i - 1] if i else None)
        s = f.state()
        tg, qg = np.array(s.pose.t), np.array(s.pose.q)
        Pg = np.array(s.P).reshape(12, 12)
        dt_, dr_ = np.linalg.norm(tg - of.s.t), rot_angle(qg, of.s.q)
        eP = np.linalg.norm(Pg - of.s.P) / np.linalg.norm(of.s.P)
        print(f"step {i}: |dt| {dt_:.2e} m, dR {dr_:.2e} rad, P {eP:.2e}, position error to the truth "
              f"{np.linalg.norm(tg - tr.t[i]):.4f} m", flush=True)
        assert s.flags == 0
        assert dt_ <= pose_bar and dr_ <= pose_bar, (i, dt_, dr_)
        assert np.linalg.norm(np.concatenate([np.array(s.v), np.array(s.w)]) - np.concatenate([of.s.v, of.s.w])) <= 10 * pose_bar
        assert eP <= 1e-4, (i, eP)
        nu = of.s.last["n_updated"]
        assert abs(int(s.n_updated) - nu) <= max(10, 1e-4 * nu), i


@pytest.mark.parametrize("objective", [0, 1])
def test_filter_bias_state_matches_oracle(objective):
    """The 15-D state (pose, velocities, accelerometer bias), fed the
    accelerometer's body-frame force: 128^3 / 160x120, six frames, every step
    compared from the same start (the oracle takes the GPU filter's state,
    bias state and map before each step): pose within 1e-5, velocities and
    bias within 1e-4, the 15x15 covariance within 1e-4 relative."""
    n, width, n_frames = 128, 160, 6
    banner(f"filter 128^3 160x120 objective={objective} 15-D state, one step at a time from the GPU state")
    c = synth.trajectory_case(seed=2, n=n, width=width, height=width * 3 // 4, n_samples=n // 2, n_frames=n_frames)
    tr = c["traj"]
    fp = P().FilterParams(objective=objective, modes=P().MODE_ACCEL_BIAS)
    f = P().Filter(grid_of(c["scene"]), cam_of(c["cam"]), fp)
    f.map.init()
    P0 = np.diag([1e-6] * 6 + [1e-4] * 6 + [1e-4] * 3)
    f.reset(np.concatenate([tr.t[0], tr.q[0], tr.v[0], tr.w[0], np.zeros(3)]), P0)
    og, ocm = orc.grid_from_scene(c["scene"]), orc.cam_from(c["cam"])
    op = orc.Params(objective="p1" if objective else "p2", accel_bias=True, sigma_bias=fp.sigma_bias,
                    gravity=tuple(fp.gravity))
    D = t(c["depth"]); C = t(c["rgb"]); U = t(tr.u_body, torch.float64)
    for i in range(n_frames):
        s0, x0 = f.state(), f.bias_state()
        m0, v0 = f.map.to_dense()
        pose0 = np.concatenate([np.array(s0.pose.t), np.array(s0.pose.q)])
        of = orc.Filter(og, ocm, op, dict(t=pose0[:3], q=pose0[3:], v=np.array(s0.v), w=np.array(s0.w),
                                          b=np.array(x0.b)),
                        np.array(x0.P).reshape(15, 15), m0.cpu().numpy().astype(np.float64),
                        v0.cpu().numpy().astype(np.float64))
        if i:
            of.s.step = i
            of.s.Sbar = np.array(s0.Sbar).reshape(6, 6) if s0.has_sbar else None
            of.s.anchor = orc.render(og, of.mean, ocm, pose0, normals=True)
            of.s.anchor_pose = pose0.copy()
        f.step(D[i], C[i], U[i - 1] if i else None)
        of.step(c["depth"][i].astype(np.float64), c["rgb"][i].astype(np.float64), tr.u_body[i - 1] if i else None)
        s, xb = f.state(), f.bias_state()
        tg, qg = np.array(s.pose.t), np.array(s.pose.q)
        Pg = np.array(xb.P).reshape(15, 15)
        dt_, dr_ = np.linalg.norm(tg - of.s.t), rot_angle(qg, of.s.q)
        eP = np.linalg.norm(Pg - of.s.P) / np.linalg.norm(of.s.P)
        db = np.linalg.norm(np.array(xb.b) - of.s.b)
        print(f"step {i}: |dt| {dt_:.2e} m, dR {dr_:.2e} rad, |db| {db:.2e}, P {eP:.2e}, position error to the "
              f"truth {np.linalg.norm(tg - tr.t[i]):.4f} m, bias {np.array(xb.b)}", flush=True)
        assert s.flags == 0
        assert dt_ <= 1e-5 and dr_ <= 1e-5, (i, dt_, dr_)
        assert np.linalg.norm(np.concatenate([np.array(s.v), np.array(s.w)]) - np.concatenate([of.s.v, of.s.w])) <= 1e-4
        assert db <= 1e-4, (i, db)
        assert eP <= 1e-4, (i, eP)
        np.testing.assert_array_equal(np.array(s.P).reshape(12, 12), Pg[:12, :12])
        nu = of.s.last["n_updated"]
        assert abs(int(s.n_updated) - nu) <= max(10, 1e-4 * nu), i


def test_filter_bias_state_entry_points():
    """The 15-D state's entry points refuse the wrong state size: the 12-D
    reset on a 15-D filter, the 15-D reset and bias read-back on a 12-D one,
    and a 12-D checkpoint loaded into a 15-D filter."""
    banner("15-D state entry points")
    c = synth.trajectory_case(seed=2, n=64, width=80, height=60, n_samples=32, n_frames=2)
    tr = c["traj"]
    g, cam = grid_of(c["scene"]), cam_of(c["cam"])
    f15 = P().Filter(g, cam, P().FilterParams(modes=P().MODE_ACCEL_BIAS))
    f12 = P().Filter(g, cam, P().FilterParams())
    x12 = np.concatenate([tr.t[0], tr.q[0], tr.v[0], tr.w[0]])
    L = P().lib()
    x = (ctypes.c_double * 13)(*x12)
    Pm = (ctypes.c_double * 144)(*np.eye(12).ravel())
    assert L.prism_filter_reset(f15.h, x, Pm, None) == 2
    x = (ctypes.c_double * 16)(*np.concatenate([x12, np.zeros(3)]))
    Pm = (ctypes.c_double * 225)(*np.eye(15).ravel())
    assert L.prism_filter_reset_bias(f12.h, x, Pm, None) == 2
    out = ctypes.c_void_p()
    assert L.prism_filter_bias_state_ptr(f12.h, ctypes.byref(out)) == 2
    assert L.prism_filter_bias_state_ptr(f15.h, ctypes.byref(out)) == 0 and out.value
    f12.reset(x12, np.diag([1e-6] * 6 + [1e-4] * 6))
    f12.map.init()
    nbytes = ctypes.c_size_t()
    assert L.prism_filter_save_bytes(ctypes.byref(f12.cfg), ctypes.byref(nbytes)) == 0
    buf = torch.empty(nbytes.value, dtype=torch.uint8, device=DEV)
    assert L.prism_filter_save(f12.h, ctypes.c_void_p(buf.data_ptr()), nbytes.value, None) == 0
    torch.cuda.synchronize()
    assert L.prism_filter_load(f15.h, ctypes.c_void_p(buf.data_ptr()), nbytes.value, None) == 1
    assert b"state" in L.prism_last_error()


@pytest.mark.parametrize("mode", ["dt2", "factor1", "irls"])
def test_each_paper_mode_changes_the_step(mode):
    """Each literal form on its own changes the filter's output the way the
    oracle's does: one P2 step with the mode against the default step, on
    the GPU and in the oracle, moves the state by the same amount."""
    bit = {"dt2": P().MODE_TRANSITION_DT2, "factor1": P().MODE_LAPLACE_FACTOR1, "irls": P().MODE_IRLS_L1}[mode]
    banner(f"filter 64^3 80x60 one mode {mode}")
    base = _filter_run(64, 80, 2, 0)[1]
    mod = _filter_run(64, 80, 2, 0, modes=bit)[1]
    (tg0, qg0, vg0, _, Pg0), (to0, qo0, vo0, _, Po0) = base[0:5], base[6:11]
    (tg1, qg1, vg1, _, Pg1), (to1, qo1, vo1, _, Po1) = mod[0:5], mod[6:11]
    d_gpu = np.concatenate([tg1 - tg0, vg1 - vg0, (Pg1 - Pg0).ravel()])
    d_orc = np.concatenate([to1 - to0, vo1 - vo0, (Po1 - Po0).ravel()])
    print(f"[{mode}] |change| gpu {np.linalg.norm(d_gpu):.3e} oracle {np.linalg.norm(d_orc):.3e} "
          f"difference {np.linalg.norm(d_gpu - d_orc):.3e}", flush=True)
    assert np.linalg.norm(d_orc) > 1e-9
    assert np.linalg.norm(d_gpu - d_orc) <= 1e-2 * np.linalg.norm(d_orc) + 1e-9


def _degenerate_run(P0, frames):
    """GPU filter and oracle filter stepped on the same frames; `frames` maps
    a step index to a replacement (depth, rgb) pair."""
    c = synth.trajectory_case(seed=4, n=64, width=80, height=60, n_samples=32, n_frames=3)
    tr = c["traj"]
    g = grid_of(c["scene"], 0)
    f = P().Filter(g, cam_of(c["cam"]), P().FilterParams(objective=0))
    f.map.init()
    x0 = np.concatenate([tr.t[0], tr.q[0], tr.v[0], tr.w[0]])
    f.reset(x0, P0)
    og = orc.grid_from_scene(c["scene"])
    mean = np.zeros((4, 64, 64, 64)); mean[0] = np.float32(-0.001)
    of = orc.Filter(og, orc.cam_from(c["cam"]), orc.Params(objective="p2"),
                    dict(t=tr.t[0], q=tr.q[0], v=tr.v[0], w=tr.w[0]), P0, mean, np.full_like(mean, 1e4))
    out = []
    for i in range(3):
        d, rgb = frames.get(i, (c["depth"][i], c["rgb"][i]))
        u = tr.u[i - 1] if i else None
        f.step(t(d), t(rgb), t(u, torch.float64) if i else None)
        of.step(d.astype(np.float64), rgb.astype(np.float64), u)
        out.append((f.state(), of.s.t.copy(), of.s.q.copy(), np.concatenate([of.s.v, of.s.w]),
                    of.s.P.copy(), of.s.last["n_updated"]))
    return out


def _state_close(s, to, qo, vo, Po, rel_P=1e-9):
    assert np.linalg.norm(np.array(s.pose.t) - to) <= 1e-9
    assert rot_angle(np.array(s.pose.q), qo) <= 1e-9
    assert np.linalg.norm(np.concatenate([s.v, s.w]) - vo) <= 1e-9
    Pg = np.array(s.P).reshape(12, 12)
    assert np.linalg.norm(Pg - Po) <= rel_P * np.linalg.norm(Po)


def test_filter_step_without_valid_pixels():
    """A frame with no valid depth: the flag is raised, nothing is fused and
    the state is the pure prediction, as in the oracle."""
    banner("filter degenerate: zero depth frame")
    c0 = synth.trajectory_case(seed=4, n=64, width=80, height=60, n_samples=32, n_frames=3)
    zero = (np.zeros_like(c0["depth"][1]), c0["rgb"][1])
    P0 = np.diag([1e-6] * 6 + [1e-4] * 6)
    out = _degenerate_run(P0, {1: zero})
    s, to, qo, vo, Po, nu_o = out[1]
    print(f"flags {s.flags} n_updated {s.n_updated}", flush=True)
    assert s.flags & P().FLAG_NO_VALID_PIXELS
    assert not s.flags & P().FLAG_CHOL_FALLBACK
    assert s.n_updated == 0 and nu_o == 0
    _state_close(s, to, qo, vo, Po)
    s, to, qo, vo, Po, nu_o = out[2]   # the next frame tracks again
    assert s.flags == 0
    assert abs(int(s.n_updated) - nu_o) <= 10


def test_filter_step_with_improper_covariance():
    """A state covariance whose predicted pose block is not positive definite:
    the fallback flags are raised and the step keeps the predicted mean and
    covariance while the map is still updated at that pose."""
    banner("filter degenerate: P0 = -I")
    out = _degenerate_run(-np.eye(12), {})
    for i in (1, 2):
        s, to, qo, vo, Po, nu_o = out[i]
        print(f"step {i}: flags {s.flags} n_updated {s.n_updated} / {nu_o}", flush=True)
        assert s.flags & P().FLAG_CHOL_FALLBACK and s.flags & P().FLAG_PRIOR_NOT_PD
        _state_close(s, to, qo, vo, Po, rel_P=1e-12)
        assert abs(int(s.n_updated) - nu_o) <= 10


def test_filter_bias_state_degenerate_steps():
    """The 15-D state's degenerate steps against the oracle: an improper
    covariance (the pose block of -I predicts no proper prior) keeps the
    predicted mean, bias and 15x15 covariance; a frame without valid depth is
    pure prediction followed by the combination."""
    banner("15-D state degenerate steps")
    c = synth.trajectory_case(seed=4, n=64, width=80, height=60, n_samples=32, n_frames=3)
    tr = c["traj"]
    for case, P0, frames in (("improper", -np.eye(15), {}),
                             ("no depth", np.diag([1e-6] * 6 + [1e-4] * 6 + [1e-4] * 3),
                              {1: (np.zeros_like(c["depth"][1]), c["rgb"][1])})):
        f = P().Filter(grid_of(c["scene"], 0), cam_of(c["cam"]), P().FilterParams(modes=P().MODE_ACCEL_BIAS))
        f.map.init()
        b0 = np.array([0.02, -0.01, 0.03])
        f.reset(np.concatenate([tr.t[0], tr.q[0], tr.v[0], tr.w[0], b0]), P0)
        mean = np.zeros((4, 64, 64, 64)); mean[0] = np.float32(-0.001)
        of = orc.Filter(orc.grid_from_scene(c["scene"]), orc.cam_from(c["cam"]),
                        orc.Params(objective="p2", accel_bias=True, sigma_bias=0.001),
                        dict(t=tr.t[0], q=tr.q[0], v=tr.v[0], w=tr.w[0], b=b0), P0, mean, np.full_like(mean, 1e4))
        for i in range(3):
            d, rgb = frames.get(i, (c["depth"][i], c["rgb"][i]))
            u = tr.u_body[i - 1] if i else None
            f.step(t(d), t(rgb), t(u, torch.float64) if i else None)
            of.step(d.astype(np.float64), rgb.astype(np.float64), u)
            if i == 0:
                continue
            s, xb = f.state(), f.bias_state()
            Pg = np.array(xb.P).reshape(15, 15)
            print(f"[{case}] step {i}: flags {s.flags}, |db| {np.linalg.norm(np.array(xb.b) - of.s.b):.1e}, "
                  f"P {np.linalg.norm(Pg - of.s.P) / np.linalg.norm(of.s.P):.1e}", flush=True)
            if case == "improper":
                assert s.flags & P().FLAG_CHOL_FALLBACK and s.flags & P().FLAG_PRIOR_NOT_PD
                np.testing.assert_array_equal(np.array(xb.b), b0)
            elif i == 1:
                assert s.flags & P().FLAG_NO_VALID_PIXELS and not s.flags & P().FLAG_CHOL_FALLBACK
            # a degenerate step is prediction (and combination) only: FP64 on
            # both sides; the tracked step after the frame without depth has
            # the bar of any filter step
            tol = 1e-9 if case == "improper" or i == 1 else 1e-5
            assert np.linalg.norm(np.array(s.pose.t) - of.s.t) <= tol
            assert rot_angle(np.array(s.pose.q), of.s.q) <= tol
            assert np.linalg.norm(np.array(xb.b) - of.s.b) <= tol
            assert np.linalg.norm(Pg - of.s.P) <= (1e-9 if tol == 1e-9 else 1e-4) * np.linalg.norm(of.s.P)


# ---------------------------------------------------------------------------
# map inference by gradient descent through the renderer
# ---------------------------------------------------------------------------
def _gd_inputs(seed=5):
    c = synth.trajectory_case(seed=2, n=64, width=80, height=60, n_samples=32, n_frames=1)
    mean, _ = synth.gt_map(c["scene"])
    rng = np.random.default_rng(seed)
    m0 = np.asarray(mean, np.float32)
    m0 = (m0 + np.concatenate([rng.normal(0, 0.01, (1,) + m0.shape[1:]),
                               rng.normal(0, 0.05, (3,) + m0.shape[1:])]).astype(np.float32)).astype(np.float32)
    v0 = rng.uniform(0.5, 2.0, m0.shape).astype(np.float32)
    tr = c["traj"]
    pose = np.concatenate([tr.t[0], tr.q[0]])
    return c, m0, v0, pose


def test_map_gd_matches_oracle():
    """Descent mapping against the oracle: objective before every step, the
    means after the first step (same decisions on both sides) and after three
    (the first crossings of the second and third renders may differ on rays
    whose occupancy lands within rounding of tau)."""
    banner("map_gd 64^3 80x60, 3 steps")
    c, m0, v0, pose = _gd_inputs()
    g = grid_of(c["scene"], 0)
    cam = cam_of(c["cam"])
    og, oc = orc.grid_from_scene(c["scene"]), orc.cam_from(c["cam"])
    p = orc.Params()
    w = P().Weights.make(p.b_geo, p.b_rgb, p.gate_geo, p.gate_rgb)
    lro, lrc = 3e-6, 3e-3
    D, C, pt = t(c["depth"][0]), t(c["rgb"][0]), P().poses_tensor(pose)
    ws = P().map_gd_workspace(g, cam)
    prior = gpu_map(g, m0, v0)
    ref1, cost1 = orc.map_gd(og, m0.astype(np.float64), v0.astype(np.float64), oc, pose, c["depth"][0],
                             c["rgb"][0], p, lro, lrc, 1)
    ref3, cost3 = orc.map_gd(og, m0.astype(np.float64), v0.astype(np.float64), oc, pose, c["depth"][0],
                             c["rgb"][0], p, lro, lrc, 3)
    tol = lambda b: 1e-6 * np.maximum(np.abs(b), 1e-2)
    for n_iters, ref, rcost in ((1, ref1, cost1), (3, ref3, cost3)):
        vm = P().VoxelMap(g)
        vm.buf.copy_(prior.buf)
        cost = torch.zeros(n_iters, dtype=torch.float64, device=DEV)
        P().map_gd(g, vm, cam, pt, D, C, w, lro, lrc, n_iters, ws, cost)
        torch.cuda.synchronize()
        mg, vg = vm.to_dense()
        mg, vg = mg.cpu().numpy().astype(np.float64), vg.cpu().numpy()
        cg = cost.cpu().numpy()
        print(f"{n_iters} steps: cost gpu {cg} oracle {np.array(rcost)}", flush=True)
        np.testing.assert_allclose(cg, rcost, rtol=1e-5)
        assert np.array_equal(vg, v0), "descent must leave the variances"
        bad = np.abs(mg - ref) > tol(ref)
        moved = np.count_nonzero(ref != m0)
        print(f"  voxels moved {moved}, outside tolerance {bad.sum()}, max err {np.abs(mg - ref).max():.3e}",
              flush=True)
        assert moved > 10000
        if n_iters == 1:
            assert not bad.any()
        else:
            assert bad.sum() <= 1e-3 * moved
        # untouched voxels keep their exact values
        same = ref == m0
        assert np.array_equal(mg[same & ~bad], m0.astype(np.float64)[same & ~bad])
        # the gradient accumulators are left zero, the brick summary current
        nv = g.n ** 3
        assert not ws[:4 * nv * 8].view(torch.float64).any()
        vr = P().VoxelMap(g)
        vr.buf.copy_(vm.buf)
        vr.refresh()
        torch.cuda.synchronize()
        assert torch.equal(vr.buf, vm.buf), "brick summary not maintained"


def test_map_gd_edge_cases():
    """Zero steps and a frame without valid depth leave the map bitwise as it
    was (objective 0 at the previous means); repeated calls through one
    workspace agree bit for bit; BF16 maps are refused."""
    banner("map_gd edge cases")
    c, m0, v0, pose = _gd_inputs(seed=6)
    g = grid_of(c["scene"], 0)
    cam = cam_of(c["cam"])
    w = P().Weights.make()
    pt = P().poses_tensor(pose)
    ws = P().map_gd_workspace(g, cam)
    prior = gpu_map(g, m0, v0)
    vm = P().VoxelMap(g)
    vm.buf.copy_(prior.buf)
    P().map_gd(g, vm, cam, pt, t(c["depth"][0]), t(c["rgb"][0]), w, 1e-6, 1e-3, 0, ws)
    cost = torch.full((2,), -1.0, dtype=torch.float64, device=DEV)
    P().map_gd(g, vm, cam, pt, t(np.zeros_like(c["depth"][0])), t(c["rgb"][0]), w, 1e-6, 1e-3, 2, ws, cost)
    torch.cuda.synchronize()
    assert torch.equal(vm.buf[:8 * g.n ** 3 * 4], prior.buf[:8 * g.n ** 3 * 4])
    assert cost.cpu().tolist() == [0.0, 0.0]
    outs = []
    for _ in range(2):
        vm.buf.copy_(prior.buf)
        P().map_gd(g, vm, cam, pt, t(c["depth"][0]), t(c["rgb"][0]), w, 3e-6, 3e-3, 2, ws)
        outs.append(vm.to_dense()[0].clone())
    torch.cuda.synchronize()
    # double-precision accumulation makes the order of the atomic adds
    # invisible in all but (in principle) a handful of roundings
    ndiff = int((outs[0] != outs[1]).sum())
    print(f"repeat: {ndiff} voxel values differ", flush=True)
    assert ndiff <= 4
    gb = grid_of(c["scene"], 1)
    vb = gpu_map(gb, m0, v0)
    with pytest.raises(P().PrismError, match="FP32"):
        P().map_gd(gb, vb, cam, pt, t(c["depth"][0]), t(c["rgb"][0]), w, 1e-6, 1e-3, 1,
                   P().map_gd_workspace(gb, cam))


# ---------------------------------------------------------------------------
# the paper's pose optimiser (Adam without momentum on sampled pixels)
# ---------------------------------------------------------------------------
def test_filter_adam_matches_oracle():
    """Filter steps whose state filter is the App. G optimiser (100 steps of
    200 sampled pixels, some indices repeated or outside the image) against
    the oracle filter on the same frames and samples."""
    banner("filter adam 64^3 80x60, 2 steps x 100 Adam steps")
    c = synth.trajectory_case(seed=2, n=64, width=80, height=60, n_samples=32, n_frames=3)
    tr = c["traj"]
    g = grid_of(c["scene"], 0)
    f = P().Filter(g, cam_of(c["cam"]), P().FilterParams(objective=0))
    f.map.init()
    x0 = np.concatenate([tr.t[0], tr.q[0], tr.v[0], tr.w[0]])
    P0 = np.diag([1e-6] * 6 + [1e-4] * 6)
    f.reset(x0, P0)
    og = orc.grid_from_scene(c["scene"])
    mean = np.zeros((4, 64, 64, 64)); mean[0] = np.float32(-0.001)
    of = orc.Filter(og, orc.cam_from(c["cam"]), orc.Params(objective="p2"),
                    dict(t=tr.t[0], q=tr.q[0], v=tr.v[0], w=tr.w[0]), P0, mean, np.full_like(mean, 1e4))
    ap = P().AdamParams.make(n_steps=100, n_pixels=200)
    H, W = c["cam"].height, c["cam"].width
    for i in range(3):
        pix = synth.sample_pixels(10 + i, ap.n_steps, ap.n_pixels, H, W)
        pix[3, :4] = pix[3, 4:8]
        pix[5, 0], pix[7, 1] = -1, H * W + 5
        u = tr.u[i - 1] if i else None
        f.step_adam(t(c["depth"][i]), t(c["rgb"][i]), t(u, torch.float64) if i else None, ap,
                    t(pix, torch.int32))
        of.step(c["depth"][i].astype(np.float64), c["rgb"][i].astype(np.float64), u,
                adam=dict(pixels=pix, lr_t=ap.lr_t, lr_r=ap.lr_r, beta2=ap.beta2, eps=ap.eps))
        s = f.state()
        dt_ = np.linalg.norm(np.array(s.pose.t) - of.s.t)
        dr = rot_angle(np.array(s.pose.q), of.s.q)
        print(f"step {i}: flags {s.flags} |dt| {dt_:.3e} dR {dr:.3e} (moved {np.linalg.norm(of.s.t - tr.t[i]):.4f} "
              f"m from truth)", flush=True)
        assert s.flags == 0
        assert dt_ <= 1e-5 and dr <= 1e-5
        Pg = np.array(s.P).reshape(12, 12)
        assert np.linalg.norm(Pg - of.s.P) <= 1e-4 * np.linalg.norm(of.s.P)
        assert abs(int(s.n_updated) - of.s.last["n_updated"]) <= max(10, 1e-4 * of.s.last["n_updated"])


@pytest.mark.parametrize("n_pixels,n_steps,lr_r", [(1, 3, 0.00036), (64, 1, 0.00036), (255, 4, 0.00036),
                                                   (256, 5, 0.00036), (257, 4, 0.00036), (700, 3, 0.02)])
def test_adam_sample_counts_and_step_sizes(n_pixels, n_steps, lr_r):
    """The optimiser at the edges of its work split (a lane's one sample, the
    256 of a step, more), odd and single step counts, and steps of more than
    0.01 rad, against the oracle: the pose bar of the filter tests."""
    banner(f"adam {n_pixels} pixels x {n_steps} steps, lr_r {lr_r}")
    c = synth.trajectory_case(seed=4, n=64, width=75, height=61, n_samples=32, n_frames=2)
    tr = c["traj"]
    f = P().Filter(grid_of(c["scene"], 0), cam_of(c["cam"]), P().FilterParams(objective=0))
    f.map.init()
    x0 = np.concatenate([tr.t[0], tr.q[0], tr.v[0], tr.w[0]])
    P0 = np.diag([1e-6] * 6 + [1e-4] * 6)
    f.reset(x0, P0)
    mean = np.zeros((4, 64, 64, 64)); mean[0] = np.float32(-0.001)
    of = orc.Filter(orc.grid_from_scene(c["scene"]), orc.cam_from(c["cam"]), orc.Params(objective="p2"),
                    dict(t=tr.t[0], q=tr.q[0], v=tr.v[0], w=tr.w[0]), P0, mean, np.full_like(mean, 1e4))
    ap = P().AdamParams.make(n_steps=n_steps, n_pixels=n_pixels, lr_r=lr_r)
    for i in range(2):
        pix = synth.sample_pixels(20 + i, n_steps, n_pixels, c["cam"].height, c["cam"].width)
        pix[-1, -1] = -7 if n_pixels > 1 else pix[-1, -1]
        u = tr.u[i - 1] if i else None
        f.step_adam(t(c["depth"][i]), t(c["rgb"][i]), t(u, torch.float64) if i else None, ap, t(pix, torch.int32))
        of.step(c["depth"][i].astype(np.float64), c["rgb"][i].astype(np.float64), u,
                adam=dict(pixels=pix, lr_t=ap.lr_t, lr_r=ap.lr_r, beta2=ap.beta2, eps=ap.eps))
    s = f.state()
    dt_ = np.linalg.norm(np.array(s.pose.t) - of.s.t)
    dr = rot_angle(np.array(s.pose.q), of.s.q)
    print(f"|dt| {dt_:.3e} dR {dr:.3e}", flush=True)
    assert dt_ <= 1e-5 and dr <= 1e-5


@pytest.mark.parametrize("lr_r", [1e-5, 0.03, 0.06, 0.4, 1.2])
def test_velocities_follow_the_pose_error(lr_r):
    """The posterior velocities are the predicted ones plus D times the error of
    the pose to its prior, for errors on both sides of the angle up to which the
    rotation's logarithm is a series (one optimiser step turns by sqrt(3) lr_r:
    1.7e-5, 0.052, 0.104, 0.69 and 2.08 rad).  Both sides start from the stored
    quaternions; the error in double precision is below 1e-14, times the sum of
    a row of D."""
    banner(f"velocities after a turn of {3 ** 0.5 * lr_r:.2g} rad")
    c = synth.trajectory_case(seed=4, n=64, width=75, height=61, n_samples=32, n_frames=2)
    tr = c["traj"]
    f = P().Filter(grid_of(c["scene"], 0), cam_of(c["cam"]), P().FilterParams(objective=0))
    f.map.init()
    f.reset(np.concatenate([tr.t[0], tr.q[0], tr.v[0], tr.w[0]]), np.diag([1e-6] * 6 + [1e-4] * 6))
    f.step(t(c["depth"][0]), t(c["rgb"][0]), None)
    ap = P().AdamParams.make(n_steps=1, n_pixels=64, lr_r=lr_r)
    pix = synth.sample_pixels(20, 1, 64, c["cam"].height, c["cam"].width)
    f.pose_update_adam(t(c["depth"][1]), t(c["rgb"][1]), t(tr.u[0], torch.float64), ap, t(pix, torch.int32))
    s = f.state()
    Ra, Rb = (orc.quat_to_rot(np.array(x.q)) for x in (s.iter, s.prior))
    e = np.concatenate([np.array(s.iter.t) - np.array(s.prior.t), orc.so3_log(Ra @ Rb.T)])
    assert abs(np.linalg.norm(e[3:]) - 3 ** 0.5 * lr_r) <= 1e-2 * lr_r
    D = np.array(s.D).reshape(6, 6)
    want = np.array(s.vel_prior) + D @ e
    got = np.concatenate([np.array(s.v), np.array(s.w)])
    assert np.all(np.abs(got - want) <= 1e-14 * (1.0 + np.abs(D).sum(1)) * max(1.0, np.abs(e).max()))


def test_adam_rejects_p1_and_bad_samples():
    banner("adam argument checks")
    c = synth.trajectory_case(seed=2, n=64, width=80, height=60, n_samples=32, n_frames=1)
    g = grid_of(c["scene"], 0)
    ap = P().AdamParams.make(n_steps=4, n_pixels=8)
    pix = torch.zeros((4, 8), dtype=torch.int32, device=DEV)
    f1 = P().Filter(g, cam_of(c["cam"]), P().FilterParams(objective=1))
    f1.map.init()
    with pytest.raises(P().PrismError, match="P2"):
        f1.step_adam(t(c["depth"][0]), t(c["rgb"][0]), None, ap, pix)
    f2 = P().Filter(g, cam_of(c["cam"]), P().FilterParams(objective=0))
    f2.map.init()
    with pytest.raises(P().PrismError, match="n_pixels"):
        f2.step_adam(t(c["depth"][0]), t(c["rgb"][0]), None, P().AdamParams.make(n_steps=4, n_pixels=0),
                     torch.zeros((4, 0), dtype=torch.int32, device=DEV))
    with pytest.raises(P().PrismError, match="beta2"):
        f2.step_adam(t(c["depth"][0]), t(c["rgb"][0]), None, P().AdamParams.make(n_steps=4, n_pixels=8, beta2=1.0),
                     pix)


# ---------------------------------------------------------------------------
# predictive rollouts
# ---------------------------------------------------------------------------
def test_rollout_15d_matches_oracle():
    """Rollout from a seeded 15-D belief (accelerometer bias, body-frame force
    controls) and the ground-truth map: sampled poses, the 16-value means and
    15x15 covariances, and the frames, against the oracle on the same
    belief, map and draws."""
    banner("rollout 15-D state, 64^3 80x60, 3 samples x 4 steps")
    c = synth.trajectory_case(seed=2, n=64, width=80, height=60, n_samples=32, n_frames=1)
    tr = c["traj"]
    g = grid_of(c["scene"], 0)
    mean, var = synth.gt_map(c["scene"])
    fp = P().FilterParams(objective=0, modes=P().MODE_ACCEL_BIAS, sigma_bias=0.01)
    f = P().Filter(g, cam_of(c["cam"]), fp, vmap=gpu_map(g, mean, var))
    rng = np.random.default_rng(8)
    A = rng.normal(size=(15, 15)) * 0.01
    Pb = A @ A.T + np.diag([1e-5] * 6 + [1e-4] * 6 + [1e-5] * 3)
    x = dict(t=tr.t[0], q=tr.q[0], v=tr.v[0], w=tr.w[0], b=np.array([0.02, -0.03, 0.01]))
    f.reset(np.concatenate([x["t"], x["q"], x["v"], x["w"], x["b"]]), Pb)
    k, S = 4, 3
    u = rng.normal(size=(k, 6)) + np.array([0.0, 0.0, 9.81, 0.0, 0.0, 0.0])
    z = rng.normal(size=(S, k + 1, 15))
    out = f.rollout(t(u, torch.float64), t(z, torch.float64), moments=True, frames=True)
    torch.cuda.synchronize()
    op = orc.Params(accel_bias=True, sigma_bias=fp.sigma_bias, gravity=tuple(fp.gravity))
    ref = orc.rollout(orc.grid_from_scene(c["scene"]), oracle_map_values(mean, 0), orc.cam_from(c["cam"]), x, Pb,
                      u, z, op)
    assert int(out["flags"].item()) == 0 and ref["ok"]
    pg = out["poses"].cpu().numpy()
    for s_ in range(S):
        for j in range(k):
            assert np.linalg.norm(orc.pose_error(pg[s_, j], ref["poses"][s_, j])) < 1e-9
    np.testing.assert_allclose(out["mean"].cpu().numpy(), ref["mean"], rtol=0, atol=1e-12)
    cg = out["cov"].cpu().numpy()
    assert cg.shape == (k, 15, 15)
    assert np.linalg.norm(cg - ref["cov"]) <= 1e-10 * np.linalg.norm(ref["cov"])
    for n in range(S * k):
        r = ref["frames"][n]
        mk = out["mask"][n].cpu().numpy()
        np.testing.assert_array_equal(mk, r["mask"])
        v = mk == 1
        assert np.all(depth_close(out["depth"][n].cpu().numpy()[v], r["depth"][v]))


def test_rollout_matches_oracle():
    """Rollout from a seeded belief and the ground-truth map: sampled poses,
    the closed-form moments and the frames rendered at the sampled poses
    against the oracle on the same belief, map and draws."""
    banner("rollout 64^3 80x60, 3 samples x 4 steps")
    c = synth.trajectory_case(seed=2, n=64, width=80, height=60, n_samples=32, n_frames=1)
    tr = c["traj"]
    g = grid_of(c["scene"], 0)
    cam = cam_of(c["cam"])
    mean, var = synth.gt_map(c["scene"])
    f = P().Filter(g, cam, P().FilterParams(objective=0), vmap=gpu_map(g, mean, var))
    rng = np.random.default_rng(7)
    A = rng.normal(size=(12, 12)) * 0.01
    Pb = A @ A.T + np.diag([1e-5] * 6 + [1e-4] * 6)
    x = dict(t=tr.t[0], q=tr.q[0], v=tr.v[0], w=tr.w[0])
    f.reset(np.concatenate([x["t"], x["q"], x["v"], x["w"]]), Pb)
    k, S = 4, 3
    u = rng.normal(size=(k, 6))
    z = rng.normal(size=(S, k + 1, 12))
    out = f.rollout(t(u, torch.float64), t(z, torch.float64), moments=True, frames=True)
    torch.cuda.synchronize()
    ref = orc.rollout(orc.grid_from_scene(c["scene"]), oracle_map_values(mean, 0), orc.cam_from(c["cam"]), x, Pb,
                      u, z, orc.Params())
    assert int(out["flags"].item()) == 0 and ref["ok"]
    pg = out["poses"].cpu().numpy()
    for s in range(S):
        for j in range(k):
            assert np.linalg.norm(orc.pose_error(pg[s, j], ref["poses"][s, j])) < 1e-9
    np.testing.assert_allclose(out["mean"].cpu().numpy(), ref["mean"], rtol=0, atol=1e-12)
    cg = out["cov"].cpu().numpy()
    assert np.linalg.norm(cg - ref["cov"]) <= 1e-10 * np.linalg.norm(ref["cov"])
    hk_fail = 0
    for n in range(S * k):
        r = ref["frames"][n]
        mk = out["mask"][n].cpu().numpy()
        hk_fail += int((mk != r["mask"]).sum())
        v = (mk == 1) & (r["mask"] == 1)
        d = out["depth"][n].cpu().numpy()
        assert np.all(depth_close(d[v], r["depth"][v]))
        rgb = out["rgb"][n].cpu().numpy()
        assert np.all(rgb_close(rgb[v], r["rgb"][v]))
    print(f"mask mismatches over {S * k} frames: {hk_fail}", flush=True)
    assert hk_fail == 0
    # an improper covariance: flag raised, samples start at the mean
    f.reset(np.concatenate([x["t"], x["q"], x["v"], x["w"]]), -np.eye(12))
    z0 = z.copy()
    z0[:, 1:] = 0.0
    out = f.rollout(t(u, torch.float64), t(z0, torch.float64), moments=False)
    ref = orc.rollout(None, None, None, x, -np.eye(12), u, z0, orc.Params(), frames=False)
    assert int(out["flags"].item()) == P().FLAG_CHOL_FALLBACK and not ref["ok"]
    pg = out["poses"].cpu().numpy()
    for s in range(S):
        assert np.linalg.norm(orc.pose_error(pg[s, 0], ref["poses"][s, 0])) < 1e-9


# ---------------------------------------------------------------------------
# the relative pose of the association recipe
# ---------------------------------------------------------------------------
def _write_state(f, field, values):
    """Overwrite a field of doubles of the filter's device state."""
    a = f._state_off + getattr(P().FilterState, field).offset
    v = torch.as_tensor(np.asarray(values, np.float64), device=DEV)
    f.state_buf[a:a + 8 * v.numel()].view(torch.float64).copy_(v)


def _flat_anchor(f, depth, rgb):
    """Replace the filter's anchor frame: the given images, everywhere valid,
    normals along the optical axis."""
    a = f.anchor()
    a["depth"].copy_(depth)
    a["rgb"].copy_(rgb)
    a["mask"].fill_(1)
    a["nmask"].fill_(1)
    a["normals"].copy_(torch.tensor([0.0, 0.0, -1.0], device=DEV).expand_as(a["normals"]))
    return a


@pytest.mark.parametrize("n_gn", [0, 1, 3])
@pytest.mark.parametrize("bias", [False, True])
def test_filter_tracks_from_its_stored_pose(n_gn, bias):
    """A filter's tracking objective is that of track_p2 at the pose it stores:
    the relative pose is formed from the stored quaternions.  A camera at rest
    that sees its anchor frame again: every residual is the rounding of the
    two poses' double-precision algebra, so a pose that differs from the
    stored one in its last bits gives other sums.  16x16 pixels are one row of
    sums, which both calls pass on unchanged: equal bit for bit."""
    banner(f"stored pose n_gn={n_gn} bias={bias}")
    n, W, H = 16, 16, 16
    grid = P().Grid.make(n, 0.2, (-1.6, -1.6, -1.6))
    cam = P().Camera.make(W, H, 12.0, 12.0, 8.0, 8.0, 0.1, 3.0, 16)
    rng = np.random.default_rng(5)
    D = t(rng.uniform(1.0, 2.0, (H, W)))
    C = t(rng.uniform(0.1, 0.9, (H, W, 3)))
    prm = P().FilterParams(n_gn=n_gn, modes=P().MODE_ACCEL_BIAS if bias else 0, gravity=(0.0, 0.0, 0.0))
    zero = torch.zeros(6, dtype=torch.float64, device=DEV)
    moved = 0
    for _ in range(6):
        q = rng.normal(size=4)
        q /= np.linalg.norm(q) * np.sign(q[0])
        f = P().Filter(grid, cam, prm)
        f.map.init()
        x0 = np.concatenate([rng.uniform(-0.3, 0.3, 3), q, np.zeros(9 if bias else 6)])
        f.reset(x0, np.diag([1e-4] * (15 if bias else 12)))
        f.step(D, C, None)
        anchor = _flat_anchor(f, D, C)
        prev = f.state().anchor
        f.pose_update(D, C, zero)
        s = f.state()
        pose, before = (np.array(list(p.t) + list(p.q)) for p in (s.iter, prev))
        out = P().track_p2(cam, P().poses_tensor(pose), P().poses_tensor(before), D, C, anchor, f.cfg.w)
        a, b = np.array(s.neq), out["neq"][0].cpu().numpy()
        assert a[28] >= 200
        moved += int(np.any(a[21:27] != 0.0))
        np.testing.assert_array_equal(a, b)
    assert moved >= 5     # rounding residuals, not exact zeros


def _fma64(a, b, c):
    """Round-to-nearest of the exact a b + c."""
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def _edge_cases(count):
    """Poses and cameras for which the relative translation rounds to another
    float when its sum of products is contracted, and the anchor pixel of the
    image centre is inside the image with one of the two floats only.  The
    current rotation is the identity; yields (anchor quaternion, camera
    translation, fx, fy, inside) with `inside` by the uncontracted recipe."""
    f32, rng, u0 = np.float32, np.random.default_rng(11), 8
    D, out, want = f32(1.0), [], [count // 2, count - count // 2]
    while sum(want):
        # anchor: a small rotation, so that row 0 of its transpose is near x
        q = np.concatenate([[1.0], rng.normal(scale=0.05, size=3)])
        q /= np.linalg.norm(q)
        w, x, y, z = (float(v) for v in q)
        nrm = float(np.sqrt(w * w + x * x + y * y + z * z))
        w, x, y, z = w / nrm, x / nrm, y / nrm, z / nrm
        Q = [[1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y - w * z), 2.0 * (x * z + w * y)],
             [2.0 * (x * y + w * z), 1.0 - 2.0 * (x * x + z * z), 2.0 * (y * z - w * x)],
             [2.0 * (x * z - w * y), 2.0 * (y * z + w * x), 1.0 - 2.0 * (x * x + y * y)]]
        # a translation whose x in the anchor frame lies next to the middle of two floats
        d = [float(v) for v in rng.uniform(-0.1, 0.1, 3)]
        lo = f32(rng.uniform(-0.9, -0.6))
        mid = 0.5 * (float(lo) + float(np.nextafter(lo, f32(0.0))))
        d[0] = (mid - Q[1][0] * d[1] - Q[2][0] * d[2]) / Q[0][0]
        d[0] += float(np.spacing(d[0])) * int(rng.integers(-2, 3))

        def rel_t(a):
            p = [Q[k][a] * d[k] for k in range(3)]
            return f32((p[0] + p[1]) + p[2])
        fused = {f32(_fma64(Q[2][0], d[2], _fma64(Q[1][0], d[1], Q[0][0] * d[0]))),
                 f32(_fma64(Q[2][0], d[2], _fma64(Q[0][0], d[0], Q[1][0] * d[1])))}
        t0 = rel_t(0)
        if len(fused) > 1 or t0 in fused:
            continue
        # the centre pixel's point is (0, 0, D): its column in the anchor frame
        R = [f32(Q[2][a]) for a in range(3)]      # third column of Q^T I
        Y2 = f32(f32(R[2] * D) + rel_t(2))
        quot = [f32(f32(f32(R[0] * D) + tx) / Y2) for tx in (t0, fused.pop())]
        if quot[0] == quot[1] or Y2 <= 0.5:
            continue
        cx = f32(u0 + 0.5)
        fx = f32(float(cx) / -float(quot[0]))
        for _ in range(-8, 9):
            col = [f32(f32(fx * qq) + cx) for qq in quot]
            if (col[0] >= 0) != (col[1] >= 0):
                break
            fx = np.nextafter(fx, f32(0.0)) if col[0] < 0 else np.nextafter(fx, f32(100.0))
        else:
            continue
        inside = int(col[0] >= 0)
        if want[inside]:
            want[inside] -= 1
            out.append((q, d, float(fx), inside))
    return out


def test_adam_decides_without_contraction():
    """The optimiser's later steps place their samples with the relative pose
    of the recipe, products and sums rounded one by one.  Poses found so that
    a fused multiply-add anywhere in that sum moves the anchor pixel of the
    one sample across the image's border: a sample inside moves the iterate,
    one outside leaves it as predicted.  (The first of the two steps samples
    no pixel, so the second starts from the predicted pose.)"""
    banner("adam at the image border")
    W = H = 17
    grid = P().Grid.make(16, 0.2, (-1.6, -1.6, -1.6))
    D = torch.ones((H, W), device=DEV)
    C = torch.full((H, W, 3), 0.5, device=DEV)
    zero = torch.zeros(6, dtype=torch.float64, device=DEV)
    ap = P().AdamParams.make(n_steps=2, n_pixels=1)
    pixels = torch.tensor([[-1], [8 * W + 8]], dtype=torch.int32, device=DEV)
    for q, d, fx, inside in _edge_cases(12):
        cam = P().Camera.make(W, H, fx, 4.0, 8.5, 8.5, 0.1, 3.0, 16)
        f = P().Filter(grid, cam, P().FilterParams(gate_geo=1e6))
        f.map.init()
        f.reset(np.concatenate([d, [1.0, 0, 0, 0], np.zeros(6)]), np.diag([1e-4] * 12))
        f.step(D, C, None)
        _flat_anchor(f, D, C)
        _write_state(f, "anchor", np.concatenate([np.zeros(3), q]))
        f.pose_update_adam(D, C, zero, ap, pixels)
        s = f.state()
        assert list(s.prior.t) == d and list(s.prior.q)[1:] == [0.0, 0.0, 0.0]
        assert (list(s.iter.t) != d) == bool(inside), (q, d, fx, inside)
