"""Dense planes <-> the library's brick order, at grids whose brick rows do
and do not fill the four bricks a wavefront copies, for both storage types,
buffers aligned to 4 bytes only, and one side left out; and the brick summary
of maps whose last word of free-space bits is partly used."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, P, banner
from test_gpu_freebits import _aux

pytestmark = pytest.mark.gpu


def _bricks(x, n):
    nb = n // 8
    return x.reshape(-1, nb, 8, nb, 8, nb, 8).permute(0, 1, 3, 5, 2, 4, 6).reshape(x.shape[0], -1)


def _unaligned(x):
    """The same values in a contiguous tensor whose data starts 4 bytes past a 16-byte boundary."""
    buf = torch.empty(x.numel() + 4, dtype=x.dtype, device=x.device)
    out = buf[1:1 + x.numel()].view(x.shape)
    out.copy_(x)
    assert out.data_ptr() % 16 == 4
    return out


@pytest.mark.parametrize("n", [8, 24, 40, 64, 136])
@pytest.mark.parametrize("dtype", [0, 1])
def test_dense_and_brick_order(n, dtype):
    banner(f"dense <-> bricks n={n} dtype={dtype}")
    pr = P()
    g = torch.Generator(device=DEV)
    g.manual_seed(n + dtype)
    mean = torch.randn((4, n, n, n), generator=g, device=DEV)
    mean[0, : n // 2] = -mean[0, : n // 2].abs()       # free bricks and others
    var = torch.rand((4, n, n, n), generator=g, device=DEV) + 0.1
    held = (lambda x: x.to(torch.bfloat16).float()) if dtype else (lambda x: x)
    grid = pr.Grid.make(n, 0.05, dtype=dtype)
    for load in (lambda x: x, _unaligned):
        vm = pr.VoxelMap(grid).init()
        vm.from_dense(load(mean), load(var))
        raw = vm.buf[: 8 * n ** 3 * (2 if dtype else 4)].view(torch.bfloat16 if dtype else torch.float32)
        both = torch.cat([_bricks(held(mean), n), _bricks(held(var), n)])
        assert torch.equal(raw.float().view(8, -1), both)
        m2, v2 = vm.to_dense()
        assert torch.equal(m2, held(mean)) and torch.equal(v2, held(var))
        bmax, plain, dil = _aux(grid, vm)
        occ = _bricks(held(mean)[:1], n).view(-1, 512).amax(1).cpu().numpy()
        assert np.array_equal(bmax, occ)
        nb3 = (n // 8) ** 3
        bits = np.unpackbits(np.ascontiguousarray(plain).view(np.uint8), bitorder="little")
        assert np.array_equal(bits[:nb3], occ <= 0) and not bits[nb3:].any()
        # the summary formed from the stored map, and after variances alone, is the same
        vm.refresh()
        assert all(np.array_equal(a, b) for a, b in zip(_aux(grid, vm), (bmax, plain, dil)))
        vm.from_dense(None, load(2 * var))
        assert all(np.array_equal(a, b) for a, b in zip(_aux(grid, vm), (bmax, plain, dil)))
        m2, v2 = vm.to_dense()
        assert torch.equal(m2, held(mean)) and torch.equal(v2, held(2 * var))


@pytest.mark.parametrize("n,channels", [(8, 1), (40, 3), (64, 8)])
def test_plane_copies(n, channels):
    banner(f"planes n={n} channels={channels}")
    pr = P()
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    dense = torch.randn((channels, n, n, n), generator=g, device=DEV)
    for load in (lambda x: x, _unaligned):
        bricks = pr.dense_to_bricks(n, load(dense))
        assert torch.equal(bricks, _bricks(dense, n))
        assert torch.equal(pr.bricks_to_dense(n, load(bricks)), dense)


@pytest.mark.parametrize("dtype", [0, 1])
def test_summary_of_maps_with_nan(dtype):
    """The summary of a loaded map is that of the stored means, NaN among
    them: the largest mean that is a number, and NaN (not free) for a brick
    that holds none."""
    banner(f"summary with NaN dtype={dtype}")
    n, nan = 16, float("nan")
    mean = torch.full((4, n, n, n), -0.5, device=DEV)
    mean[0, :8, :8, :8] = nan                                  # brick 0: no number
    mean[0, :8, :8, 8:] = nan                                  # brick 1: one number, negative
    mean[0, 3, 4, 13] = -0.25
    mean[0, :8, 8:, :8] = nan                                  # brick 2: one number, positive
    mean[0, 7, 15, 0] = 0.25
    mean[0, 8:, :8, :8] = nan                                  # brick 4: lowest finite value and -infinity
    mean[0, 8, 0, 0] = -float("inf")
    mean[0, 9, 1, 1] = torch.finfo(torch.float32).min if dtype == 0 else -3.0e38
    mean[0, 8:, 8:, 8:] = -float("inf")                        # brick 7
    grid = P().Grid.make(n, 0.05, dtype=dtype)
    vm = P().VoxelMap(grid).init()
    vm.from_dense(mean, None)
    held = (mean.to(torch.bfloat16).float() if dtype else mean).cpu().numpy()
    want = np.fmax.reduce(_bricks(torch.from_numpy(held[:1]), n).view(8, 512).numpy(), axis=1)
    bmax, plain, dil = _aux(grid, vm)
    np.testing.assert_array_equal(bmax, want)
    bits = np.unpackbits(np.ascontiguousarray(plain).view(np.uint8), bitorder="little")
    assert np.array_equal(bits[:8], want <= 0) and np.isnan(want[0]) and not bits[0]
    vm.refresh()
    assert all(np.array_equal(a, b, equal_nan=a.dtype == np.float32)
               for a, b in zip(_aux(grid, vm), (bmax, plain, dil)))
