"""GPU: the paths of the site extraction kernel (sizes around its four-voxel loads,
an unaligned volume, plateaus that overflow the candidate list, long chains of
linked points) against the oracle; integer results, equal bit for bit."""
import numpy as np
import pytest

from oracle.site_extract import extract

pytestmark = pytest.mark.gpu


def volume(kind, shape, rng):
    v = rng.random(shape).astype(np.float32)
    if kind == "plateau":      # more voxels at the cut than the candidate list holds
        v = (v > 0.3).astype(np.float32)
    elif kind == "zeros":
        v[:] = 0.0
    elif kind == "snake":      # one long chain of linked points and noise below it
        v *= 0.5
        i = np.arange(shape[2])
        v[(i // 3) % shape[0], np.abs(i - shape[1]) % shape[1], i] = 1.0 + rng.random(shape[2])
    elif kind == "signed":
        v = v - 0.5
        v.reshape(-1)[::7] = -0.0
    return v


@pytest.mark.parametrize("kind,shape,top_n,shift", [
    ("noise", (1, 1, 1), 5, 0),
    ("noise", (1, 1, 7), 7, 1),           # not a multiple of four, unaligned
    ("signed", (3, 5, 11), 100, 0),
    ("signed", (16, 16, 16), 1000, 3),    # one voxel per strip, unaligned
    ("noise", (17, 16, 16), 1024, 0),     # strips of one and two voxels
    ("noise", (61, 64, 63), 1024, 2),
    ("noise", (64, 64, 64), 20, 0),
    ("plateau", (24, 24, 24), 200, 0),
    ("zeros", (20, 20, 20), 333, 1),
    ("snake", (12, 40, 200), 200, 0),
])
def test_site_paths(kind, shape, top_n, shift):
    import gpu_common as gc
    import paper_2303_09916_amd as D
    torch = gc.torch_cuda()
    vol = volume(kind, shape, np.random.default_rng(7))
    flat = torch.zeros(vol.size + shift, dtype=torch.float32, device="cuda")
    flat[shift:] = torch.from_numpy(vol.reshape(-1)).cuda()
    ws = gc.dev_bytes(torch, D.dsdp_site_points_workspace_bytes(top_n))
    nz, ny, nx = shape
    origin = (0.0, 0.0, 0.0)
    for _ in range(2):
        pts, lab, cen = D.dsdp_site_points(flat[shift:], (nx, ny, nz), origin, 1.0, top_n, ws)
        order, opts, olab, ocen = extract(vol, origin, 1.0, top_n)
        ijk = np.round(pts).astype(np.int64)
        np.testing.assert_array_equal(ijk[:, 2] * ny * nx + ijk[:, 1] * nx + ijk[:, 0], order)
        np.testing.assert_array_equal(lab, olab)
        np.testing.assert_array_equal(cen, ocen)
