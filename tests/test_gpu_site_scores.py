"""GPU: site extraction from volumes that hold infinities, NaN, signed zeros and denormal
numbers.  Scores rank by the order of their bits (sign taken into account: NaN with a clear
sign above +infinity, with a set one below -infinity), ties to the lower index, so the result
is that of a volume of the voxels' ranks."""
import numpy as np
import pytest

from oracle.site_extract import extract

pytestmark = pytest.mark.gpu


def ranks(vol):
    """Distinct whole numbers in the order of the scores."""
    b = vol.reshape(-1).view(np.uint32)
    key = np.where(b >> 31, ~b, b | np.uint32(0x80000000))
    order = np.lexsort((-np.arange(len(b)), key))        # ascending; of equal scores the higher index first
    r = np.empty(len(b), np.float32)
    r[order] = np.arange(len(b), dtype=np.float32)
    return r.reshape(vol.shape)


@pytest.mark.parametrize("share", [0.0005, 0.01, 0.6])
@pytest.mark.parametrize("shape,top_n", [((36, 36, 36), 200), ((7, 9, 11), 693), ((40, 33, 31), 1000)])
def test_scores_that_are_not_finite(shape, top_n, share):
    import gpu_common as gc
    import paper_2303_09916_amd as D
    torch = gc.torch_cuda()
    rng = np.random.default_rng(11)
    vol = (rng.random(shape) - 0.3).astype(np.float32)
    odd = np.array([0x7F800000, 0xFF800000, 0x7FC00000, 0xFFC00000, 0x7F800001, 0xFFFFFFFF, 0x7FFFFFFF, 0, 0x80000000, 1,
                    0x80000001, 0x7F7FFFFF, 0xFF7FFFFF], np.uint32)
    flat = vol.reshape(-1).view(np.uint32)
    at = rng.random(flat.size) < share
    flat[at] = rng.choice(odd, int(at.sum()))
    nz, ny, nx = shape
    ws = gc.dev_bytes(torch, D.dsdp_site_points_workspace_bytes(top_n))
    d = torch.from_numpy(vol.view(np.int32).copy()).cuda().view(torch.float32)
    pts, lab, _ = D.dsdp_site_points(d, (nx, ny, nz), (0.0, 0.0, 0.0), 1.0, top_n, ws)
    order, _, olab, _ = extract(ranks(vol), (0.0, 0.0, 0.0), 1.0, top_n)
    ijk = np.round(pts).astype(np.int64)
    np.testing.assert_array_equal(ijk[:, 2] * ny * nx + ijk[:, 1] * nx + ijk[:, 0], order)
    np.testing.assert_array_equal(lab, olab)
