"""GPU: the map kernel at the edges of its tiles, of its staging and of its split
over map types, against the FP64 oracle with the tolerance of the other map
tests (|dE| <= 1e-4 * sum|terms| + 4e-6 * sum|h'| + tie + 1e-6, and the same rule per
gradient component)."""
import numpy as np
import pytest

import oracle as O
from synth import make_receptor, make_box
from helpers import box32

pytestmark = pytest.mark.gpu

ALL = list(range(17))


@pytest.mark.parametrize("size,spacing,n_rec,types", [
    ((1.5, 1.5, 1.5), 0.5, 200, ALL),             # 4^3 nodes: one wave's block
    ((2.0, 4.0, 2.0), 0.5, 200, [16]),            # 5 x 9 x 5: one node past a block and a tile
    ((3.5, 3.5, 1.5), 0.5, 200, [0, 1]),          # 8 x 8 x 4: a whole tile, two maps of one radius
    ((40.0, 24.0, 30.0), 2.0, 4000, [8, 0, 10]),  # wide tiles: more atoms than one staging pass holds
    ((5.0, 6.0, 7.0), 0.375, 60, [13, 5, 2, 9, 0, 11, 12, 4, 3, 7]),   # ten maps in the caller's own order
])
def test_map_tiles(size, spacing, n_rec, types):
    import gpu_common as gc
    rec = make_receptor(n_rec, radius=35.0 if n_rec > 1000 else 12.0, seed=n_rec)
    box = box32(make_box(rec.pocket, size, spacing=spacing))
    xyz = np.array(rec.xyz, dtype=np.float32)
    n, origin = gc.D.dsdp_grid_dims(box)
    xyz[0] = origin + np.float32(box["spacing"]) * np.array([1, 1, 1], np.float32)   # an atom on a node
    ref = O.Grid(xyz, rec.types, box, types)
    g = gc.GpuGrid(xyz, rec.types, box, types)
    m = g.maps_host()
    assert m.shape == ref.maps.shape and np.isfinite(m).all()
    tolE = 1e-4 * ref.mass[..., 0] + 4e-6 * ref.mass[..., 1] + ref.tie[..., 0] + 1e-6
    tolG = 1e-4 * ref.mass[..., 1] + ref.tie[..., 1] + 1e-6
    assert np.all(np.abs(m[..., 0] - ref.maps[..., 0]) <= tolE)
    # at the node under the atom the gradient has no direction (the oracle's node,
    # in double precision, lies a rounding error off the atom): energy only
    defined = np.ones(m.shape[:-1], bool)
    defined[:, 1, 1, 1] = False
    assert np.all((np.max(np.abs(m[..., 1:] - ref.maps[..., 1:]), axis=-1) <= tolG)[defined])


def test_map_bits_do_not_depend_on_the_other_maps():
    """A type's map is the same, bit for bit, alone and in any run of types."""
    import gpu_common as gc
    rec = make_receptor(300, radius=12.0, seed=9)
    box = box32(make_box(rec.pocket, (9.0, 7.7, 8.3), spacing=0.4))
    whole = gc.GpuGrid(rec.xyz, rec.types, box, ALL).maps_host()
    for types in ([0], [16, 3], [1, 8, 2, 10, 0], ALL[::-1], ALL[:12]):
        part = gc.GpuGrid(rec.xyz, rec.types, box, types).maps_host()
        for k, t in enumerate(types):
            assert np.array_equal(part[k], whole[t]), (types, t)
