"""The tile sweep (teams of waves handing pencil faces to each other in LDS)
against the pencil sweep, bit for bit, and the oracle: meshes whose pencil grid
is no multiple of a tile, x extents around the face words' wrap (below 8, at
and next to multiples of 8) and the phases of the pencils' chunk grids (more
than 8 pencil diagonals), one block and more blocks than items, and ticket
rings longer than a team's (several items per team)."""
import numpy as np
import pytest

import oracle
from parity import parity_err, sampled_fp32_excess, sign_change_voxels
from synthetic.workloads import SourceSpec, random_small_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
dsn = pytest.importorskip("paper_1910_11335_amd")

MESHES = [(1, 17, 9), (3, 40, 24), (7, 33, 8), (8, 9, 41), (9, 70, 25), (15, 16, 72), (17, 66, 34), (24, 8, 9)]


@pytest.mark.parametrize("fixup,density", [(1, False), (0, True)])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", MESHES, ids=["x".join(map(str, n)) for n in MESHES])
def test_tile_shapes_equal_pencil_shapes(n, precision, fixup, density):
    p = random_small_problem(60 + n[0], n=n, sn=4, L=1, G=2, n_mat=3, fixup=fixup, density=density)
    ext = np.array([p.nx * p.dx, p.ny * p.dy, p.nz * p.dz])
    srcs = [SourceSpec(position=(-2.3, 0.6 * ext[1], 0.45 * ext[2]), spectrum=np.array([1.0, 0.4])),
            SourceSpec(position=tuple(0.37 * ext + 0.011), spectrum=np.array([0.5, 1.0]))]
    fixed = [3, 2]
    h = dsn.Problem(p, precision)
    default = h.solve(srcs, fixed_iters=fixed)["phi_total"]
    h.set_sweep_shape(1, 64)
    ref = h.solve(srcs, fixed_iters=fixed)["phi_total"]
    assert torch.equal(default, ref)
    want = oracle.solve(p, srcs[0], fixed_iters=fixed)["phi_total"]
    got = ref[0].cpu().numpy()
    if precision == "fp64":
        assert parity_err(got, want, p) < 1e-12
    else:  # 1e-4, or where pure DD cancels 4x what single-precision cells alone do
        golden = dict(idx=np.arange(p.V), phi=want, gmax=np.abs(want).max(1),
                      sc=np.array([sign_change_voxels(w, n) for w in want]))
        if not fixup:
            golden["phi_single"] = oracle.solve(p, srcs[0], fixed_iters=fixed, cell_single=True)["phi_total"]
        assert sampled_fp32_excess(got, golden)[0] < 1.0
    for r in (2, 4):
        for blocks in (1, 3, 2000):
            h.set_sweep_shape(1, blocks, 0, r)
            out = h.solve(srcs, fixed_iters=fixed)
            assert out["sweep_shape"] == (1, blocks, 0, r)
            assert torch.equal(out["phi_total"], ref), (blocks, r)
    h.close()
