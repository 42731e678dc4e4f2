"""The adjoint on tile shapes: its forward, reversed, recording and transposed
sweeps against the same handle type pinned to pencil items, and the pencils in
FP64 against the oracle.  Every team size, meshes whose pencil grid is no
multiple of a tile, with several tile diagonals, and x extents below 8 (face
words in plain slots) and above.  With the fixup the cells are optically thick,
so many of them have fixed axes."""
import numpy as np
import pytest

import oracle
from synthetic.workloads import SourceSpec, random_small_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
dsn = pytest.importorskip("paper_1910_11335_amd")

MESHES = [(3, 40, 24), (5, 17, 70), (17, 34, 26), (9, 72, 40)]
TILES = {"fp32": [(1, 2), (2, 2), (1, 4), (2, 4)], "fp64": [(1, 2), (1, 4)]}


def _problem(n, fixup):
    p = random_small_problem(200 + n[0], n=n, sn=6, L=1, G=2, n_mat=3, fixup=fixup, density=True)
    if fixup:
        p.sigma_t = p.sigma_t * 6.0
        p.sigma_s = p.sigma_s * 6.0
    ext = np.array([p.nx * p.dx, p.ny * p.dy, p.nz * p.dz])
    s = SourceSpec(position=(-2.3, 0.6 * ext[1], 0.45 * ext[2]), spectrum=np.array([1.0, 0.4]))
    W = np.random.default_rng(n[1]).uniform(0, 1, (p.G, p.V))
    return p, s, W


def _grad_err(got, want, floor=1e-6):
    sel = np.abs(want) > floor * np.abs(want).max()
    return (np.abs(got - want)[sel] / np.abs(want[sel])).max()


@pytest.mark.parametrize("fixup", [0, 1])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", MESHES, ids=["x".join(map(str, n)) for n in MESHES])
def test_adjoint_on_tiles_equals_pencils(n, precision, fixup):
    """phi bit for bit; J and the gradient, which sum in any order, to 1e-12
    (1e4 terms of 1e-16 each at most)."""
    p, s, W = _problem(n, fixup)
    Wt = torch.tensor(W, device="cuda")
    kw = dict(fixed_iters=[3, 4], want_phi=True)
    h = dsn.Problem(p, precision)
    h.set_sweep_shape(1, 64)
    ref = h.adjoint(s, Wt, **kw)
    phi, grad = ref["phi_total"].clone(), ref["grad"].cpu().numpy()
    for w, r in TILES[precision]:
        for blocks in (2, 500):
            h.set_sweep_shape(w, blocks, 0, r)
            out = h.adjoint(s, Wt, **kw)
            assert torch.equal(out["phi_total"], phi), (w, r, blocks)
            assert abs(out["J"] / ref["J"] - 1) < 1e-12, (w, r, blocks)
            assert _grad_err(out["grad"].cpu().numpy(), grad) < 1e-12, (w, r, blocks)
    h.close()


@pytest.mark.parametrize("fixup", [0, 1])
@pytest.mark.parametrize("n", MESHES[:3], ids=["x".join(map(str, n)) for n in MESHES[:3]])
def test_adjoint_on_pencils_fp64_matches_oracle(n, fixup):
    p, s, W = _problem(n, fixup)
    ref = oracle.adjoint(p, s, W, tol=1e-13)
    if fixup:
        assert oracle.solve(p, s, tol=1e-13)["nneg"] > 0
    h = dsn.Problem(p, "fp64")
    h.set_sweep_shape(2, 64)
    out = h.adjoint(s, torch.tensor(W, device="cuda"), tol=1e-13)
    assert abs(out["J"] / ref["J"] - 1) < 1e-12
    assert _grad_err(out["grad"].cpu().numpy(), ref["grad"]) < 1e-10
    assert list(out["iters"][0]) == list(ref["iters_fwd"])
    assert list(out["iters"][1]) == list(ref["iters_adj"])
    h.close()
