"""Paths of the two sweep kernels that depend on the launch shape in use: the
ticket decode against the diagonal table in device memory and the bounded waits,
each on a handle pinned to pencil items and on one pinned to tiles."""
import numpy as np
import pytest

import oracle
from parity import parity_err
from synthetic.workloads import SourceSpec, random_small_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
dsn = pytest.importorskip("paper_1910_11335_amd")

SHAPES = {"pencils": (1, 64, 0, 0), "tiles": (1, 64, 0, 2)}


@pytest.mark.parametrize("shape", SHAPES)
def test_long_mesh_decodes_tickets_from_device_memory(shape):
    """258 pencils along y: 258 pencil diagonals, more than a pencil block
    keeps in LDS, or 65 tile diagonals, more than a wave has lanes."""
    p = random_small_problem(17, n=(2, 2064, 8), sn=4, L=1, G=2, n_mat=3, fixup=1)
    ext = np.array([p.nx * p.dx, p.ny * p.dy, p.nz * p.dz])
    s = SourceSpec(position=(0.5 * ext[0], -2.0, 0.5 * ext[2]), spectrum=np.array([1.0, 0.4]))
    fixed = [3, 2]
    want = oracle.solve(p, s, fixed_iters=fixed)["phi_total"]
    h = dsn.Problem(p, "fp64")
    h.set_sweep_shape(*SHAPES[shape])
    out = h.solve([s], fixed_iters=fixed)
    assert out["sweep_shape"] == SHAPES[shape]
    assert parity_err(out["phi_total"][0].cpu().numpy(), want, p) < 1e-12
    h.close()


@pytest.mark.parametrize("fixup", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_dependency_timeout_reports_error_and_recovers(shape, fixup):
    """A wait limit of one poll (forced from the host) makes a downstream wave
    give up at its first missing face: the sweeps abort, the call reports a
    device error, and the same handle then solves normally.  (More blocks
    than a diagonal has items, or no wave would have to wait.)"""
    wpb, _, xcd, relay = SHAPES[shape]
    p = random_small_problem(9, n=(24, 40, 35), sn=8, L=1, G=2, n_mat=2, fixup=fixup)
    ext = np.array([p.nx * p.dx, p.ny * p.dy, p.nz * p.dz])
    s = SourceSpec(position=(ext[0] + 7.0, 0.5 * ext[1], 0.5 * ext[2]), spectrum=np.array([1.0, 0.5]))
    h = dsn.Problem(p, "fp64")
    ref = h.solve([s], fixed_iters=[2, 2])["phi_total"].clone()
    h.set_sweep_shape(wpb, 2000, xcd, relay)
    with pytest.raises(dsn.DsnError) as err:
        h.solve([s], fixed_iters=[1, 1], wait_limit=1)
    assert err.value.status == dsn.dsn.DSN_ERR_DEVICE
    assert torch.equal(h.solve([s], fixed_iters=[2, 2])["phi_total"], ref)
    h.close()
