"""GPU test of the batched launches' search for the solve of a tile, 64 solves at a time:
counts of admitted solves at the edges of 64, every result bitwise that of the same solve
on a single grid."""
import numpy as np
import pytest

from paper_1909_13263_amd import hjw
from paper_1909_13263_amd import workloads as W

pytestmark = pytest.mark.gpu


def _problem(i):
    return W.burgers2d(16 + 7 * (i % 13), 0.01 + 0.001 * (i % 3), ny=20 + 5 * (i % 11))


@pytest.fixture(scope="module")
def alone():
    out = []
    for i in range(130):
        pr = _problem(i)
        g = hjw.grid_for(pr, hjw.FP32_MIXED)
        g.set_phi(pr.phi0())
        info = g.step_to(pr.t_final, pr.cfl)
        out.append((info.steps, g.get_phi()))
        g.close()
    return out


@pytest.mark.parametrize("count", [1, 63, 64, 65, 127, 128, 129, 130])
def test_every_count_of_solves_finds_its_tiles(alone, count):
    srv = hjw.Server(hjw.FP32_MIXED, pool_bytes=256 << 20, max_active=count)
    ids = {srv.submit(_problem(i)): i for i in range(count)}
    results = srv.drain()
    assert len(results) == count
    for res in results:
        steps, phi = alone[ids[res.rid]]
        assert res.status == hjw.OK and res.info.steps == steps
        assert np.array_equal(res.phi, phi), ids[res.rid]
    srv.close()
