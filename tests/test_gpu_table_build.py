"""The table build sums the rates of a node over its channels in groups of eight and stages their
constants 64 at a time: channel counts around both, against the oracle's tables.  Each
rate carries a few roundings more than the oracle's where a power law extends a table (about
1e-14 relative), and a sum of positive rates no more than its worst term plus one rounding
each, 129 x 1.1e-16: 1e-13 in all."""
import numpy as np
import pytest

import oracle
import synth
from synth.tables import ELASTIC

pytestmark = pytest.mark.gpu


def _gas(n):
    pool = [c for i in range(40) for comp in synth.cfg5_request(i).components for c in comp.channels]
    elastic = next(c for c in pool if c.kind == ELASTIC)
    others = [c for c in pool if c.kind != ELASTIC][:n - 1]
    comp = synth.cfg5_request(0).components[0]
    return synth.SwarmConfig([type(comp)(comp.mass_amu, 1.0, others[: (n - 1) // 2] + [elastic] + others[(n - 1) // 2:])],
                             synth.td_to_field(50.0), B_T=0.5, B_angle_rad=1.0)


@pytest.mark.parametrize("n", [1, 7, 8, 9, 63, 64, 65, 72, 129])
def test_tables_of_many_channels(gpu, n):
    cfg = _gas(n)
    nodes, cum, majorant = gpu.Swarm.from_config(cfg, gpu.SWARM_FP64).tables()
    m = oracle.OracleModel.from_config(cfg)
    onodes, ocum = m.tables()
    assert cum.shape == ocum.shape and n in cum.shape
    assert np.array_equal(nodes, onodes)
    np.testing.assert_allclose(cum, ocum, rtol=1e-13, atol=0)
    assert abs(majorant / m.majorant - 1) < 1e-13
