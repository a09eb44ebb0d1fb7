"""Real-secondaries runs of a few dozen electrons that ionise nothing: their slices grow after a
few, although so few electrons say little about a small rate of ionisation."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_e, most", [(25, 16), (50, 10), (200, 8)])
def test_slices_of_few_electrons_grow(gpu, n_e, most):
    """Argon at 3 Td ionises nothing.  `most` follows from the rule: slices of 64, doubled when a
    quarter of a secondary would be less than a four-hundredth of the electrons of one slice."""
    s = gpu.Swarm.from_config(synth.SwarmConfig([synth.argon_like()], synth.td_to_field(3.0), secondaries=synth.REAL), 1)
    s.run(n_e, 10_000, 3)
    assert s.tallies()["n_created"] == 0
    assert s.launches()[0] <= most, s.launches()
