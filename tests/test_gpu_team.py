"""Runs with few electrons give each one a team of lanes.  That changes the schedule only: the
records are the bits of the one-lane kernel, which a run takes when its block size is asked
for.  Sizes around the edges of waves and of the rule's ranges; one to 92 channels (the channel
search in one round, in several, and behind a bisection); every option of the kernels."""
import numpy as np
import pytest

import synth
from swarm_testutil import sort_by_id

pytestmark = pytest.mark.gpu

ONE_LANE = {"block_size": 128}


def _pair(sw, cfg, precision, n_e, n_c, seed=3):
    s = sw.Swarm.from_config(cfg, precision)
    s.run(n_e, n_c, seed)
    team = (s.records(), s.tallies())
    s.set_launch_opts(ONE_LANE)
    s.run(n_e, n_c, seed)
    return team, (s.records(), s.tallies())


GASES = {
    "maxwell": synth.cfg1_maxwell(),
    "argon-1Td": synth.cfg2_argon_sweep()[0],
    "argon-1000Td": synth.cfg2_argon_sweep()[31],
    "mixture": synth.cfg3_mixture_real().scaled(secondaries=0),
    "mixture-2Td": synth.SwarmConfig(synth.mixture_ar_co2(0.93, 0.07), synth.td_to_field(2.4)),
    "92-channels": synth.cfg5_request(13),
}
OPTIONS = {"plain": {}, "variable": {"trial_strategy": 1}, "variable-grace3": {"trial_strategy": 1, "trial_grace": 3},
           "binned": {"trial_strategy": 2, "trial_grace": 40}, "thermal": {"thermal_targets": 1}}


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("gas", list(GASES))
def test_team_records_equal_one_lane_records(gpu, gas, precision):
    for name, opt in OPTIONS.items():
        cfg = GASES[gas].scaled(**opt)
        for n_e, n_c in ((1, 400), (63, 120)) + (((1027, 60), (5000, 40), (13001, 25)) if name == "plain" else ()):
            (a, ta), (b, tb) = _pair(gpu, cfg, precision, n_e, n_c)
            assert a.tobytes() == b.tobytes(), (name, n_e)
            assert ta["n_real"] == tb["n_real"]


def test_team_relativistic_and_anisotropic(gpu):
    base = GASES["mixture"]
    aniso = base.scaled(components=[base.components[0].with_scattering(1), base.components[1].with_scattering(2, 0.5)])
    for cfg, precision in ((base.scaled(relativistic=1), 0), (GASES["argon-1Td"].scaled(relativistic=1), 0), (aniso, 0),
                           (aniso, 1)):
        (a, _), (b, _) = _pair(gpu, cfg, precision, 70, 60)
        assert a.tobytes() == b.tobytes()


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "fp32"])
def test_team_lineages_equal_one_lane_lineages(gpu, precision):
    """Real secondaries: in slices of the lineage budget with eager and default parking, in whole
    generations (no parking), budgets around a slice's end, and a capacity that overflows."""
    cfg = synth.cfg3_mixture_real()
    for n_e, n_c in ((3, 900), (700, 900), (40, 63), (40, 64), (40, 65), (4100, 130), (30500, 260)):
        ref = None
        for shape in ({"park_lanes": -1, **ONE_LANE}, {"park_lanes": -1}, {}, ONE_LANE, {"park_lanes": 64}):
            s = gpu.Swarm.from_config(cfg, precision)
            s.set_launch_opts(shape)
            s.run(n_e, n_c, 5)
            got = sort_by_id(s.records())
            if ref is None:
                ref = got
                assert s.launches()[1] == 0
            assert got.tobytes() == ref.tobytes(), (n_e, n_c, shape)
    s = gpu.Swarm.from_config(cfg, precision, capacity=800)
    with pytest.raises(gpu.SwarmError) as err:
        s.run(700, 2000, 5)
    assert err.value.status == gpu.SWARM_ERR_CAPACITY
    rec = s.records()
    assert len(rec) == 800 and len(np.unique(rec["id"])) == 800


def test_team_batches_and_served_requests(gpu):
    cfgs = [GASES["argon-1Td"], GASES["mixture-2Td"], GASES["92-channels"]]
    jobs = [(300, 90, 1), (37, 200, 2), (1100, 40, 3)]
    one = [gpu.Swarm.from_config(c, 1) for c in cfgs]
    gpu.swarm_batch_run([h.h for h in one], jobs, ONE_LANE)
    team = [gpu.Swarm.from_config(c, 1) for c in cfgs]
    gpu.swarm_batch_run([h.h for h in team], jobs, {})
    srv = gpu.swarm_server_create(1 << 30, gpu.SWARM_FP32_MIXED, quantum_collisions=17)
    try:
        got = [gpu.swarm_server_submit_records(srv, c.components, gpu.params_from_config(c, 1), *j)
               for c, j in zip(cfgs, jobs)]
        gpu.swarm_server_drain(srv)
        for (ticket, rec), a, b in zip(got, one, team):
            assert gpu.swarm_server_poll(srv, ticket)[0]
            assert a.records().tobytes() == b.records().tobytes() == rec.tobytes()
    finally:
        gpu.swarm_server_destroy(srv)
