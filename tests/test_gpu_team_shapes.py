"""That runs of few electrons do run them in teams, of every size the library uses, down to a
gas of one channel, and that their records are those of one lane per electron.  (With a
constant collision rate every trial of the Maxwell gas hits, and it keeps one lane; a trial
frequency of three times its rate gives its electrons null collisions, and teams.)"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

ONE_LANE = {"block_size": 128}
MAXWELL = (synth.cfg1_maxwell().scaled(user_majorant=3.0e12), ((20, 60), (1000, 40), (10_000, 20), (40_000, 12)), {2, 4, 8, 16})
MIXTURE = (synth.SwarmConfig(synth.mixture_ar_co2(), synth.td_to_field(60.0), B_T=0.4, B_angle_rad=0.8),
           ((20, 60), (1000, 40), (8000, 20), (30_000, 12)), {2, 4, 8, 16})
CHANNELS_92 = (synth.cfg5_request(13), ((20, 60), (20_000, 12)), {16})


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("gas", [MAXWELL, MIXTURE, CHANNELS_92], ids=["one-channel", "28-channels", "92-channels"])
def test_every_team_size_gives_the_one_lane_records(gpu, gas, precision):
    cfg, runs, want = gas
    sizes = set()
    for n_e, n_c in runs:
        s = gpu.Swarm.from_config(cfg, precision)
        s.run(n_e, n_c, 11)
        team, rec = s.team(), s.records()
        assert team in (2, 4, 8, 16), (n_e, team)
        sizes.add(team)
        s.set_launch_opts(ONE_LANE)
        s.run(n_e, n_c, 11)
        assert s.team() == 1
        assert rec.tobytes() == s.records().tobytes(), n_e
    assert sizes == want, sizes


def test_team_of_the_last_run_is_reported(gpu):
    cfg = MIXTURE[0]
    s = gpu.Swarm.from_config(cfg, 1)
    with pytest.raises(gpu.SwarmError):
        s.team()
    s.run(500_000, 3, 1)                       # enough electrons for one lane each
    assert s.team() == 1
    s.run(64, 30, 1)
    assert s.team() > 1
    s.set_trace(np.arange(4), 64)              # traced runs take the one-lane kernel
    s.run(64, 30, 1)
    assert s.team() == 1
    real = gpu.Swarm.from_config(cfg.scaled(secondaries=1), 1)
    real.run(64, 30, 1)
    assert real.team() > 1
    hs = [gpu.Swarm.from_config(cfg, 1) for _ in range(2)]
    for opts, teams in (({}, True), (ONE_LANE, False)):
        gpu.swarm_batch_run([h.h for h in hs], [(40, 30, 1), (50, 30, 2)], opts)
        assert all((h.team() > 1) == teams for h in hs)
