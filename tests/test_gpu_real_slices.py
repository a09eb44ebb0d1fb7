"""Real-secondaries runs of few electrons go in slices of the lineage budget, which pays only
where secondaries follow: gases that cannot ionise run whole generations, and slices grow where
little is ionised.  Slices change the schedule only, also for the lineages of the other trial
strategies, of moving targets and of the relativistic mover, which pass through the saved
state at every slice's end."""
import math

import pytest

import synth
from swarm_testutil import sort_by_id

pytestmark = pytest.mark.gpu

REAL = {"secondaries": synth.REAL}


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "fp32"])
def test_gases_without_ionisation_run_in_one_launch(gpu, precision):
    s = gpu.Swarm.from_config(synth.cfg1_maxwell().scaled(**REAL), precision)
    for n_e, n_c in ((25, 5000), (20_000, 500)):
        s.run(n_e, n_c, 3)
        assert s.launches() == (1, 0), n_e


def test_slices_grow_where_little_is_ionised(gpu):
    """Doubled from 64 or 128 collisions on, or after four slices of one length (25 electrons say
    little about a rate below one in four hundred): far fewer launches than the budget has slices."""
    cfg = synth.SwarmConfig(synth.mixture_ar_co2(), synth.td_to_field(5.0), **REAL)
    for n_e, n_c in ((2000, 4000), (20_000, 3000)):
        s = gpu.Swarm.from_config(cfg, 1)
        s.run(n_e, n_c, 3)
        assert s.launches()[0] <= math.log2(n_c / 64) + 2, (n_e, s.launches())
    s = gpu.Swarm.from_config(cfg, 1, capacity=4000)
    s.run(25, 10_000, 3)
    assert s.launches()[0] <= 10_000 / 64 / 3, s.launches()
    s = gpu.Swarm.from_config(cfg.scaled(E_V_per_m=synth.td_to_field(100.0)), 1)
    s.run(2000, 1000, 3)
    assert s.launches()[0] >= 1000 / 128            # an avalanche stays in short ones


OPTIONS = {"variable": {"trial_strategy": 1}, "variable-grace3": {"trial_strategy": 1, "trial_grace": 3},
           "binned": {"trial_strategy": 2, "trial_grace": 40}, "thermal": {"thermal_targets": 1},
           "thermal-variable": {"thermal_targets": 1, "trial_strategy": 1},
           "relativistic": {"relativistic": 1, "B_T": 0.0}}


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("option", list(OPTIONS))
def test_slices_change_no_record_of_any_option(gpu, option, precision):
    cfg = synth.cfg3_mixture_real().scaled(**OPTIONS[option])
    if cfg.relativistic and precision == 1:
        pytest.skip("the relativistic mover runs in FP64")
    for n_e, n_c in ((60, 500), (5000, 300)):
        out = []
        for opts in ({}, {"park_lanes": -1}, {"park_lanes": -1, "block_size": 128}):
            s = gpu.Swarm.from_config(cfg, precision)
            s.set_launch_opts(opts)
            s.run(n_e, n_c, 5)
            assert (s.launches()[1] > 0) == (not opts)
            out.append(sort_by_id(s.records()).tobytes())
        assert out[0] == out[1] == out[2], n_e
