"""The autotuner knows the library's own launch shape, which runs the electrons of small batches
in teams of lanes: it times it and returns it (service_waves -1) where it is the fastest."""
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_small_batches_are_tuned_to_the_librarys_own_shape(gpu):
    """16 argon fields x 50 electrons: one lane per electron takes four times as long as teams."""
    hs = [gpu.Swarm.from_config(c, gpu.SWARM_FP32_MIXED) for c in synth.cfg2_argon_sweep()[::2]]
    jobs = [(50, 1500, i) for i in range(len(hs))]
    handles = [h.h for h in hs]
    best = gpu.swarm_autotune(handles, jobs, 300)
    assert best["service_waves"] == -1
    gpu.swarm_batch_run(handles, jobs, best)
    assert hs[0].team() > 1
    tuned = [h.records().tobytes() for h in hs]
    gpu.swarm_batch_run(handles, jobs, {"block_size": 128})
    assert hs[0].team() == 1
    assert [h.records().tobytes() for h in hs] == tuned


def test_own_shape_ignores_the_shape_fields(gpu):
    s = gpu.Swarm.from_config(synth.cfg2_argon_sweep()[3], gpu.SWARM_FP32_MIXED)
    s.set_launch_opts({"block_size": 512, "chunk": 2048, "pending_trigger": 7, "service_waves": -1})
    s.run(50, 300, 1)
    own = s.team(), s.records().tobytes()
    s.set_launch_opts({})
    s.run(50, 300, 1)
    assert own == (s.team(), s.records().tobytes()) and own[0] > 1
