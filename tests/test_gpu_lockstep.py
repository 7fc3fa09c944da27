"""Asynchronous runs at the default pacing, whose middle generations run in the
streaming form: state, genomes taken and the generation of the last one from
each side as in the persistent launch (a cap on its wavefronts asks for that),
and the mail left so that skewed interleavings after it, which read genomes late
and overwritten, go on alike."""
import numpy as np
import pytest

from gpu_helpers import assert_same_state, oracle_after, say
from paper_2405_03605_amd import ASYNC_UNPACED, SCHEDULE_ASYNC, GARun
from paper_2405_03605_amd.workloads import run_config

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


SHAPES = [
    dict(width=1, height=1, pop=64, sites=32, k=2, seed=91),
    dict(width=2, height=5, pop=32, sites=64, k=3, seed=92),
    dict(width=40, height=1, pop=16, sites=32, k=2, model=1, seed=93),
    dict(width=33, height=29, pop=8, sites=32, k=2, seed=94),
    dict(width=21, height=50, pop=4, sites=64, k=5, model=2, policy=2, seed=95),
    dict(width=50, height=40, pop=32, sites=32, k=2, seed=96),
]


@pytest.mark.parametrize("edge", SHAPES,
                         ids=lambda e: "-".join(f"{k}{v}" for k, v in e.items()))
def test_streamed_lockstep_leaves_what_the_persistent_launch_does(edge):
    cfg = run_config(schedule=SCHEDULE_ASYNC, **edge)
    say(f"lockstep through the streaming form, {cfg}")
    pair = []
    for cap in (0, 1024):
        run = GARun(cfg)
        seen = []
        for n in (48, 49, 5, 51):
            run.set_async(cap)
            run.step(n)
            seen.append((run.async_taken(), run.async_last_taken().copy()))
        assert_same_state(run.read(), oracle_after(run_config(**edge), 153), f"cap {cap}")
        run.set_async(1, ASYNC_UNPACED, 2)   # genomes arrive late from here on
        run.step(7)
        run.set_async(cap)
        run.step(50)
        run.set_async(1, ASYNC_UNPACED, 3)
        run.step(6)
        seen.append((run.async_taken(), run.async_last_taken().copy()))
        assert run.async_waits() == 0
        pair.append((seen, run.read()))
        run.close()
    for (ta, la), (tb, lb) in zip(pair[0][0], pair[1][0]):
        assert ta == tb
        assert (la == lb).all()
    for name in ("f", "T", "D"):
        assert np.array_equal(pair[0][1][name].view(np.uint32), pair[1][1][name].view(np.uint32))


def test_streamed_lockstep_past_2_32_generations():
    edge = dict(width=24, height=17, pop=32, sites=32, k=2, seed=97)
    say(f"lockstep past 2^32 generations, {edge}")
    out = []
    for cap in (0, 1024):
        run = GARun(run_config(schedule=SCHEDULE_ASYNC, **edge))
        run.step(3)
        got = run.read()
        run.write(got["f"], got["T"], got["D"], None, 2 ** 32 - 30)
        run.set_async(cap)
        run.step(60)
        out.append((run.async_taken(), run.async_last_taken().copy(), run.read()))
        assert run.async_waits() == 0
        run.close()
    assert out[0][0] == out[1][0]
    assert (out[0][1] == out[1][1]).all()
    for name in ("f", "T", "D"):
        assert np.array_equal(out[0][2][name].view(np.uint32), out[1][2][name].view(np.uint32))
