"""Asynchronous runs at the default pacing whose generation was written: back to an
earlier one, to one past 2^30 more and across 2^31 and 2^32. The launch must wait for its
neighbours' new headers whatever generation the old ones name, so state and genomes
taken are the synchronous schedule's."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_same_state, say
from paper_2405_03605_amd import SCHEDULE_ASYNC, GARun
from paper_2405_03605_amd.workloads import run_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base", [5, 6, 2 ** 30 + 7, 2 ** 31 - 20, 2 ** 32 - 21])
@pytest.mark.parametrize("kw", [dict(width=24, height=17, pop=32, sites=32, k=2, seed=97),
                                dict(width=64, height=48, pop=16, sites=64, k=3, seed=98)],
                         ids=lambda k: f"{k['width']}x{k['height']}")
def test_written_generation(kw, base):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    say(f"async set to generation {base}, {kw}")
    run = GARun(run_config(schedule=SCHEDULE_ASYNC, **kw))
    islands = kw["width"] * kw["height"]
    run.step(47)
    for steps in (40, 33):
        mid, before = run.read(), run.async_taken()
        run.write(mid["f"], mid["T"], mid["D"], None, base)
        run.step(steps)      # persistent launches: calls below 48 generations
        ref = oracle.OracleRun(run_config(**kw))
        ref.set_population(mid["f"], mid["T"], mid["D"])
        ref.set_outbox(np.zeros(islands, np.uint8), np.zeros(islands, np.uint8),
                       np.zeros(islands, np.float32), np.zeros(islands, np.uint32),
                       np.zeros((islands, ref.words), np.uint32))
        ref.set_generation(base)
        ref.step(steps)
        assert run.async_waits() == 0
        assert run.async_taken() - before == islands * (steps - 1)
        assert_same_state(run.read(), ref, f"from {base}")
    run.close()
