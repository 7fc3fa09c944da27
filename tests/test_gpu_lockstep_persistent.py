"""The persistent lockstep launch over many generations (a cap on its wavefronts,
here beyond what the GPU holds, asks for it; calls of fewer than 48 generations take
it by default), whose middle generations otherwise run in the streaming form: small
grids against the oracle, full-size ones against the synchronous kernel."""
import numpy as np
import pytest

from gpu_helpers import assert_same_state, oracle_after, say
from paper_2405_03605_amd import SCHEDULE_ASYNC, GARun
from paper_2405_03605_amd.workloads import run_config

pytestmark = pytest.mark.gpu

UNCAPPED = 1 << 20


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("kw,gens", [
    (dict(width=64, height=64, pop=32, sites=64, k=5), (500, 500)),
    (dict(width=100, height=37, pop=8, sites=32, k=3), (400, 400)),
    (dict(width=256, height=256, pop=32, sites=32), (100, 100)),
], ids=lambda e: f"{e['width']}x{e['height']}" if isinstance(e, dict) else str(sum(e)))
def test_persistent_launches_match_the_oracle(kw, gens):
    say(f"persistent lockstep {kw}, {gens} generations")
    run = GARun(run_config(schedule=SCHEDULE_ASYNC, **kw))
    run.set_async(UNCAPPED)
    for n in gens:
        run.step(n)
    islands = kw["width"] * kw["height"]
    assert run.async_waits() == 0
    assert run.async_taken() == islands * (sum(gens) - 1)
    assert_same_state(run.read(), oracle_after(run_config(**kw), sum(gens)), f"persistent {kw}")
    run.close()


@pytest.mark.parametrize("kw,gens,cap", [
    (dict(width=1024, height=512), (500, 500), UNCAPPED),
    (dict(width=256, height=256), (1000, 2000), UNCAPPED),
    (dict(width=256, height=256), (47,) * 12, 0),
], ids=["1024x512", "256x256", "256x256-short-calls"])
def test_persistent_launches_at_full_size(kw, gens, cap):
    cfg = run_config(pop=32, sites=32, k=2, **kw)
    say(f"persistent lockstep vs synchronous {kw}, {sum(gens)} generations")
    sync = GARun(cfg)
    sync.step(sum(gens))
    want = sync.read(outbox=False)
    sync.close()
    run = GARun(dict(cfg, schedule=SCHEDULE_ASYNC))
    run.set_async(cap)
    for n in gens:
        run.step(n)
    got = run.read()
    assert run.async_waits() == 0
    run.close()
    for key in ("f", "T", "D"):
        assert np.array_equal(got[key].view(np.uint32), want[key].view(np.uint32)), key


@pytest.mark.parametrize("pop,ipw,wpg,width,height,model", [
    (4, 32, 1, 512, 448, 1), (1, 64, 1, 1024, 448, 0), (1, 64, 2, 1024, 480, 0)])
def test_groups_by_the_lds_they_are_given(pop, ipw, wpg, width, height, model):
    # 28 and 30 wavefronts a CU by the LDS asked for, 25 and 28 by the LDS given out
    kw = dict(width=width, height=height, pop=pop, sites=32, k=2, model=model)
    say(f"persistent lockstep at {ipw} x {wpg}, {kw}")
    sync = GARun(run_config(**kw))
    sync.step(60)
    want = sync.read(outbox=False)
    sync.close()
    run = GARun(run_config(schedule=SCHEDULE_ASYNC, **kw))
    run.set_launch(ipw, wpg)
    run.set_async(UNCAPPED)
    run.step(60)
    got = run.read()
    assert run.async_waits() == 0
    assert run.async_taken() == width * height * 59
    run.close()
    for key in ("f", "T", "D") + (("P",) if model else ()):
        assert np.array_equal(got[key].view(np.uint32), want[key].view(np.uint32)), key
