"""The LDS-resident form where its wavefronts and tiles meet, bit for bit
against the oracle: tilings of more small tiles than the plain register budget
holds at once (the dense variant), wavefronts with more than 64 neighbours
outside their tile, more passes than a wavefront keeps in registers, every
tournament size, and a run set back to an earlier generation (the exchange area
then holds later generations than the ones waited for)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_same_state, oracle_after, say
from paper_2405_03605_amd import FORM_RESIDENT, GARun
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
    # dense: 4,900 and 4,356 one-wavefront tiles, over 16 per CU
    (dict(width=70, height=70, pop=64, sites=32, k=2, seed=41), (1, 1)),
    (dict(width=66, height=66, pop=64, sites=64, k=5, seed=42), (1, 1)),
    # two columns of 64 one-agent islands: 64 + 2 pairs outside a wavefront's share
    (dict(width=6, height=128, pop=1, sites=32, k=1, seed=43), (2, 64)),
    (dict(width=7, height=66, pop=2, sites=64, k=7, model=1, seed=44), (1, 33)),
    # two, four and eight passes a wavefront
    (dict(width=40, height=33, pop=16, sites=32, k=4, seed=45), (40, 11)),
    (dict(width=64, height=35, pop=8, sites=32, k=6, seed=46), (32, 32)),
    (dict(width=64, height=48, pop=4, sites=32, k=3, seed=47), (64, 24)),
    (dict(width=50, height=40, pop=8, sites=32, k=8, model=2, policy=1, seed=48), (25, 20)),
    # closed islands: nothing crosses between tiles
    (dict(width=24, height=16, pop=32, sites=32, k=2, migration=0, seed=49), (8, 8)),
]


@pytest.mark.parametrize("edge,tiles", SHAPES,
                         ids=lambda e: "-".join(f"{k}{v}" for k, v in e.items())
                         if isinstance(e, dict) else f"t{e[0]}x{e[1]}")
def test_tiles_match_oracle(edge, tiles):
    cfg = run_config(**edge)
    say(f"tiles {tiles} on {cfg}")
    run = GARun(cfg)
    run.set_launch(form=FORM_RESIDENT)
    run.set_tiles(*tiles)
    assert run.tiles()[:2] == tiles
    for n in (1, 7, 40):
        run.step(n)
    assert_same_state(run.read(), oracle_after(cfg, 48), f"tiles {tiles} {edge}")
    run.close()


def test_set_back_to_an_earlier_generation():
    cfg = run_config(width=48, height=40, pop=32, sites=32, k=2, seed=50)
    say(f"resident run set back, {cfg}")
    run = GARun(cfg)
    run.set_launch(form=FORM_RESIDENT)
    run.set_tiles(12, 8)
    run.step(20)
    snap = run.read()
    run.step(33)
    run.write(snap["f"], snap["T"], snap["D"], snap["outbox"], 5)
    run.step(30)
    ref = oracle.OracleRun(cfg)
    ref.set_population(snap["f"], snap["T"], snap["D"])
    ob = snap["outbox"]
    ref.set_outbox(ob["valid"], ob["dir"], ob["f"], ob["T"], ob["D"])
    ref.set_generation(5)
    ref.step(30)
    assert_same_state(run.read(), ref, "set back")
    run.close()
    assert np.isfinite(snap["f"]).all()


@pytest.mark.parametrize("edge", [
    dict(width=8, height=8, pop=32, k=2, seed=51),          # 2,048 agents: one tile
    dict(width=13, height=5, pop=32, k=2, seed=52),         # the first size past it
    dict(width=41, height=50, pop=1, k=1, seed=53),
    dict(width=1000, height=3, pop=16, sites=64, k=4, model=2, policy=2, seed=54),
    dict(width=67, height=61, pop=16, k=2, seed=55),        # just under one tile per CU
    dict(width=211, height=97, pop=2, k=2, seed=56),
], ids=lambda e: "-".join(f"{k}{v}" for k, v in e.items()))
def test_default_tilings_match_oracle(edge):
    import torch
    cfg = run_config(**edge)
    run = GARun(cfg)
    tw, th, n = run.tiles()
    say(f"default tiling {tw} x {th}, {n} tiles, of {cfg}")
    agents = edge["width"] * edge["height"] * edge["pop"]
    assert (n == 1) == (agents <= 2048)
    assert n <= torch.cuda.get_device_properties(0).multi_processor_count
    for steps in (1, 8, 31):
        run.step(steps)
    assert_same_state(run.read(), oracle_after(cfg, 40), f"tiling {edge}")
    run.close()
