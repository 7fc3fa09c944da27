"""Closed islands (no migration) in several LDS-resident tiles with emissions
pending from a written state, bit for bit against the oracle: every pending genome
is absorbed in the first generation, across tile edges too, for step counts that
end on either outbox plane."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_same_state, say
from paper_2405_03605_amd import FORM_RESIDENT, GARun
from paper_2405_03605_amd.workloads import run_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [(1,), (2,), (4, 2), (7, 100)])
@pytest.mark.parametrize("edge,tiles", [
    (dict(width=64, height=64, pop=32, sites=32), (4, 4)),
    (dict(width=37, height=11, pop=4, sites=64, k=5), (5, 3)),
], ids=lambda e: "-".join(map(str, e)) if isinstance(e, tuple) else f"N{e['pop']}")
def test_pending_emissions_reach_closed_islands(edge, tiles, steps):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = run_config(migration=0, seed=61, **edge)
    say(f"closed islands, tiles {tiles}, steps {steps}, {cfg}")
    rng = np.random.default_rng(62)
    islands, words = cfg["width"] * cfg["height"], cfg["sites"] // 32
    ob = {"valid": rng.integers(0, 4, islands).clip(0, 1).astype(np.uint8),
          "dir": rng.integers(0, 4, islands).astype(np.uint8),
          "f": np.full(islands, 100.0, np.float32),
          "T": rng.integers(0, 1000, islands).astype(np.uint32),
          "D": rng.integers(0, 1 << 32, (islands, words), dtype=np.uint64).astype(np.uint32)}
    agents = islands * cfg["pop"]
    pop = (np.zeros(agents, np.float32), np.zeros(agents, np.uint32),
           np.zeros((agents, words), np.uint32))
    run = GARun(cfg)
    run.set_launch(form=FORM_RESIDENT)
    run.set_tiles(*tiles)
    assert run.tiles()[2] > 1
    run.write(*pop, ob, 8)
    ref = oracle.OracleRun(cfg)
    ref.set_population(*pop)
    ref.set_outbox(ob["valid"], ob["dir"], ob["f"], ob["T"], ob["D"])
    ref.set_generation(8)
    for n in steps:
        run.step(n)
        ref.step(n)
        got = run.read()
        assert_same_state(got, ref, f"closed islands after {n}")
    assert (got["f"] >= 90).any()  # the pending genomes are fit enough to stay
    run.close()
