"""The LDS-resident form at the edges of what it accepts, bit for bit against the
oracle: tiles within 400 bytes of a CU's LDS, with islands of one, two and four
agents, and tiles of a few such islands, whose read-ahead ends past their outbox;
as many tiles as are resident at once, and the refusal of more."""
import pytest

from gpu_helpers import assert_same_state, oracle_after, say
from paper_2405_03605_amd import FORM_RESIDENT, GAError, GARun
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


def check(edge, tiles, steps=(1, 6)):
    cfg = run_config(**edge)
    say(f"tiles {tiles} on {cfg}")
    run = GARun(cfg)
    run.set_launch(form=FORM_RESIDENT)
    run.set_tiles(*tiles)
    assert run.tiles()[:2] == tiles
    for n in steps:
        run.step(n)
    assert_same_state(run.read(), oracle_after(cfg, sum(steps)), f"tiles {tiles} {edge}")
    run.close()


@pytest.mark.parametrize("edge,tiles", [
    (dict(width=2, height=1022, pop=1, sites=64, k=1), (1, 1022)),
    (dict(width=4, height=612, pop=1, sites=64, k=1, model=1), (2, 612)),
    (dict(width=4, height=581, pop=2, sites=64, k=2), (2, 581)),
    (dict(width=7, height=375, pop=2, sites=64, k=3, model=2), (3, 375)),
    (dict(width=10, height=217, pop=4, sites=64, k=2), (5, 217)),
], ids=lambda e: f"N{e['pop']}m{e.get('model', 0)}" if isinstance(e, dict) else f"t{e[0]}x{e[1]}")
def test_tiles_that_fill_the_lds(edge, tiles):
    check(edge, tiles)


@pytest.mark.parametrize("pop", [1, 2, 4])
@pytest.mark.parametrize("sites,model", [(32, 0), (64, 0), (64, 1)])
def test_tiles_of_a_few_islands(pop, sites, model):
    check(dict(width=3, height=4, pop=pop, sites=sites, model=model, k=1, seed=81), (1, 1))
    check(dict(width=7, height=5, pop=pop, sites=sites, model=model, k=1, seed=82), (3, 2))


def test_many_waiting_wavefronts_a_cu():
    # 24 one-wavefront tiles on every CU: most wait for a neighbour at any time,
    # and the ones waited for must still get their turn
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    check(dict(width=8 * 24 * cus // 64, height=8 * 64, pop=1, sites=32, k=1, seed=84), (8, 8),
          (60, 40))
    # and of two wavefronts each, 32-agent islands
    check(dict(width=2 * 10 * cus // 64, height=2 * 64, pop=32, sites=32, k=2, seed=85), (2, 2),
          (60, 40))


@pytest.mark.parametrize("policy", [0, 1])
def test_one_agent_islands_at_28_wavefronts_a_cu(policy):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    # one-wavefront tiles, 28 on every CU
    check(dict(width=8 * 28, height=8 * cus, pop=1, sites=32, k=1, policy=policy, seed=83), (8, 8),
          (1, 40))


@pytest.mark.parametrize("edge,tile,most", [
    (dict(pop=1, sites=64, k=1), (8, 8), 21),
    (dict(pop=1, sites=64, k=1), (16, 8), 11),
    (dict(pop=1, sites=64, k=1, model=2, policy=1), (16, 16), 5),
    (dict(pop=1, sites=32, k=1), (8, 8), 28),
    (dict(pop=32, sites=32, k=2, model=1), (2, 1), 24),
    (dict(pop=32, sites=32, k=2, model=1), (2, 2), 12),
    (dict(pop=64, sites=32, k=2, model=2), (1, 1), 24)],
    ids=lambda e: f"N{e['pop']}S{e['sites']}m{e.get('model', 0)}" if isinstance(e, dict) else None)
def test_most_tiles_a_cu(edge, tile, most):
    # by the LDS each takes (in pieces of 1,280 bytes), or by its wavefronts
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    size = dict(height=tile[1] * cus // 4)
    check(dict(edge, width=tile[0] * 4 * most, seed=88, **size), tile, (1, 20))
    run = GARun(run_config(**edge, width=tile[0] * 4 * (most + 1), seed=89, **size))
    run.set_launch(form=FORM_RESIDENT)
    with pytest.raises(GAError):
        run.set_tiles(*tile)
        run.tiles()
    run.close()


@pytest.mark.parametrize("edge", [
    dict(width=40, height=40, pop=1, k=1, seed=86), dict(width=5, height=5, pop=1, sites=64, k=1),
    dict(width=29, height=17, pop=2, sites=64, model=1, k=2, seed=87)],
    ids=lambda e: f"{e['width']}x{e['height']}x{e['pop']}")
def test_default_tilings_of_small_islands(edge):
    cfg = run_config(**edge)
    run = GARun(cfg)
    tw, th, n = run.tiles()
    say(f"default tiling {tw} x {th}, {n} tiles, of {cfg}")
    assert n > 1 and tw * th <= 16
    for steps in (1, 8, 31):
        run.step(steps)
    assert_same_state(run.read(), oracle_after(cfg, 40), f"tiling {edge}")
    run.close()
