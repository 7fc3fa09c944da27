"""The launch-shape autotuner's choices on the CPU, with a stand-in batch whose
steps take a time that the test sets."""
import pytest

from paper_2405_03605_amd import autotune
from paper_2405_03605_amd.workloads import run_config

CFGS = [run_config(width=20, height=10, pop=8), run_config(width=12, height=12, pop=32, sites=32)]
CLASSES = [(3, 2), (5, 1)]


class FakeRun:
    def __init__(self, cfg):
        self.cfg = cfg

    def close(self):
        pass


class FakeBatch:
    """Chunks of the rule, or a setting cut to what a launch of two takes."""
    rule = {(3, 2): 8, (5, 1): 2}
    most = {(3, 2): 16, (5, 1): 16}
    steps = []                       # the settings of each timed step

    def __init__(self):
        self.settings, self.launch = {}, None

    def add(self, run, budget):
        pass

    def close(self):
        pass

    def set_launch(self, ipw, wpg):
        self.launch = (ipw, wpg)

    def set_class_launch(self, log2n, words, ipw=0):
        self.settings[(log2n, words)] = ipw

    def class_launch(self, log2n, words):
        k = (log2n, words)
        return (min(self.settings[k], self.most[k]) if self.settings.get(k) else self.rule[k]), 1


@pytest.fixture
def tuner(monkeypatch):
    def tune(seconds, cfgs=CFGS):
        FakeBatch.steps = []

        def time_batch(batch, gens, torch, reps=2):
            used = {k: batch.class_launch(*k)[0] for k in CLASSES}
            FakeBatch.steps.append((used, batch.launch[1]))
            return seconds(used, batch.launch[1])
        monkeypatch.setattr(autotune, "GARun", FakeRun)
        monkeypatch.setattr(autotune, "GABatch", FakeBatch)
        monkeypatch.setattr(autotune, "_time_batch", time_batch)
        batch = FakeBatch()
        return batch, autotune.autotune_batch(batch, cfgs, use_cache=False)
    return tune


def test_where_nothing_wins_the_rule_stays(tuner):
    batch, chosen = tuner(lambda used, wpg: 1.0 if used == FakeBatch.rule else 1.2)
    assert {k: batch.class_launch(*k)[0] for k in CLASSES} == FakeBatch.rule
    assert all(not batch.settings[k] for k in CLASSES)
    assert {k: chosen[k] for k in CLASSES} == FakeBatch.rule
    assert set(chosen["by_rule"]) == set(CLASSES)
    # the rule is what the first timing is of, and no chunk is timed twice
    assert FakeBatch.steps[0][0] == FakeBatch.rule
    assert len({tuple(sorted(u.items())) for u, _ in FakeBatch.steps}) == len(FakeBatch.steps)
    # pairs go in groups of one wavefront: there is nothing to choose
    assert {w for _, w in FakeBatch.steps} == {4}


def test_a_faster_chunk_is_kept_and_the_rest_stay_on_the_rule(tuner):
    batch, chosen = tuner(lambda used, wpg: 0.5 if used[(5, 1)] == 8 else 1.0)
    assert batch.settings[(5, 1)] == 8 and chosen[(5, 1)] == 8
    assert not batch.settings[(3, 2)] and chosen["by_rule"] == ((3, 2),)
    # the choice carries over to a pool as it is
    pool = FakeBatch()
    autotune.apply_shapes(pool, chosen)
    assert pool.settings == {(3, 2): 0, (5, 1): 8} and pool.launch == (0, 4)


def test_a_card_that_warms_up_makes_nothing_win(tuner):
    clock = [1.0]

    def seconds(used, wpg):
        clock[0] *= 0.97             # every timing 3% faster than the one before
        return clock[0] * (1.0 if used == FakeBatch.rule else 1.02)
    batch, chosen = tuner(seconds)
    assert set(chosen["by_rule"]) == set(CLASSES)
    assert {k: batch.class_launch(*k)[0] for k in CLASSES} == FakeBatch.rule


def test_group_size_is_searched_where_single_generations_run(tuner):
    cfgs = [run_config(width=9, height=9, pop=2)] + CFGS
    FakeBatch.rule[(1, 2)] = FakeBatch.most[(1, 2)] = 64
    batch, chosen = tuner(lambda used, wpg: 1.0 / wpg, cfgs)
    assert chosen["waves_per_group"] == max(autotune.WPG_CANDIDATES)


def test_tile_lds_estimate_is_the_kernels():
    import ctypes

    from paper_2405_03605_amd import _lib
    lds = ctypes.CDLL(_lib.LIB_PATH)._ZN2ga14tile_lds_bytesEjjjjjj   # ga::tile_lds_bytes
    lds.restype = ctypes.c_size_t
    for pop in (1, 2, 4, 8, 16, 32, 64):
        for sites, model in ((32, 0), (64, 0), (32, 1), (64, 2)):
            cfg = run_config(pop=pop, sites=sites, model=model)
            for tw, th in ((1, 1), (3, 2), (8, 8), (37, 5), (64, 24), (100, 13)):
                want = lds(tw, th, pop.bit_length() - 1, sites // 32, model,
                           4 if (sites, model) == (32, 0) else 8)
                assert autotune.tile_lds_estimate(tw, th, cfg) == want, (pop, sites, model, tw, th)


@pytest.mark.parametrize("kw,chunks", [
    (dict(pop=32, sites=32), [2, 4, 8, 16]), (dict(pop=32, sites=64), [2, 4, 8]),
    (dict(pop=64, sites=32), [1, 2, 4, 8]), (dict(pop=64, sites=32, model=1), [1, 2, 4]),
    (dict(pop=16, sites=64), [4, 8, 16]), (dict(pop=4, sites=32), [16])])
def test_single_run_candidates_are_the_chunks_that_differ(kw, chunks):
    from paper_2405_03605_amd import FORM_STREAMING
    cands = autotune.candidates(run_config(width=40, height=30, **kw))
    streaming = [c for c in cands if c[2] == FORM_STREAMING]
    assert streaming == [(i, 4, FORM_STREAMING) for i in chunks]
    assert len(set(cands)) == len(cands)


def test_single_generations_are_searched_in_both_directions():
    from paper_2405_03605_amd import FORM_STREAMING
    cands = autotune.candidates(run_config(width=40, height=30, pop=2))
    assert {c[:2] for c in cands if c[2] == FORM_STREAMING} == {
        (i, w) for i in (32, 64) for w in (1, 2, 4, 8)}
