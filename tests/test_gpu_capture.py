"""Runs created while a stream is being captured: on the capturing stream (the
founders and the steps are then part of the graph, so every replay starts over) and
on another thread and stream, whose allocations must not end the capture. And
destroyed while another stream is busy, which they must not wait for."""
import ctypes
import threading

import pytest
import torch

from gpu_helpers import assert_same_state, oracle_after, say
from paper_2405_03605_amd import FORM_RESIDENT, FORM_STREAMING, GARun, load
from paper_2405_03605_amd.run import make_config
from paper_2405_03605_amd.workloads import run_config

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    load()
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("form", [FORM_STREAMING, FORM_RESIDENT])
def test_run_created_and_stepped_under_capture(form):
    cfg = run_config(width=40, height=24, pop=32, sites=32, k=2, seed=71)
    say(f"init and 14 generations captured, form {form}")
    # (the form's kernel is loaded before the capture)
    warm = GARun(cfg)
    warm.set_launch(form=form)
    warm.step(14)
    warm.read()
    warm.close()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run = GARun(cfg)
        run.set_launch(form=form)
        run.set_graph_block(0)
        run.step(14)
    ref = oracle_after(cfg, 14)
    for replay in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert_same_state(run.read(), ref, f"replay {replay}")
        other = GARun(cfg)
        other.step(5)
        other.close()
    run.close()


def test_run_created_while_another_thread_captures():
    cfg = run_config(width=40, height=24, pop=32, sites=32, k=2, seed=72)
    say("init on a second thread during a capture")
    lib = load()
    c = make_config(dict(cfg, law=0, p_ben32=0))
    n = int(lib.ga_state_bytes(ctypes.byref(c)))
    mem = torch.empty(n, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.Stream()
    x = torch.zeros(64, device="cuda")
    torch.cuda.synchronize()
    h, codes = ctypes.c_void_p(), []

    def other():
        torch.cuda.set_device(0)
        codes.append(lib.ga_init(ctypes.byref(c), ctypes.c_void_p(mem.data_ptr()), n,
                                 ctypes.c_void_p(stream.cuda_stream), ctypes.byref(h)))

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x += 1
        thread = threading.Thread(target=other)
        thread.start()
        thread.join()
        x += 1
    for _ in range(2):
        graph.replay()
    torch.cuda.synchronize()
    assert codes == [0] and float(x[0]) == 4.0
    assert lib.ga_step(h, 8) == 0
    lib.ga_destroy(h)


def test_destroying_a_run_does_not_wait_for_other_streams():
    say("destroy beside another stream's work")
    cfg = run_config(width=40, height=24, pop=32, sites=32, k=2, seed=73)
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    busy, done = torch.cuda.Stream(), torch.cuda.Event()
    runs = [GARun(cfg) for _ in range(3)]
    for r in runs:
        r.step(6)
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        for _ in range(200):
            b = a @ a
        done.record(busy)
    for r in runs:
        r.close()
    again = GARun(cfg)     # takes what they left
    again.step(21)
    got = again.read()
    assert not done.query(), "the other stream's work was waited for"
    assert_same_state(got, oracle_after(cfg, 21), "run in memory taken over")
    again.close()
    assert torch.isfinite(b[0, 0])
