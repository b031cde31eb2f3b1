"""Training steps whose fine grid scatter runs on a side stream of the library (8,192 positions or more, atomic
mode): bfloat16 and FP32 one-trunk steps and the two-network step, whose colour network has 16 positions a block.
Captured in a HIP graph, on callers' own streams, from two host threads, and eagerly while another stream
is being captured.  Against steps run alone on the default stream: the atomics' order is the only difference (the
bounds of test_train_step_graph_replay)."""
import dataclasses
import threading

import numpy as np
import pytest
import torch

from cases import TrainProblem
from test_gpu_faithful_train import Problem
from util import ensure_built
from paper_2407_09543_amd import ntbc, synth

pytestmark = pytest.mark.gpu

N = 16384


@pytest.fixture(scope="module")
def problems():
    ensure_built()
    cfg = dataclasses.replace(synth.config_mid(256), grid_u8=False)
    return TrainProblem(cfg, synth.material_five(256, 12), 12), Problem("all", 13)


def make(problems, kind):
    """(trainer, ids, gradients and parameters) of a problem of which a step forks."""
    one, two = problems
    rng = np.random.default_rng(14)
    if kind == "paper":
        tr = two.trainer(N // 16, 100)
        ids = rng.integers(0, two.bw * two.bh, N // 16)
        state = tr.grads, tr.params
    else:
        tr = ntbc.Trainer(one.desc, one.grid_d, one.flat_d, one.tg_gpu, N, 100, precision=ntbc.PRECISIONS[kind])
        ids = rng.integers(0, one.cfg.n_positions, N)
        state = [tr.d_grid, tr.d_w], [tr.grid, tr.weights]
    return tr, torch.from_numpy(ids.astype(np.int32)).cuda(), state


def agree(a, b, what):
    for bound, x, y in ((1e-5, a[0], b[0]), (1e-4, a[1], b[1])):
        for p, q in zip(x, y):
            rel = (torch.linalg.vector_norm(p - q) / torch.linalg.vector_norm(p)).item()
            assert rel < bound, (what, rel)


KINDS = ["bf16", "fp32", "paper"]


@pytest.mark.parametrize("kind", KINDS)
def test_captured_step(problems, kind):
    eager, ids, want = make(problems, kind)
    graphed, _, got = make(problems, kind)
    stream = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    warm, _, _ = make(problems, kind)
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        warm.step(ids, 5)  # the streams and the kernel attributes exist before the capture
        stream.synchronize()
        with torch.cuda.graph(g, stream=stream):
            graphed.step(ids, 5)
    torch.cuda.synchronize()
    for rep in range(3):
        eager.step(ids, 5)
        g.replay()
        torch.cuda.synchronize()
        agree(want, got, f"replay {rep}")
        _ = torch.ones(1000, device="cuda").sum().item()  # eager work between the replays


@pytest.mark.parametrize("kind", KINDS)
def test_eager_step_during_a_capture(problems, kind):
    # the side stream that the captured step drew into its graph is not touched by the eager step of another stream
    # (whose work would become part of the graph), and the graph holds its own step alone
    alone, ids, want = make(problems, kind)
    eager, _, seen = make(problems, kind)
    graphed, _, got = make(problems, kind)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    for s in (a, b):
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            make(problems, kind)[0].step(ids, 5)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=a, capture_error_mode="thread_local"):
        graphed.step(ids, 5)
        with torch.cuda.stream(b):
            eager.step(ids, 5)
            eager.step(ids, 6)
        graphed.step(ids, 6)
    torch.cuda.synchronize()
    for k in (5, 6):
        alone.step(ids, k)
    torch.cuda.synchronize()
    agree(want, seen, "eager")
    after = [t.clone() for t in seen[0] + seen[1]]
    for rep in range(2):
        if rep:
            for k in (5, 6):
                alone.step(ids, k)
        g.replay()
        torch.cuda.synchronize()
        agree(want, got, f"replay {rep}")
        assert all(torch.equal(x, y) for x, y in zip(after, seen[0] + seen[1]))


@pytest.mark.parametrize("threads", [False, True], ids=["streams", "threads"])
def test_trainers_on_their_own_streams(problems, threads):
    alone = [make(problems, k) for k in KINDS]
    for tr, ids, _ in alone:
        for k in range(4):
            tr.step(ids, k)
    torch.cuda.synchronize()
    runs = [make(problems, k) + (torch.cuda.Stream(),) for k in KINDS]
    torch.cuda.synchronize()

    def step(run, k):
        with torch.cuda.stream(run[3]):
            run[0].step(run[1], k)
    if threads:
        failed = []

        def all_steps(run):
            try:
                for k in range(4):
                    step(run, k)
            except Exception as e:  # reported below: a thread's exception would be lost
                failed.append(e)
        ts = [threading.Thread(target=all_steps, args=(r,)) for r in runs]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert not failed
    else:
        for k in range(4):
            for r in runs:
                step(r, k)
    torch.cuda.synchronize()
    for (_, _, want), run, kind in zip(alone, runs, KINDS):
        # four steps of Adam from zero moments: a gradient within rounding of zero may take another sign there, so
        # the parameters are compared by the losses they give
        losses = [x[0].losses[:4].cpu().numpy() for x in (alone[KINDS.index(kind)], run)]
        assert np.allclose(losses[0], losses[1], rtol=1e-3), (kind, losses)
        assert run[0].losses[4] == 0
