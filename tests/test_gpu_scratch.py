"""The context's scratch blocks under HIP graph capture: a captured call does not
lose its scratch to later calls of other kinds, and finds it whichever queues were
filled in the calls before."""
import threading

import numpy as np
import pytest
import torch

import oracle
import parity
from paper_2209_00159_amd import orloj as O
from paper_2209_00159_amd import workloads as W

pytestmark = pytest.mark.gpu


def captured(stream, call):
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        call()
    return g


def replay_and_compare(g, sc, wl, stream, ora):
    for buf in (sc.finish_prob, sc.expected_finish, sc.expected_latency, sc.score_out):
        buf.fill_(-7.0)
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        sc.select()
        sc.ctx.sync()
    parity.compare(wl, sc.fetch(), ora)


def few_queues(n_models, seed):
    """The first model's queue holds 40 requests, the others none."""
    return W.random_affine(seed, n_models=n_models, n_classes=8, n_bins=600,
                           batch_sizes=(5, 17, 40), queue_lens=[40] + [0] * (n_models - 1))


@pytest.mark.parametrize("warm", ["same call", "larger launch"])
def test_captured_affine_call(warm):
    print("scratch", warm, flush=True)
    stream = torch.cuda.Stream()
    ctx = O.Context(stream=stream)
    n = 200
    wl = few_queues(n, 7)
    many = W.random_affine(8, n_models=n, n_classes=8, n_bins=600, batch_sizes=(5, 17, 40),
                           queue_lens=[40] * n)
    sc, big = O.Scorer(wl, ctx), O.Scorer(many, ctx)
    torch.cuda.synchronize()
    sc.build()
    # the affine sums' block is as large for few filled queues as for many
    (sc if warm == "same call" else big).run()
    g = captured(stream, sc.score)
    ora = oracle.score_workload_affine(wl, wl.c0_ms, wl.c1)
    replay_and_compare(g, sc, wl, stream, ora)
    # eager work of other kinds, each with more scratch than the one before
    laws = W.random_case(9, n_models=1, n_classes=16, n_bins=8192, queue_lens=[0],
                         batch_sizes=tuple(range(1, 65)))
    it = O.Iterator(laws, ctx)
    torch.cuda.synchronize()
    it.build()
    if warm == "same call":
        big.run()
    ctx.sync()
    junk = torch.full((1 << 22,), 3.0, device="cuda")  # takes freed memory, if any
    for _ in range(3):
        replay_and_compare(g, sc, wl, stream, ora)
    assert float(junk.min()) == 3.0 and float(junk.max()) == 3.0


@pytest.mark.parametrize("warm", ["one queue filled", "every queue filled"])
def test_affine_bits_do_not_depend_on_the_scratch(warm):
    """A call warmed by another number of filled queues of the same grid can be
    captured, and has the bits of the eager and of the allocation-free call."""
    print("affine bits", warm, flush=True)
    n = 200
    few = few_queues(n, 7)
    many = W.random_affine(8, n_models=n, n_classes=8, n_bins=600, batch_sizes=(5, 17, 40),
                           queue_lens=[40] * n)
    first, wl = (few, many) if warm == "one queue filled" else (many, few)
    stream = torch.cuda.Stream()
    ctx = O.Context(stream=stream)
    a, b = O.Scorer(first, ctx), O.Scorer(wl, ctx)
    torch.cuda.synchronize()
    a.run()
    b.build()
    g = captured(stream, b.score)

    def outputs(call):
        for buf in (b.finish_prob, b.expected_finish, b.expected_latency, b.score_out):
            buf.fill_(-7.0)
        torch.cuda.synchronize()
        call()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            b.select()
            ctx.sync()
        return b.fetch()

    got = outputs(g.replay)
    parity.compare(wl, got, oracle.score_workload_affine(wl, wl.c0_ms, wl.c1))
    for call in (b.score, lambda: b.score(noalloc=True), g.replay):
        for k, v in outputs(call).items():
            assert np.array_equal(v.view(np.uint8), got[k].view(np.uint8)), k


def test_first_model_laws_while_another_thread_captures():
    """The scratch of few pairs' laws is allocated by the first call that needs it, which
    must not end the capture of another thread's stream nor fail because of it."""
    ctx, ref = O.Context(stream=torch.cuda.Stream()), O.Context()
    wl = W.random_case(13, n_models=1, n_classes=8, n_bins=8192, queue_lens=[0],
                       batch_sizes=tuple(range(1, 17)))
    it, want = O.Iterator(wl, ctx), O.Iterator(wl, ref)
    x = torch.zeros(64, device="cuda")
    want.build()
    ref.sync()
    failed = []

    def laws():
        try:
            it.build()
        except Exception as e:                 # (a thread's exception would be lost)
            failed.append(e)

    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream(), capture_error_mode="global"):
        x += 1.0
        t = threading.Thread(target=laws)
        t.start()
        t.join()
        x += 1.0
    assert not failed, failed
    ctx.sync()
    for a, b in ((it.law, want.law), (it.disc, want.disc), (it.model_el, want.model_el)):
        assert torch.equal(a, b)
    for n in (1, 2):
        g.replay()
        torch.cuda.synchronize()
        assert float(x.min()) == float(x.max()) == 2.0 * n


def test_captured_model_laws_use_no_scratch():
    stream = torch.cuda.Stream()
    ctx = O.Context(stream=stream)
    wl = W.random_case(11, n_models=1, n_classes=9, n_bins=700, queue_lens=[0], batch_sizes=(1, 4))
    it = O.Iterator(wl, ctx)
    torch.cuda.synchronize()
    it.build()
    ctx.sync()
    want = [t.cpu().numpy() for t in (it.law, it.disc, it.model_el)]
    g = captured(stream, it.build)
    larger = W.random_case(12, n_models=2, n_classes=9, n_bins=4096, queue_lens=[0, 0],
                           batch_sizes=tuple(range(1, 33)))
    other = O.Iterator(larger, ctx)
    torch.cuda.synchronize()
    other.build()
    ctx.sync()
    for _ in range(3):
        for t in (it.law, it.disc, it.model_el):
            t.fill_(-7.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = [t.cpu().numpy() for t in (it.law, it.disc, it.model_el)]
        for a, b in zip(got, want):
            assert np.array_equal(a.view(np.uint8), b.view(np.uint8))


@pytest.mark.parametrize("kept", ["affine sums", "drop phase"])
def test_scoring_and_iteration_grow_blocks_of_their_own(kept):
    """A captured affine call whose sums lie in emax_kernel's block replays after an
    iteration of long queues has grown its scratch past them, and a captured
    iteration after a larger affine call."""
    print("scratch of scoring and iteration", kept, flush=True)
    stream = torch.cuda.Stream()
    ctx = O.Context(stream=stream)

    def scorer(n):                             # 3 n pairs: score_kernel and emax_kernel
        wl = W.random_affine(21, n_models=n, n_classes=4, n_bins=300, batch_sizes=(5, 17, 40),
                             queue_lens=[40] * n)
        return wl, O.Scorer(wl, ctx)

    def iterator(n, queue, sizes):
        return O.Iterator(W.random_case(22, n_models=n, n_classes=4, n_bins=64, batch_sizes=sizes,
                                        queue_lens=[queue] * n, tau_range=(0.0, 90.0)), ctx)

    if kept == "affine sums":                  # 200 x 2 x 40 sums against 8 x 16 x 140 x 8 bytes
        (wl, sc), other = scorer(200), iterator(8, 4096, tuple(range(1, 141)))
        torch.cuda.synchronize()
        sc.run()
        g = captured(stream, sc.score)
        ora = oracle.score_workload_affine(wl, wl.c0_ms, wl.c1)

        def replay():
            replay_and_compare(g, sc, wl, stream, ora)
    else:
        it, other = iterator(1, 1100, (1, 8)), scorer(600)[1]
        torch.cuda.synchronize()
        want = it.run()
        g = captured(stream, it.iterate)

        def replay():
            for t in (it.timed_out, it.score, it.cand_bs, it.batch):
                t.fill_(-7)
            torch.cuda.synchronize()
            g.replay()
            for k, v in it.fetch().items():
                assert np.array_equal(v.view(np.uint8), want[k].view(np.uint8)), k

    replay()
    other.run()
    junk = torch.full((1 << 22,), 3.0, device="cuda")  # takes freed memory, if any
    for _ in range(3):
        replay()
    assert float(junk.min()) == 3.0 and float(junk.max()) == 3.0
