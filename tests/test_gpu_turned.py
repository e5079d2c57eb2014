"""turned_kernel (launches of few (model, batch size) pairs, with eight waves a
workgroup and with four) and score_kernel (larger ones) on the same models, against
the oracle and against each other.

The sizes lie at turned_kernel's edges: prefixes of 16, 32 and 64 members (parts
of a block), one, two and four blocks of 64 prefix lengths, blocks of 16, 32 and
64 bins, tiles of 128 and 512 bins, rows shorter than a block, deadlines beyond the grid
where the grid's end lies inside a block and on its edge, a single member.
"""
import dataclasses
import sys

import numpy as np
import pytest

import oracle
import parity
from paper_2209_00159_amd import orloj as O
from paper_2209_00159_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return O.Context()


CASES = [
    dict(seed=100, queue_lens=[1, 1], batch_sizes=(1,), n_bins=1),
    dict(seed=101, queue_lens=[15, 16], batch_sizes=(1, 15, 16), n_bins=63),
    dict(seed=102, queue_lens=[17, 16], batch_sizes=(16, 17), n_bins=64),
    dict(seed=103, queue_lens=[32, 31], batch_sizes=(31, 32), n_bins=65, tau_range=(-5.0, 200.0)),
    dict(seed=104, queue_lens=[33, 34], batch_sizes=(32, 33, 34), n_bins=128, tau_range=(-5.0, 400.0)),
    dict(seed=105, queue_lens=[64, 63], batch_sizes=(48, 63, 64), n_bins=129, tau_range=(0.0, 300.0)),
    dict(seed=106, queue_lens=[65, 64], batch_sizes=(64, 65), n_bins=127, tau_range=(0.0, 300.0)),
    dict(seed=107, queue_lens=[128, 80], batch_sizes=(1, 80, 127, 128), n_bins=255, tau_range=(0.0, 300.0)),
    dict(seed=108, queue_lens=[129, 130], batch_sizes=(129, 130), n_bins=256, tau_range=(0.0, 500.0)),
    dict(seed=109, queue_lens=[256, 193], batch_sizes=(192, 193, 256), n_bins=257, n_classes=9,
         tau_range=(0.0, 400.0)),
    dict(seed=110, queue_lens=[40, 3], batch_sizes=(1, 2, 40), n_bins=1, tau_range=(-1.0, 3.0)),
    dict(seed=111, queue_lens=[64, 20], batch_sizes=(20, 64), n_bins=1025, tau_range=(-10.0, 1400.0), sparsity=0.95),
    dict(seed=112, queue_lens=[100, 0, 7], n_models=3, batch_sizes=(5, 90), n_bins=600, b_expo=0.2,
         tau_range=(-10.0, 900.0)),
    dict(seed=113, queue_lens=[30, 60], batch_sizes=(30, 60), n_bins=8192, n_classes=2, tau_range=(0.0, 12000.0)),
    # every deadline in the first bin: 1024 bins past the members (narrow tiles), one more
    # (wide tiles), a wide tile of one bin, of all its bins, members in two and four blocks
    dict(seed=114, queue_lens=[16, 9], batch_sizes=(9, 16), n_bins=64 + 1024, tau_range=(-0.1, 0.4)),
    dict(seed=115, queue_lens=[16, 9], batch_sizes=(9, 16), n_bins=64 + 1025, tau_range=(-0.1, 0.4)),
    dict(seed=116, queue_lens=[40, 33], batch_sizes=(33, 40), n_bins=16 + 1536, tau_range=(-0.1, 0.4),
         sparsity=0.95),
    dict(seed=117, queue_lens=[70, 66], batch_sizes=(64, 70), n_bins=64 + 1537, tau_range=(-0.1, 0.4)),
    dict(seed=118, n_models=1, queue_lens=[200], batch_sizes=(130, 200), n_bins=2600, n_classes=5,
         tau_range=(-0.1, 0.4)),
]


def run(wl, ctx, mode, trim):
    return O.Scorer(wl, ctx, prefix_mode=mode, trim=trim).run(build=True)


def cost_of(wl, seed):
    r = np.random.default_rng(seed)
    return dataclasses.replace(wl, cost=r.uniform(0.0, 3.0, size=wl.cls.size))


@pytest.mark.parametrize("law", ["tabulated", "affine"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"seed{c['seed']}")
def test_both_kernels_against_the_oracle(ctx, case, law):
    print("turned", law, case, flush=True)
    mode = case["seed"] % 2
    one = W.random_affine(**case) if law == "affine" else W.random_case(**case)
    if case["seed"] % 3 == 0:
        one = cost_of(one, case["seed"])
    small = run(one, ctx, mode, True)
    for k, v in run(one, ctx, mode, False).items():        # trimming changes no bits
        assert np.array_equal(v.view(np.uint8), small[k].view(np.uint8)), k
    ora = (oracle.score_workload_affine(one, one.c0_ms, one.c1, prefix_mode=mode) if law == "affine"
           else oracle.score_workload(one, prefix_mode=mode))
    parity.compare(one, small, ora, mode=mode)
    # the same models over and over: in one launch of more workgroups than compute units
    # (four waves each), and in one of more than turned_kernel takes
    groups, longest = parity.turned_groups(one, mode)
    for most in (parity.N_CU, parity.past_turned(law == "affine", one.n_bins, longest)):
        check_large(ctx, one, mode, most // groups + 1, small, ora)


def check_large(ctx, one, mode, reps, small, ora):
    M = one.n_models
    large = run(one.subset(list(range(M)) * reps), ctx, mode, True)
    n, npr = small["score"].size, small["finish_prob"].size
    for r in (0, reps - 1):
        part = {k: v[r * (npr if k == "finish_prob" else M if k.startswith("sel") else n):][:v.size // reps]
                for k, v in large.items()}
        parity.compare(one, part, ora, mode=mode)
        # between the kernels, or two splits of the bins: G's products agree to 256 x 2^-53, so P to one
        # fp32 rounding (2^-24 at most) and E to the sum of the members' 2^-45
        assert np.abs(part["finish_prob"] - small["finish_prob"]).max(initial=0.0) <= 2.0**-24
        assert np.allclose(part["expected_finish"], small["expected_finish"], rtol=1e-12, atol=1e-12)
        # E[L_B]: score_kernel adds fp32 sums, each rounded once per panel
        # (2^-25 of it) after a six-level fp32 tree (6 x 2^-24)
        assert np.allclose(part["expected_latency_ms"], small["expected_latency_ms"], rtol=8 * 2.0**-24, atol=0)


@pytest.mark.parametrize("law", ["tabulated", "affine"])
@pytest.mark.parametrize("every", [4, 10])
def test_mostly_empty_launches(ctx, law, every):
    """300 models with a queue, too many to list, among 1200 (turned_kernel, with workgroups
    that find nothing to do) and among 3000 (score_kernel: most would)."""
    print("mostly empty", law, every, flush=True)
    n = 300 * every
    case = dict(seed=130 + every, n_models=n, n_classes=2, n_bins=40, batch_sizes=(14,),
                queue_lens=[14 if q % every == every - 1 else 0 for q in range(n)])
    wl = W.random_affine(**case) if law == "affine" else W.random_case(**case)
    ora = (oracle.score_workload_affine(wl, wl.c0_ms, wl.c1) if law == "affine"
           else oracle.score_workload(wl))
    parity.compare(wl, run(wl, ctx, 0, True), ora)
