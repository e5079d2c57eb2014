"""orloj_set_score_chunk: every setting is accepted and has no effect on the results, in
launches that turned_kernel takes and in launches that score_kernel takes."""
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


def same_bits(a, b):
    for k in a:
        assert np.array_equal(np.asarray(a[k]).view(np.uint8), np.asarray(b[k]).view(np.uint8)), k


CASES = [
    dict(seed=0),
    dict(seed=1, n_models=3, queue_lens=[0, 7, 13], batch_sizes=(1, 4, 16)),
    dict(seed=2, n_bins=2500, n_classes=4, queue_lens=[64, 40], batch_sizes=(1, 8, 33, 64),
         tau_range=(-20.0, 3000.0)),
    dict(seed=3, n_bins=4096, n_classes=6, queue_lens=[70, 64], batch_sizes=(16, 64),
         tau_range=(-5.0, 6000.0)),
    dict(seed=4, n_bins=300, sparsity=0.9, total=3, queue_lens=[50, 20]),
    dict(seed=5, n_bins=64, tau_range=(-50.0, -1.0), queue_lens=[30, 30]),     # all dead
    dict(seed=6, n_bins=64, tau_range=(500.0, 900.0), queue_lens=[30, 30]),    # beyond the grid
    dict(seed=7, n_models=1, n_bins=100, queue_lens=[200], batch_sizes=(128, 200)),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"seed{c['seed']}")
@pytest.mark.parametrize("law", ["tabulated", "affine"])
def test_every_setting_on_both_kernels(ctx, case, law):
    print("chunk settings", law, case, flush=True)
    wl = W.random_case(**case) if law == "tabulated" else W.random_affine(**case)
    ora = (oracle.score_workload(wl) if law == "tabulated"
           else oracle.score_workload_affine(wl, wl.c0_ms, wl.c1))
    ref = O.Scorer(wl, ctx).run()
    parity.compare(wl, ref, ora)
    large = parity.on_score_kernel(wl, ctx, ora)
    try:
        ctx.set_score_chunk(8)
        same_bits(O.Scorer(wl, ctx).run(), ref)
        same_bits(parity.on_score_kernel(wl, ctx, ora), large)
    finally:
        ctx.set_score_chunk(-1)


@pytest.mark.parametrize("seed", [20, 21])
def test_rect_mode_on_both_kernels(ctx, seed):
    wl = W.random_case(seed, n_models=2, queue_lens=[90, 33], batch_sizes=(1, 8, 40),
                       n_bins=1500, tau_range=(-10.0, 1800.0))
    ora = oracle.score_workload(wl, prefix_mode=1)
    parity.compare(wl, O.Scorer(wl, ctx, prefix_mode=1).run(), ora, mode=1)
    parity.on_score_kernel(wl, ctx, ora, mode=1)


def test_trimming_off(ctx):
    wl = W.random_case(30, n_models=2, queue_lens=[64, 50], batch_sizes=(2, 32, 64),
                       n_bins=3000, tau_range=(-10.0, 4000.0))
    ora = oracle.score_workload(wl)
    got = O.Scorer(wl, ctx).run()
    parity.compare(wl, got, ora)
    same_bits(O.Scorer(wl, ctx, trim=False).run(), got)
    parity.on_score_kernel(wl, ctx, ora)


def test_config2(ctx):
    wl = W.make(2, slo_scale=3.0)
    err = parity.compare(wl, O.Scorer(wl, ctx).run(), oracle.score_workload(wl))
    print("  cfg2 x3: max errors", err)


def test_config5_models(ctx):
    # eight models of the saturated state (four 1024-bin panels, 64 batch sizes)
    wl = W.make(5, models=[0, 17, 33, 50, 71, 90, 111, 127], workers=8)
    parity.compare(wl, O.Scorer(wl, ctx).run(), oracle.score_workload(wl))
    aw = W.affine(wl)
    parity.compare(aw, O.Scorer(aw, ctx).run(), oracle.score_workload_affine(aw, aw.c0_ms, aw.c1))


def test_small_config5_launch_against_the_oracle(ctx):
    # the scheduling loop's shape: a few idle models, every batch size
    wl = W.make(5, models=[5, 64], workers=8, slo_scale=2.0)
    err = parity.compare(wl, O.Scorer(wl, ctx).run(), oracle.score_workload(wl))
    print("  cfg5, 2 models: max errors", err)


def test_bad_chunk_is_rejected(ctx):
    with pytest.raises(O.OrlojError) as ei:
        ctx.set_score_chunk(-2)
    assert ei.value.code == O.ORLOJ_E_INVALID
