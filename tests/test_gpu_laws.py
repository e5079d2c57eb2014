"""Model laws of few (model, batch size) pairs (laws_mix_kernel and
laws_row_kernel) against the same rows in a launch of many (laws_kernel): the
same products, scans and sums in the same order, so the same bits.  Row lengths lie
at the edges of the threads' chunks and of the 16-byte loads."""

import numpy as np
import pytest

from paper_2209_00159_amd import orloj as O
from paper_2209_00159_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return O.Context()


def laws(wl, ctx, weights):
    it = O.Iterator(wl, ctx, class_weights=weights)
    it.build()
    ctx.sync()
    return it.law.cpu().numpy(), it.disc.cpu().numpy(), it.model_el.cpu().numpy()


@pytest.mark.parametrize("n_bins", [1, 3, 4, 255, 256, 257, 1000, 1023, 2048, 4097, 8192])
@pytest.mark.parametrize("n_classes", [8, 16, 33])   # (8: rows of 512 bins or more)
def test_few_pairs_give_the_bits_of_many(ctx, n_bins, n_classes):
    print("laws", n_bins, n_classes, flush=True)
    one = W.random_case(n_bins, n_models=1, n_classes=n_classes, n_bins=n_bins, queue_lens=[0],
                        batch_sizes=(1, 2, 7))
    wts = np.random.default_rng(n_bins).uniform(0.1, 2.0, size=(1, n_classes))
    reps = 90                                  # 270 pairs: more than the compute units
    few, many = laws(one, ctx, wts), laws(one.subset([0] * reps), ctx, np.repeat(wts, reps, axis=0))
    for q in (0, reps - 1):
        for a, b in zip(few, many):
            assert np.array_equal(a[0].view(np.uint8), b[q].view(np.uint8))
