"""GPU tests of the fp32 attention kernel at the sizes of its lists: chunks of 32 listed keys, 64 columns
a tile, 32 tiles a round.  Against the fp64 oracle within the fp32 bar (gpu_util.TOL: dot products of at
most 128 terms and hardware exponentials give a few 1e-7; the sums of these rows are longer but
positive)."""
import numpy as np
import pytest

from paper_2012_02030_amd import synth

from gpu_util import run_and_compare

pytestmark = pytest.mark.gpu


def inputs(seed, B, H, Lq, Lk, D):
    rng = np.random.default_rng([synth.SEED, 3232, seed])
    return tuple(rng.standard_normal((B, H, L, D), dtype=np.float32) for L in (Lq, Lk, Lk))


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("n_keys", [1, 31, 32, 33, 64, 65, 127, 129])
def test_number_of_listed_keys(n_keys, D):
    """Exactly n_keys keys are listed for the first 32 queries, none for the second 32, all for the last."""
    Q, K, V = inputs(n_keys, 1, 2, 70, 200, D)
    rng = np.random.default_rng(n_keys)
    mask = np.zeros((2, 70, 200), np.uint8)
    for h in range(2):
        for j in rng.permutation(200)[:n_keys]:
            mask[h, rng.integers(0, 32, size=3), j] = 1
        mask[h, 64:] = 1
    run_and_compare(Q, K, V, mask, "f32", False)


@pytest.mark.parametrize("Lk", [2048, 2049, 4096 + 70])
@pytest.mark.parametrize("density", [0.002, 0.3])
def test_rows_of_more_tiles_than_one_round(Lk, density):
    Q, K, V = inputs(Lk, 1, 1, 33, Lk, 64)
    run_and_compare(Q, K, V, synth.random_mask(1, 33, Lk, density, seed=Lk), "f32", False)
    run_and_compare(Q, K, V, synth.random_mask(1, 33, Lk, density, seed=Lk), "f32", True)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("Lq", [1, 32, 33, 95, 129])
def test_ragged_query_groups(Lq, D):
    Q, K, V = inputs(Lq, 2, 3, Lq, Lq + 7, D)
    run_and_compare(Q, K, V, synth.random_mask(3, Lq, Lq + 7, 0.2, seed=Lq), "f32", True)
    run_and_compare(Q, K, V, np.ones((3, Lq, Lq + 7), np.uint8), "f32", True)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("Lk", [1, 31, 32, 33, 63, 64, 65])
def test_few_keys(Lk, D):
    """Two wavefronts per 32 queries up to 64 keys, four from 65 on: one chunk of keys, two, three; all kept, and few."""
    Q, K, V = inputs(Lk, 3, 2, min(Lk, 45), Lk, D)
    for density in (1.0, 0.1):
        mask = synth.random_mask(2, min(Lk, 45), Lk, density, seed=Lk)
        run_and_compare(Q, K, V, mask, "f32", False)
        run_and_compare(Q, K, V, mask, "f32", True)
