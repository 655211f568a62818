"""Host-only checks of the choice of tiles for fp32 products: what it returns has a kernel, at every size."""
import random

from tests.f32_form import form

KERNELS = {False: {(128, 1), (64, 1), (64, 4), (32, 4), (16, 4)}, True: {(128, 1), (64, 1), (64, 4), (32, 4), (32, 8), (16, 4)}}


def test_every_size_has_a_kernel():
    rng = random.Random(7)
    seen = {False: set(), True: set()}
    for _ in range(20000):
        M, N, K = (int(2.0 ** rng.uniform(0, 14)) for _ in range(3))
        for wgrad in (False, True):
            tile, split, patches = form(M, N, K, wgrad)
            seen[wgrad].add((tile, split))
            if patches:
                assert (tile, split) in ({(32, 8)} if wgrad else {(32, 4), (16, 4)})
            assert form(M, N, K, wgrad, reach16=False)[0] != 16
    assert seen == KERNELS


def test_small_results_take_small_tiles_at_most_two_or_one_a_unit():
    for wgrad, blocks in ((False, 512), (True, 256)):
        assert form(16, 16 * blocks, 72, wgrad) == (16, 4, 0)
        assert form(16, 16 * blocks + 1, 72, wgrad)[0] > 16


def test_patches_from_operands_beyond_an_l2_on():
    for n, patches in ((7, 0), (8, 1)):
        assert form(64, 128 * n - 64, 1024, False) == (16, 4, 0)      # one block a unit at most: plain order
        assert form(64, 2048 - 64, 512 + n - 7, False) == (16, 4, patches)
