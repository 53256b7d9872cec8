"""Deep launches over many more tiles than fit on the device at once, where a
workgroup looks at several tiles: stops in such launches (a period-2 image, a
fixed point), the pass after a period-2 stop, and many-image launches of the
same kind.  The images are blocks that cannot reach each other, an alternating
patch in the middle of each of every third one, so the oracle's result for one
block is that of them all."""
import numpy as np
import pytest

import oracle
from paper_1306_5390_amd import synth
from tests.test_gpu_deep import DENSE, _check_batch, _oscillating, _run

pytestmark = pytest.mark.gpu

ROWS, COLS = 56, 232             # of a block
DOWN, ACROSS = 95, 25            # blocks of the image: 5320 x 5800, 2100 tiles of the largest kind


def _tiled(block, blank):
    pick = np.arange(DOWN * ACROSS).reshape(DOWN, ACROSS) % 3 == 0
    img = np.where(pick[:, None, :, None], block[None, :, None, :], blank)
    return np.ascontiguousarray(img.reshape(DOWN * ROWS, ACROSS * COLS).astype(np.uint8)), int(pick.sum())


def _block_image(alpha, beta, k, seed, cycle):
    """(image, its result, iterations, counts), by the oracle's on one block."""
    block = np.full((ROWS, COLS), 128, np.uint8)
    block[8:48, 8:208] = _oscillating(40, 200, seed)
    out, it, ch = (oracle.denoise_cycle if cycle else oracle.denoise)(block, alpha, beta, k)
    for edge in (out[:4], out[-4:], out[:, :4], out[:, -4:]):
        assert (edge == 128).all()               # no block reaches the next one
    img, n = _tiled(block, 128)
    return img, _tiled(out, 128)[0], it, [n * c for c in list(ch)[:it]]


# (beta, alpha, seed of the block, passes to the stop).  The launches' passes
# end at 7, 21, 35 at beta 1 and at 5, 11, 17 at beta 2: the stop comes in the
# second and in the third, an even and an odd number of passes from its end.
@pytest.mark.parametrize("beta,alpha,seed,stop", [(1, 4, 5, 12), (1, 4, 0, 13), (1, 2, 52, 23), (1, 2, 9, 24),
                                                  (2, 2, 0, 8), (2, 2, 1, 9), (2, 2, 32, 13), (2, 2, 42, 9)])
def test_period2_stop(beta, alpha, seed, stop):
    img, want, it, ch = _block_image(alpha, beta, 40, seed, True)
    assert it == stop
    got = _run(img, alpha, beta, 40, cycle=True)
    assert np.array_equal(got[0], want) and got[1] == it and got[2] == ch + [0] * (40 - it)


def test_fixed_point():
    img, want, it, ch = _block_image(2, 2, 40, 42, False)
    assert it == 9 and ch[-1] == 0
    got = _run(img, 2, 2, 40)
    assert np.array_equal(got[0], want) and got[1] == it and got[2] == ch + [0] * (40 - it)


def test_batch():
    """Two groups of 4000 tiles and more a launch, with an image that comes to
    a fixed point and others that have fewer launches than the group."""
    noise = np.tile(synth.noisy_image(1100, 1200, 0.2, 9), (5, 5))[:5303, :5899]
    fixed, out, it, ch = _block_image(2, 2, 40, 42, False)
    specs, imgs, want = [], [], []
    for beta in (1, 2):
        specs.append(noise.shape + (20, beta, 40))
        imgs.append(noise)
        want.append(_run(noise, 20, beta, 40, shape=DENSE))
        specs.append(fixed.shape + (2, beta, 40))
        imgs.append(fixed)
        want.append((out, it, ch) if beta == 2 else _run(fixed, 2, 1, 40, shape=DENSE))
        for k in (1, 5, 12):
            small = synth.noisy_image(300, 500, 0.3, k)
            specs.append(small.shape + (20, beta, k))
            imgs.append(small)
            want.append(oracle.denoise(small, 20, beta, k))
    assert want[6][1] < 40                       # (the fixed point at beta 2)
    _check_batch(specs, imgs, want)
