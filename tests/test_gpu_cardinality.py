"""Cardinality matrix at the edges of its two kernels' ranges (a wave per 256
columns of 8 rows; a thread per pixel below 64 columns), and the sum of
squared differences at every relative alignment, against the oracle."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1306_5390_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("beta", [1, 2, 3, 4])
@pytest.mark.parametrize("rows,cols", [(1, 63), (1, 64), (7, 65), (8, 255), (9, 256), (17, 259), (33, 516), (3, 1031)])
def test_cardinality_both_types(beta, rows, cols):
    import torch
    import paper_1306_5390_amd as m
    lib = m.load_library()
    for i, alpha in enumerate((0, 1, 20, 255)):
        img = synth.noisy_image(rows, cols, 0.3, 10 + i)
        img[img > 200] = 255
        want = oracle.cardinality(img, alpha, beta)
        buf = torch.zeros(rows * cols + 4, dtype=torch.uint8, device="cuda:0")
        t = buf[i:i + rows * cols].view(rows, cols)      # every byte offset
        t.copy_(torch.from_numpy(img))
        assert np.array_equal(m.cardinality(t, alpha, beta).cpu().numpy(), want)
        card = torch.full((rows * cols + 8,), -1, dtype=torch.int16, device="cuda:0")
        s = torch.cuda.current_stream().cuda_stream
        m.check(lib.phgrms_cardinality(t.data_ptr(), rows, cols, alpha, beta, card.data_ptr() + 2, ctypes.c_void_p(s)))
        got = card.cpu().numpy()
        assert np.array_equal(got[1:1 + rows * cols].reshape(rows, cols), want)
        assert got[0] == -1 and (got[1 + rows * cols:] == -1).all()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4096, 70001, 1 << 20])
def test_squared_differences(n):
    import torch
    import paper_1306_5390_amd as m
    rng = np.random.Generator(np.random.PCG64(n))
    a, b = (rng.integers(0, 256, n + 32, dtype=np.uint8) for _ in range(2))
    a[:n // 2], b[:n // 2] = 0, 255                       # the largest differences
    ta, tb = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    for oa, ob in [(0, 0), (3, 3), (16, 0), (5, 21), (0, 1), (7, 2)]:
        want = int(((a[oa:oa + n].astype(np.int64) - b[ob:ob + n]) ** 2).sum())
        assert int(m.sq_diff_sum(ta[oa:oa + n].view(1, n), tb[ob:ob + n].view(1, n)).item()) == want


@pytest.mark.parametrize("oi,oo", [(0, 0), (1, 1), (3, 3), (0, 1), (2, 3)])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 1027])
def test_noise_at_every_alignment(n, oi, oo):
    import torch
    import paper_1306_5390_amd as m
    img = synth.noisy_image(1, n, 0.0, n)
    tp, ts = synth.noise_thresholds(0.5)
    want = oracle.salt_pepper(img, 99, tp, ts)
    src = torch.full((n + 8,), 5, dtype=torch.uint8, device="cuda:0")
    dst = torch.full((n + 8,), 6, dtype=torch.uint8, device="cuda:0")
    src[oi:oi + n].copy_(torch.from_numpy(img).view(-1))
    m.salt_pepper(src[oi:oi + n].view(1, n), 99, tp, ts, out=dst[oo:oo + n].view(1, n))
    got = dst.cpu().numpy()
    assert np.array_equal(got[oo:oo + n], np.asarray(want).reshape(-1))
    assert (got[:oo] == 6).all() and (got[oo + n:] == 6).all()


# From 2^24 pixels on images that start at different places have more workgroups.
@pytest.mark.parametrize("n", [(1 << 24) - 1, 1 << 24, (1 << 24) + 4097])
def test_squared_differences_of_many_bytes(n):
    import torch
    import paper_1306_5390_amd as m
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    a, b = (torch.randint(0, 256, (n + 16,), dtype=torch.uint8, device="cuda:0", generator=gen) for _ in range(2))
    a[:n // 2], b[:n // 2] = 0, 255
    for oa, ob in [(0, 0), (0, 1), (7, 2)]:
        want = int((a[oa:oa + n].long() - b[ob:ob + n].long()).square().sum())
        assert int(m.sq_diff_sum(a[oa:oa + n].view(1, n), b[ob:ob + n].view(1, n)).item()) == want


def _check_cardinality(beta, rows, cols, alpha, offset):
    import torch
    import paper_1306_5390_amd as m
    lib = m.load_library()
    img = synth.noisy_image(rows, cols, 0.3, beta + offset)
    want = oracle.cardinality(img, alpha, beta)
    buf = torch.zeros(rows * cols + 4, dtype=torch.uint8, device="cuda:0")
    t = buf[offset:offset + rows * cols].view(rows, cols)
    t.copy_(torch.from_numpy(img))
    assert np.array_equal(m.cardinality(t, alpha, beta).cpu().numpy(), want)
    card = torch.full((rows * cols + 8,), -1, dtype=torch.int16, device="cuda:0")
    m.check(lib.phgrms_cardinality(t.data_ptr(), rows, cols, alpha, beta, card.data_ptr() + 2,
                                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    got = card.cpu().numpy()
    assert np.array_equal(got[1:1 + rows * cols].reshape(rows, cols), want)
    assert got[0] == -1 and (got[1 + rows * cols:] == -1).all()


# The most pixels of a thread per pixel, and some more: a wave per strip.
@pytest.mark.parametrize("beta,rows,cols", [(1, 384, 1023), (1, 384, 1024), (2, 320, 1023), (2, 320, 1024), (3, 511, 512),
                                            (3, 512, 513), (4, 255, 257), (4, 257, 256)])
def test_cardinality_of_small_images(beta, rows, cols):
    _check_cardinality(beta, rows, cols, 20, 0)


# A wave per strip at the edges of its strips: rows about 8, columns about 256, every
# byte offset, the extremes of the band.
@pytest.mark.parametrize("beta", [1, 2, 3, 4])
@pytest.mark.parametrize("rows,cols", [(1, 400001), (7, 60001), (8, 50180), (9, 50175), (6145, 64), (6151, 65), (1601, 255),
                                       (1600, 256), (1537, 259), (1543, 516)])
def test_cardinality_by_strips(beta, rows, cols):
    for offset, alpha in enumerate((0, 1, 20, 255)):
        _check_cardinality(beta, rows, cols, alpha, offset)
