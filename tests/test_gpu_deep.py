"""Deep shape: the pass loop with several passes per launch that follow only
what the pass before changed, against the oracle (bit for bit) and, on an
image whose launches look at several tiles per workgroup, against the dense
one-pass shape."""
import numpy as np
import pytest

import oracle
from paper_1306_5390_amd import synth

pytestmark = pytest.mark.gpu

DEEP = 13        # the deep shape
DENSE = 3        # one dense pass per launch
COLS = 224       # owned columns of a tile


def _modules():
    import torch
    import paper_1306_5390_amd as m
    return torch, m


def _oscillating(rows, cols, seed):
    """Tilted plane with a little noise: pixels at the steps alternate."""
    rng = np.random.Generator(np.random.PCG64(seed))
    y, x = np.mgrid[0:rows, 0:cols]
    img = 60 + (y * 7 + x * 11) // 9 % 120 + rng.integers(0, 3, size=(rows, cols)) * 12
    return np.clip(img, 0, 255).astype(np.uint8)


def _run(img, alpha, beta, k, shape=DEEP, offset=0, in_place=False, cycle=False):
    torch, m = _modules()
    rows, cols = img.shape
    cls = m.size_class(rows * cols)
    saved = m.get_tuning_class(beta, cls)
    m.set_tuning_class(beta, cls, shape)
    try:
        buf = torch.zeros(rows * cols + 8, dtype=torch.uint8, device="cuda:0")
        src = buf[offset:offset + rows * cols].view(rows, cols)
        src.copy_(torch.from_numpy(img))
        out = src if in_place else torch.full((rows, cols), 77, dtype=torch.uint8, device="cuda:0")
        ws = torch.full((m.workspace_bytes(rows, cols, alpha, beta, k),), 0xA5, dtype=torch.uint8,
                        device="cuda:0")
        got, ch, it = m.denoise_async(src, alpha, beta, k, out=out, workspace=ws, stop_on_cycle=cycle)
        return got.cpu().numpy(), int(it.item()), ch.cpu().tolist()
    finally:
        m.set_tuning_class(beta, cls, saved)


def _check(img, alpha, beta, k, **kw):
    ref, rit, rch = (oracle.denoise_cycle if kw.get("cycle") else oracle.denoise)(img, alpha, beta, k)
    got, it, ch = _run(img, alpha, beta, k, **kw)
    assert np.array_equal(got, ref), (img.shape, alpha, beta, k, kw)
    assert it == rit and ch[:it] == list(rch)[:rit] and not any(ch[it:]), (it, rit, ch, rch)


@pytest.mark.parametrize("beta", [1, 2, 3, 4])
@pytest.mark.parametrize("rows,cols", [(1, 1), (2 * 4 + 1, COLS), (65, COLS + 1), (70, 2 * COLS - 1),
                                       (131, 3 * COLS + 16), (260, 241)])
def test_sizes_and_launch_counts(beta, rows, cols):
    """Around the edges of tiles; k around the passes of one launch and of two."""
    most = {1: 16, 2: 8}.get(beta, 4)
    for i, k in enumerate((1, most - 1, most, most + 1, 2 * most + 3)):
        img = synth.noisy_image(rows, cols, (0.05, 0.3, 0.5)[i % 3], 40 + i)
        _check(img, (20, 35)[i % 2], beta, k, offset=i % 4, in_place=i % 2 == 1)


@pytest.mark.parametrize("beta", [1, 2, 3, 4])
def test_alternating_images(beta):
    """Tiles that only alternate between two images: skipped within a launch
    and by later launches, whose counts and parity must still be right."""
    for i, k in enumerate((9, 24, 33, 40)):
        _check(_oscillating(150, 500 + i, i), 6 + 2 * i, beta, k)


@pytest.mark.parametrize("alpha", [0, 1, 255])
@pytest.mark.parametrize("beta", [1, 3])
def test_band_extremes(alpha, beta):
    """alpha 0: every pixel is a candidate in every pass (dense strips, full
    queues); alpha 255: none is."""
    _check(synth.noisy_image(90, 470, 0.4, 3), alpha, beta, 12)


def test_narrow_tall_image_without_maps():
    """256 columns and many rows: the change maps do not fit the workspace,
    and every launch tests every pixel in its first pass."""
    _check(_oscillating(2500, 256, 5), 8, 1, 40)


@pytest.mark.parametrize("beta,k", [(1, 40), (2, 26), (3, 13)])
def test_many_tiles_per_workgroup(beta, k):
    """More tiles than two grids that fit on the device: a workgroup looks at
    several, most of them idle after the first launches."""
    img = synth.noisy_image(1100, 1200, 0.2, 9)
    img = np.tile(img, (5, 5))[:5303, :5900]
    ref = _run(img, 20, beta, k, shape=DENSE)
    got = _run(img, 20, beta, k)
    assert np.array_equal(got[0], ref[0]) and got[1:] == ref[1:]


@pytest.mark.parametrize("big", [False, True])
@pytest.mark.parametrize("in_place", [False, True])
def test_batch_of_mixed_images(big, in_place):
    """Every beta in one batch, with empty images, k 0 and k across launches;
    `big` adds images that make the batch one with dense lead launches.  Two
    runs (the second replays the captured graph)."""
    torch, m = _modules()
    specs, imgs = [], []
    for i, (r, c, k) in enumerate([(70, 300, 5), (33, 225, 0), (0, 40, 7), (129, 448, 33), (5, 700, 9), (200, 223, 17),
                                   (64, 64, 1), (150, 500, 40)]):
        for beta in (1, 2, 3, 4):
            specs.append((r, c, 12 + i, beta, k))
            imgs.append(_oscillating(r, c, i) if i % 2 else synth.noisy_image(r, c, 0.3, 60 + i))
    want = [oracle.denoise(im, s[2], s[3], s[4]) for s, im in zip(specs, imgs)]
    if big:
        im = np.tile(synth.noisy_image(512, 600, 0.3, 5), (6, 6))
        for beta in (1, 2):
            specs.append(im.shape + (20, beta, 21))
            imgs.append(im)
            want.append(_run(im, 20, beta, 21, shape=DENSE))
    for b in (1, 2, 3, 4):
        assert m.get_batch_tuning_class(b, 0) == DEEP
    plan = m.Batch(specs)
    src = plan.new_arena()
    dst = src if in_place else plan.new_arena()
    stream = torch.cuda.Stream()
    for _ in range(2):
        for i, im in enumerate(imgs):
            plan.view(src, i).copy_(torch.from_numpy(im))
        stream.wait_stream(torch.cuda.current_stream())
        plan.run(src, dst, stream=stream)
        torch.cuda.synchronize()
        for i, ((it, ch), w) in enumerate(zip(plan.results(), want)):
            assert np.array_equal(plan.view(dst, i, out=True).cpu().numpy(), w[0]), specs[i]
            assert it == w[1] and list(ch) == list(w[2])[:it], specs[i]
    plan.close()


# Up to 256 tiles a batch has low tiles of 16 waves (256 and 257 images of one
# tile, 70 of four), and all images of one beta share their launches.
@pytest.mark.parametrize("specs", [[(1, 1, 1, 3)], [(40, 200, b, 17) for b in (1, 2, 3, 4)],
                                   [(300, 700, 1, 20), (301, 701, 2, 20), (131, 449, 3, 9), (500, 230, 4, 5)],
                                   [(64, 4 * COLS, 1, 9)] * 70, [(30, COLS, 2, 9)] * 256, [(30, COLS, 2, 9)] * 257],
                         ids=["one", "betas", "low", "four-tiles", "full", "over"])
def test_small_batches(specs):
    _check_batch([(r, c, 9, b, k) for r, c, b, k in specs],
                 [_oscillating(r, c, i % 5) if i % 2 else synth.noisy_image(r, c, 0.3, i % 7)
                  for i, (r, c, _, _) in enumerate(specs)])


# From 2^24 pixels on images share launches only if no beta has most of the work.
@pytest.mark.parametrize("betas", [(1, 2, 1, 2), (1, 1, 1, 2)])
def test_large_batches(betas):
    im = np.tile(synth.noisy_image(512, 600, 0.3, 5), (4, 4))[:, :2399]
    specs = [im.shape + (20, b, 21) for b in betas]
    want = {b: _run(im, 20, b, 21, shape=DENSE) for b in betas}
    _check_batch(specs, [im] * len(betas), [want[b] for b in betas])


def _check_batch(specs, imgs, want=None):
    torch, m = _modules()
    plan = m.Batch(specs)
    src, dst = plan.new_arena(), plan.new_arena()
    for i, im in enumerate(imgs):
        plan.view(src, i).copy_(torch.from_numpy(im))
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    seen = {}
    for _ in range(2):
        plan.run(src, dst, stream=stream)
        torch.cuda.synchronize()
        for i, (s, im, (it, ch)) in enumerate(zip(specs, imgs, plan.results())):
            key = (s, im.tobytes())
            if key not in seen:
                seen[key] = want[i] if want else oracle.denoise(im, s[2], s[3], s[4])
            w = seen[key]
            assert np.array_equal(plan.view(dst, i, out=True).cpu().numpy(), w[0]), (i, s)
            assert it == w[1] and list(ch) == list(w[2])[:it], (i, s)
    plan.close()


@pytest.mark.parametrize("passes", [0, 1, 4, -1])
def test_served_requests(passes):
    """Requests at different launches share a step's deep launch."""
    _, m = _modules()
    import time
    import torch
    srv = m.Server(96 << 20, passes_per_step=passes)
    todo = {}
    for i in range(24):
        im = synth.noisy_image(40 + 17 * i, 230 + 29 * i, 0.25, i) if i % 3 else _oscillating(90, 300 + i, i)
        p = (20, 1 + i % 4, 1 + 3 * (i % 7))
        todo[srv.submit(torch.from_numpy(im).cuda(), *p)] = oracle.denoise(im, *p)
    end = time.time() + 60
    while todo and time.time() < end:
        for rid in srv.next_done():
            out, it, ch, _ = srv.poll(rid)
            ref, rit, rch = todo.pop(rid)
            assert np.array_equal(out.cpu().numpy(), ref) and it == rit and list(ch) == list(rch)[:it]
            srv.release(rid)
    assert not todo
    srv.close()


# _oscillating(40, 200, seed) stops with pass `last`: around the first pass of
# the second launch (15 at beta 1, 7 at beta 2, 3 at beta 3), which that launch
# runs again to have the image two passes before its next one.
@pytest.mark.parametrize("beta,alpha,seed,last", [(1, 6, 4, 14), (1, 6, 26, 15), (1, 2, 10, 16), (2, 2, 2, 6),
                                                  (2, 2, 0, 7), (2, 2, 1, 8), (3, 2, 4, 4)])
def test_period2_stop_around_launches(beta, alpha, seed, last):
    img = _oscillating(40, 200, seed)
    assert oracle.denoise_cycle(img, alpha, beta, 40)[1] == last + 1
    for i, k in enumerate((last, last + 1, last + 2, last + 16, 40)):
        _check(img, alpha, beta, k, cycle=True, in_place=i % 2 == 1, offset=i % 3)


@pytest.mark.parametrize("beta", [1, 2, 3, 4])
@pytest.mark.parametrize("rows,cols", [(1, 1), (2 * 4 + 1, COLS), (70, 2 * COLS - 1), (131, 3 * COLS + 16)])
def test_period2_sizes(beta, rows, cols):
    for i, k in enumerate((1, 2, 3, 6, 9, 24)):
        img = synth.noisy_image(rows, cols, 0.3, 5 + i) if i % 2 == 0 else _oscillating(rows, cols, i)
        _check(img, 8, beta, k, cycle=True, offset=i % 4, in_place=i % 3 == 1)


# From 2^22 pixels on the first launch is shorter, and rows on dword boundaries
# decide, with the pixels and passes, between deep and one-pass launches.
@pytest.mark.parametrize("beta", [1, 2, 3, 4])
@pytest.mark.parametrize("cols", [2048, 2051])
def test_period2_large_images(beta, cols):
    img = synth.noisy_image(2050, cols, 0.2, 9)
    for k in (2, 3, 5, 9, 20):
        got, ref = (_run(img, 20, beta, k, shape=s, cycle=True) for s in (DEEP, DENSE))
        assert np.array_equal(got[0], ref[0]) and got[1:] == ref[1:], (beta, cols, k, got[1:], ref[1:])


def test_period2_many_tiles_per_workgroup():
    img = np.tile(synth.noisy_image(1100, 1200, 0.2, 9), (5, 5))[:5303, :5899]
    got, ref = (_run(img, 20, 1, 40, shape=s, cycle=True) for s in (DEEP, DENSE))
    assert np.array_equal(got[0], ref[0]) and got[1:] == ref[1:]


# The longest loops that run by one-pass launches only, one and three passes more, in
# each range of sizes that the rule tells apart (the largest against the dense shape).
@pytest.mark.parametrize("beta,rows,cols,few", [(1, 96, 128, 1), (2, 97, 129, 1), (3, 1024, 1024, 1), (4, 500, 512, 2),
                                                (4, 1024, 1024, 4), (1, 2048, 1024, 3), (2, 2048, 1024, 3),
                                                (3, 2048, 1024, 3), (4, 2048, 1024, 5), (3, 2048, 2304, 3),
                                                (4, 2048, 2304, 4), (4, 2049, 2305, 2), (1, 4096, 4096, 4),
                                                (3, 4096, 4096, 3), (4, 8192, 256, 10), (1, 8192, 256, 6)])
def test_short_loops(beta, rows, cols, few):
    for i, k in enumerate((few, few + 1, few + 3)):
        img = synth.noisy_image(rows, cols, 0.2, i) if rows * cols < 1 << 20 else \
            np.tile(synth.noisy_image(256, 256, 0.2, i), (rows // 256 + 1, cols // 256 + 1))[:rows, :cols].copy()
        if rows * cols < 1 << 20:
            _check(img, 20, beta, k, offset=i, in_place=i % 2 == 1)
        else:
            got, ref = _run(img, 20, beta, k, in_place=i % 2 == 1), _run(img, 20, beta, k, shape=DENSE)
            assert np.array_equal(got[0], ref[0]) and got[1:] == ref[1:]


# Loops of a batch that have dense launches only, or one ahead of the deep ones, beside longer ones.
def test_batch_of_short_loops():
    specs, imgs = [], []
    for beta in (1, 2, 3, 4):
        for k in range(1, 8):
            imgs.append(synth.noisy_image(600 + k, 620 + beta, 0.3, 10 * beta + k))
            specs.append(imgs[-1].shape + (20, beta, k))
    assert sum(im.size for im in imgs) > 1 << 23
    _check_batch(specs, imgs, [_run(im, *s[2:], shape=DENSE) for s, im in zip(specs, imgs)])
