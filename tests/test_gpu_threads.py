"""The synchronous call from more threads at once than it has page-locked
result slots (16), each with its own stream and workspace: some calls read
their results back by a copy instead.  Iterations and counts of every call are
those of the asynchronous entry point, which other tests compare with the
oracle."""
import threading

import pytest

from paper_1306_5390_amd import synth

pytestmark = pytest.mark.gpu

THREADS, CALLS = 24, 8


def test_more_calls_than_slots():
    import torch
    import paper_1306_5390_amd as m
    imgs = [torch.from_numpy(synth.noisy_image(1200 + i, 1100, 0.3, i)).cuda() for i in range(THREADS)]
    specs = [(20, 1 + i % 3, 150 + i) for i in range(THREADS)]
    want = [[t.cpu() for t in m.denoise_async(im, *s)] for im, s in zip(imgs, specs)]
    torch.cuda.synchronize()
    start, wrong = threading.Barrier(THREADS), []

    def work(i):
        stream = torch.cuda.Stream()
        ws = torch.empty(m.workspace_bytes(*imgs[i].shape, *specs[i]), dtype=torch.uint8, device="cuda:0")
        torch.cuda.synchronize()
        start.wait()
        for _ in range(CALLS):
            out, it, ch = m.denoise(imgs[i], *specs[i], workspace=ws, stream=stream)
            ref, rch, rit = want[i]
            if not torch.equal(out.cpu(), ref) or it != int(rit) or ch != rch.tolist()[:it]:
                wrong.append((i, it))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(THREADS)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
