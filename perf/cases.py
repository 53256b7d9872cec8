"""The work a program gives this library: single images from a thumbnail to
8192 x 8192 through the synchronous, the asynchronous and the period-2 entry
points, a mixed batch, a burst of served requests, Algorithm 1's cardinality
matrix, and the noise and error sum around an experiment.

listed() names the cases, draw(rng) gives another one of the same ranges,
prepare(case, seed) makes what a program holds before the call, run(state) is
one pass through the public entry points, work(case) the bytes and operations
the path cannot do without, and exact(case, seed) the same results from plain
torch in 64-bit integers.

The library's committed tuning cache is applied, as bench.py applies it.
"""
import functools
import math
import random
import time

import torch

import paper_1306_5390_amd as phg
from paper_1306_5390_amd import autotune, synth

DEVICE = "cuda:0"
LARGEST = 8192 * 8192 * 32 * 25          # pixels x passes x window of the largest listed case


def listed():
    return [
        # the smallest square of the paper's resolution figure, with its k: launches and latency only
        {"name": "image_128_b1_k5", "kind": "image", "call": "sync", "rows": 128, "cols": 128,
         "alpha": 20, "beta": 1, "k": 5, "density": 0.10},
        # one frame of the paper's data set size: the ordinary interactive call, odd width
        {"name": "image_321x481_b1_k10", "kind": "image", "call": "sync", "rows": 321, "cols": 481,
         "alpha": 20, "beta": 1, "k": 10, "density": 0.10},
        # a ragged megapixel photograph with a wide window
        {"name": "image_997x1031_b3_k8", "kind": "image", "call": "sync", "rows": 997, "cols": 1031,
         "alpha": 30, "beta": 3, "k": 8, "density": 0.20},
        # the opt-in stop on a repeating image, which a program uses when it does not know k
        {"name": "cycle_1023x1537_b2_k32", "kind": "image", "call": "cycle", "rows": 1023, "cols": 1537,
         "alpha": 20, "beta": 2, "k": 32, "density": 0.15},
        # the largest square of the resolution figure, both windows, results left on the device
        {"name": "sweep_2048_b1_k32", "kind": "image", "call": "async", "rows": 2048, "cols": 2048,
         "alpha": 20, "beta": 1, "k": 32, "density": 0.30},
        {"name": "sweep_2048_b2_k32", "kind": "image", "call": "async", "rows": 2048, "cols": 2048,
         "alpha": 20, "beta": 2, "k": 32, "density": 0.30},
        # a scanned page, odd in both directions: no row starts on a dword
        {"name": "scan_4099x4001_b1_k32", "kind": "image", "call": "async", "rows": 4099, "cols": 4001,
         "alpha": 20, "beta": 1, "k": 32, "density": 0.50},
        # the benchmark's image: half its pixels are noise
        {"name": "large_8192_b2_k32", "kind": "image", "call": "async", "rows": 8192, "cols": 8192,
         "alpha": 20, "beta": 2, "k": 32, "density": 0.50},
        # a folder of pictures of mixed sizes and settings, as one batch
        {"name": "batch_48", "kind": "batch", "count": 48, "lo": 128, "hi": 2048, "k": 32},
        # a burst of requests at the server, four passes per step as the benchmark serves
        {"name": "serve_24", "kind": "serve", "count": 24, "lo": 256, "hi": 2048, "k": 16},
        # the intermediate of Algorithm 1, for inspection of a whole image
        {"name": "cardinality_2048_b2", "kind": "cardinality", "rows": 2048, "cols": 2048,
         "alpha": 20, "beta": 2, "density": 0.30},
        # an experiment's frame: noise onto a clean image, and the error sum behind its PSNR
        {"name": "noise_error_4096", "kind": "noise", "rows": 4096, "cols": 4096, "density": 0.20},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["image"] * 8 + ["batch", "serve", "cardinality", "noise"])
    if kind in ("batch", "serve"):
        return {"kind": kind, "count": _log_int(rng, 8, 48 if kind == "batch" else 24),
                "lo": 128 if kind == "batch" else 256, "hi": _log_int(rng, 512, 2048),
                "k": rng.choice([8, 16, 32] if kind == "batch" else [8, 16])}
    if kind == "image":
        while True:
            case = {"kind": kind, "call": rng.choice(["sync", "sync", "async", "async", "cycle"]),
                    "rows": _log_int(rng, 96, 8192), "cols": _log_int(rng, 96, 8192),
                    "alpha": rng.randint(10, 40), "beta": rng.choice([1, 1, 1, 2, 2, 2, 3, 4]),
                    "k": _log_int(rng, 4, 32), "density": round(rng.uniform(0.05, 0.60), 3)}
            window = (2 * case["beta"] + 1) ** 2
            if case["rows"] * case["cols"] * case["k"] * window <= LARGEST:
                return case
    case = {"kind": kind, "rows": _log_int(rng, 256, 4096), "cols": _log_int(rng, 256, 4096),
            "density": round(rng.uniform(0.05, 0.60), 3)}
    if kind == "cardinality":
        case.update(alpha=rng.randint(10, 40), beta=rng.choice([1, 2, 3, 4]),
                    rows=min(case["rows"], 2048), cols=min(case["cols"], 2048))
    return case


# ---- inputs ----------------------------------------------------------------------

def _clean(rows, cols, seed):
    """A grey image like synth.clean_image's, drawn on the GPU: eight convex
    regions on a background, a gradient of 40 levels, Gaussian texture."""
    rng = random.Random(seed)
    y = torch.arange(rows, device=DEVICE, dtype=torch.float32)[:, None]
    x = torch.arange(cols, device=DEVICE, dtype=torch.float32)[None, :]
    base = torch.full((rows, cols), rng.uniform(20, 235), device=DEVICE)
    for _ in range(8):
        cy, cx = rng.uniform(0, rows), rng.uniform(0, cols)
        rad = rng.uniform(0.1, 0.4) * min(rows, cols)
        level, start, sides = rng.uniform(20, 235), rng.uniform(0, 6.28), rng.randint(3, 8)
        inside = torch.ones((rows, cols), dtype=torch.bool, device=DEVICE)
        for s in range(sides):
            a = start + 2 * math.pi * s / sides
            inside &= (y - cy) * math.sin(a) + (x - cx) * math.cos(a) < rad * rng.uniform(0.6, 1.0)
        base[inside] = level
    theta = rng.uniform(0, 2 * math.pi)
    ramp = math.sin(theta) * y / max(rows - 1, 1) + math.cos(theta) * x / max(cols - 1, 1)
    base += 40.0 * (ramp - 0.5 * (math.sin(theta) + math.cos(theta)))
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    base += 6.0 * torch.randn((rows, cols), device=DEVICE, generator=gen)
    return base.round_().clamp_(0, 255).to(torch.uint8)


def _noisy(rows, cols, density, seed):
    img = _clean(rows, cols, seed)
    gen = torch.Generator(device=DEVICE).manual_seed(seed + 1_000_003)
    u = torch.rand((rows, cols), device=DEVICE, generator=gen)
    img[u < density] = 255
    img[u < 0.5 * density] = 0
    return img


def _members(case):
    """(rows, cols, alpha, beta, k, density) of the images of a batch or a
    burst: the case's own, whatever the seed of the pixels."""
    rng = random.Random("%s %d %d %d" % (case["kind"], case["count"], case["hi"], case["k"]))
    got = []
    for _ in range(case["count"]):
        alpha = rng.randint(10, 40) if case["kind"] == "batch" else 20
        got.append((_log_int(rng, case["lo"], case["hi"]), _log_int(rng, case["lo"], case["hi"]),
                    alpha, rng.choice([1, 2]), case["k"], rng.uniform(0.05, 0.60)))
    return got


@functools.lru_cache(maxsize=1)
def _tuned():
    return autotune.load()


def _inputs(case, seed):
    seed = 7919 * int(seed) + 17
    if case["kind"] in ("batch", "serve"):
        return [_noisy(r, c, d, seed + 31 * i) for i, (r, c, _, _, _, d) in enumerate(_members(case))]
    if case["kind"] == "noise":
        return _clean(case["rows"], case["cols"], seed)
    return _noisy(case["rows"], case["cols"], case["density"], seed)


def prepare(case, seed):
    _tuned()
    data = _inputs(case, seed)
    state = {"case": case, "data": data, "seed": int(seed)}
    if case["kind"] == "image" and case["call"] != "sync":
        # a program that leaves results on the device keeps its buffers
        state["keep"] = {
            "out": torch.empty_like(data),
            "workspace": torch.empty(phg.workspace_bytes(case["rows"], case["cols"], case["alpha"],
                                                         case["beta"], case["k"]),
                                     dtype=torch.uint8, device=DEVICE),
            "changed": torch.empty(case["k"], dtype=torch.int64, device=DEVICE),
            "iterations": torch.empty(1, dtype=torch.int32, device=DEVICE)}
    elif case["kind"] == "batch":
        plan = phg.Batch([m[:5] for m in _members(case)], device=DEVICE)
        src, dst = plan.new_arena(), plan.new_arena()
        for i, img in enumerate(data):
            plan.view(src, i).copy_(img)
        state.update(plan=plan, src=src, dst=dst, stream=torch.cuda.Stream(device=DEVICE))
    elif case["kind"] == "serve":
        need = sum(2 * img.numel() for img in data) + (256 << 20)
        state["server"] = phg.Server(need, device=DEVICE, passes_per_step=4)
    return state


# ---- one pass --------------------------------------------------------------------

def _serve(state):
    server, members = state["server"], _members(state["case"])
    place = {}
    for i, (img, m) in enumerate(zip(state["data"], members)):
        place[server.submit(img, m[2], m[3], m[4])] = i
    outs, iters, changed = [None] * len(members), [0] * len(members), [None] * len(members)
    left = len(members)
    while left:
        done = server.next_done()
        if not done:
            time.sleep(0)
        for rid in done:
            view, n, counts, _ = server.poll(rid)
            i = place[rid]
            outs[i], iters[i] = view.clone(), n
            changed[i] = counts + [0] * (members[i][4] - n)
            left -= 1
    # the arena's blocks go back once they have been read
    torch.cuda.current_stream().synchronize()
    for rid in place:
        server.release(rid)
    return outs, torch.tensor(iters), torch.tensor(changed)


def run(state):
    case, data = state["case"], state["data"]
    if case["kind"] == "image":
        a, b, k = case["alpha"], case["beta"], case["k"]
        if case["call"] != "sync":
            return phg.denoise_async(data, a, b, k, **state["keep"], stop_on_cycle=case["call"] == "cycle")
        out, n, counts = phg.denoise(data, a, b, k)
        return out, n, counts + [0] * (k - n)
    if case["kind"] == "batch":
        plan, s = state["plan"], state["stream"]
        s.wait_stream(torch.cuda.current_stream())
        plan.run(state["src"], state["dst"], stream=s)
        torch.cuda.current_stream().wait_stream(s)
        return state["dst"], plan.changed, plan.iterations
    if case["kind"] == "serve":
        return _serve(state)
    if case["kind"] == "cardinality":
        return phg.cardinality(data, case["alpha"], case["beta"])
    t_pepper, t_salt = synth.noise_thresholds(case["density"])
    noisy = phg.salt_pepper(data, state["seed"], t_pepper, t_salt)
    return noisy, phg.sq_diff_sum(data, noisy)


# ---- what the path cannot do without ------------------------------------------------

def work(case):
    """Bytes: every image read once and written once, and the counts.
    Operations: every pixel tested once against its window (two compares
    per neighbour); later passes need only follow what changed."""
    if case["kind"] in ("batch", "serve"):
        px = [(r * c, (2 * b + 1) ** 2 - 1, k) for r, c, _, b, k, _ in _members(case)]
        return {"bytes": sum(2 * n + 8 * k + 4 for n, _, k in px),
                "flops": sum(2 * n * nb for n, nb, _ in px)}
    n = case["rows"] * case["cols"]
    if case["kind"] == "noise":
        # clean read, noisy written; a 64-bit generator step per pixel; a difference and its square
        return {"bytes": 2 * n + 8, "flops": 12 * n}
    nb = (2 * case["beta"] + 1) ** 2 - 1
    if case["kind"] == "cardinality":
        return {"bytes": 5 * n, "flops": 2 * n * nb}
    return {"bytes": 2 * n + 8 * case["k"] + 4, "flops": 2 * n * nb}


# ---- the same results in 64-bit integers ---------------------------------------------

def _pass(img, alpha, beta):
    """Algorithms 1 and 2 on an int64 image: an interior pixel with at most
    two window pixels in (x - alpha, x + alpha] becomes the root mean square
    of the others."""
    rows, cols = img.shape
    out = img.clone()
    h, w = rows - 2 * beta, cols - 2 * beta
    if h <= 0 or w <= 0:
        return out
    x = img[beta:beta + h, beta:beta + w]
    count, total = torch.zeros_like(x), torch.zeros_like(x)
    for dr in range(2 * beta + 1):
        for dc in range(2 * beta + 1):
            y = img[dr:dr + h, dc:dc + w]
            far = (y <= x - alpha) | (y > x + alpha)
            count += far
            total += torch.where(far, y * y, 0)
    mean = total // count.clamp(min=1)
    rms = mean.double().sqrt().floor().long()
    out[beta:beta + h, beta:beta + w] = torch.where(count > (2 * beta + 1) ** 2 - 3, rms, x)
    return out


def _loop(img, alpha, beta, k, cycle=False):
    now, before, changed = img.long(), None, []
    for _ in range(k):
        new = _pass(now, alpha, beta)
        changed.append(int((new != now).sum()))
        repeats = cycle and before is not None and torch.equal(new, before)
        before, now = now, new
        if changed[-1] == 0 or repeats:
            break
    return now.to(torch.uint8), changed


def _noise(img, seed, t_pepper, t_salt):
    """The noise rule on the outputs of a SplitMix64 generator, in wrapping
    64-bit integers."""
    def signed(v):
        return v - (1 << 64) if v >= 1 << 63 else v

    def shifted(z, s):
        return (z >> s) & ((1 << (64 - s)) - 1)

    z = torch.arange(1, img.numel() + 1, dtype=torch.int64, device=DEVICE) * signed(0x9e3779b97f4a7c15)
    z += signed(seed & ((1 << 64) - 1))
    z = (z ^ shifted(z, 30)) * signed(0xbf58476d1ce4e5b9)
    z = (z ^ shifted(z, 27)) * signed(0x94d049bb133111eb)
    u = shifted(z ^ shifted(z, 31), 32).view(img.shape)
    noisy = img.clone()
    noisy[u < t_salt] = 255
    noisy[u < t_pepper] = 0
    return noisy


def exact(case, seed):
    data = _inputs(case, seed)
    if case["kind"] == "image":
        out, changed = _loop(data, case["alpha"], case["beta"], case["k"], case["call"] == "cycle")
        full = changed + [0] * (case["k"] - len(changed))
        if case["call"] == "sync":
            return out, len(changed), full
        return out, torch.tensor(full), torch.tensor([len(changed)], dtype=torch.int32)
    if case["kind"] in ("batch", "serve"):
        got = [_loop(img, a, b, k) for img, (_, _, a, b, k, _) in zip(data, _members(case))]
        iters = [len(ch) for _, ch in got]
        changed = [ch + [0] * (case["k"] - len(ch)) for _, ch in got]
        if case["kind"] == "serve":
            return [out for out, _ in got], torch.tensor(iters), torch.tensor(changed)
        # images lie at 256-byte aligned offsets of the arena
        arena = torch.cat([torch.nn.functional.pad(out.view(-1), (0, -out.numel() % 256)) for out, _ in got])
        return arena, torch.tensor(changed).view(-1), torch.tensor(iters, dtype=torch.int32)
    if case["kind"] == "noise":
        noisy = _noise(data, int(seed), *synth.noise_thresholds(case["density"]))
        return noisy, (data.long() - noisy.long()).square().sum().view(1)
    img, b = data.long(), case["beta"]
    rows, cols = img.shape
    padded = torch.nn.functional.pad(img, (b, b, b, b), value=1 << 20)
    card = torch.zeros_like(img)
    for dr in range(2 * b + 1):
        for dc in range(2 * b + 1):
            card += (padded[dr:dr + rows, dc:dc + cols] - img).abs() < case["alpha"]
    return card.to(torch.int32)
