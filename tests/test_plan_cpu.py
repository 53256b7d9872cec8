"""The rules by which a pass loop is cut into launches (plan.cpp), on the CPU:
every pass once, no launch of more passes than a tile's halo holds, and the
short loops, which one-pass launches run faster, without deep ones."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1306_5390_amd", "csrc")
HALO = 16                        # columns, and rows at most, around a tile

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-o", exe,
                    os.path.join(ROOT, "tests", "sanitize", "plan_driver.cpp"), os.path.join(CSRC, "plan.cpp")],
                   check=True)

    def run(cases):
        """Per case (rows, cols, beta, k, maps[, pixels of the batch]): few, lead, launches,
        cycle launches, cycle pays, the same two of a batch's image."""
        text = "".join("%d %d %d %d %d %d\n" % (*c, *(() if len(c) == 6 else (c[0] * c[1],))) for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        got = []
        for line in out.splitlines():
            left, right, batch, _ = line.split("|")
            few, lead, *launches = left.split()
            *cycle, pays = right.split()
            got.append((int(few), int(lead), [tuple(map(int, x.split(":"))) for x in launches],
                        [tuple(map(int, x.split(":"))) for x in cycle], pays == "1",
                        int(batch.split()[0]), [tuple(map(int, x.split(":"))) for x in batch.split()[1:]]))
        assert len(got) == len(cases)
        return got
    return run


SIZES = [(1, 1), (9, 224), (128, 128), (321, 481), (1024, 1024), (997, 1031), (1448, 1449), (2048, 1024),
         (2048, 2048), (2403, 3201), (4096, 4096), (4099, 4001), (6001, 8001), (8192, 8192), (46340, 46340),
         (8192, 256), (1 << 30, 1), (1, (1 << 31) - 1)]


def test_every_pass_once_within_the_halo(plans):
    cases = [(r, c, b, k, m) for r, c in SIZES for b in (1, 2, 3, 4) for k in (*range(41), 1023, 1024) for m in (0, 1)]
    for (_, _, beta, k, _), (_, lead, launches, cycle, _, blead, batch) in zip(cases, plans(cases)):
        for ahead, plan in ((lead, launches), (blead, batch)):
            at = 0
            for j, (start, passes) in enumerate(plan):
                assert start == at and 1 <= passes <= HALO // beta and (j >= ahead or passes == 1)
                at += passes
            assert at == k
        # each launch but the first begins with the last pass of the one before
        for j, (start, passes, advance) in enumerate(cycle):
            assert 2 <= passes <= HALO // beta and (j == 0 or start == at)
            at = start + passes - 1
            assert advance == (passes if j + 1 == len(cycle) else passes - 1)
            # so that tiles that only alternate are where they were
            assert j == 0 or j + 1 == len(cycle) or advance % 2 == 0
        assert k <= 1 or at == k - 1


# (rows, cols, beta): the longest loop without a deep launch
@pytest.mark.parametrize("rows,cols,beta,few", [
    (128, 128, 1, 1), (1024, 1024, 2, 1), (2048, 2048, 1, 3), (4096, 4096, 1, 4), (8192, 8192, 1, 4),
    (2048, 2048, 2, 3), (8192, 8192, 2, 3), (2048, 2048, 3, 3), (8192, 8192, 3, 3), (512, 512, 4, 2),
    (1024, 1024, 4, 4), (2048, 2048, 4, 5), (8192, 8192, 4, 4), (997, 1031, 3, 1), (4099, 4001, 4, 2)])
def test_short_loops_run_by_one_pass_launches(plans, rows, cols, beta, few):
    for k, (_, lead, launches, *_) in zip(range(1, 12), plans([(rows, cols, beta, k, 1) for k in range(1, 12)])):
        assert (lead == k and len(launches) == k) == (k <= few), (k, launches)


def test_images_without_interior_pixels(plans):
    for (_, lead, _, _, pays, *_) in plans([(9, 8, 4, 32, 1), (8, 900, 4, 32, 1), (2, 70000, 1, 32, 1)]):
        assert lead == 32 and not pays


# (pixels of the batch, beta): the longest loop without a deep launch, and the longest with
# one dense launch ahead (beta 3 and 4)
@pytest.mark.parametrize("px,beta,few,one", [(1 << 20, 1, 0, 0), (1 << 20, 4, 0, 0), (3 << 20, 4, 2, 0),
                                             (1 << 22, 1, 3, 3), (1 << 22, 2, 3, 3), (1 << 22, 3, 3, 5),
                                             (1 << 27, 4, 3, 4), (1 << 27, 2, 3, 3)])
def test_short_loops_of_batches(plans, px, beta, few, one):
    for k, (*_, lead, launches) in zip(range(1, 12), plans([(64, 64, beta, k, 1, px) for k in range(1, 12)])):
        assert (len(launches) == k and lead >= k) == (k <= few), (k, launches)
        assert beta < 3 or k <= few or lead == (1 if k <= one else 0)


@pytest.mark.parametrize("rows,cols,beta,few", [(128, 128, 1, 1), (1024, 1024, 2, 2), (128, 128, 4, 6), (1448, 1448, 4, 6),
                                                (321, 481, 4, 2), (997, 1031, 4, 2), (321, 481, 3, 1), (2048, 2048, 4, 8)])
def test_short_loops_with_the_period2_stop(plans, rows, cols, beta, few):
    got = plans([(rows, cols, beta, k, 1) for k in range(1, 12)])
    assert [pays for *_, pays, _, _ in got] == [k > few for k in range(1, 12)]
