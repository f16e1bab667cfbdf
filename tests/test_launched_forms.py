"""The forms that decode and append launches take, from the library's planner alone (no GPU).

tests/host_asan/forms_driver.cpp builds plans with plan.cpp and checks that what a launch
reads covers every token, head and key once and lies in the workspace; here it gets random
batches, and batches whose form is known."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_03077_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                                reason="needs g++ and the ROCm headers")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("forms") / "forms")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, os.path.join(CSRC, "plan.cpp"),
           os.path.join(ROOT, "tests", "host_asan", "forms_driver.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def line(lens, new, hq, hkv, cus=256, units_per_cu=3, min_split=16, max_splits=64, q_tile=0):
    """A plan for the driver; new is None for decode."""
    head = [int(new is not None), len(lens), hq, hkv, cus, units_per_cu, min_split, max_splits, q_tile]
    return " ".join(map(str, head + list(lens) + list(new or [])))


def forms(driver, lines):
    r = subprocess.run([driver], input="\n".join(lines) + "\n", capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    out = []
    for row in r.stdout.splitlines():
        f = row.split()
        out.append(dict(zip(("groups", "parts", "pages", "singles", "table_singles", "splits",
                             "workspace", "plain"), map(int, f[1:])), form=f[0]))
    assert len(out) == len(lines)
    return out


def test_random_launches_cover_every_key_once(driver):
    rng = random.Random(26)
    lines = []
    for _ in range(400):
        hkv, G = rng.choice([1, 2, 3, 8]), rng.choice([1, 2, 3, 4, 5, 7, 8, 12, 16])
        B = rng.randint(1, 24)
        new = [1 if rng.random() < 0.4 else rng.choice([2, 15, 16, 17, 31, 64, 100, 333, 1000])
               for _ in range(B)]
        prior = [rng.choice([0, 1, 15, 31, 32, 33, 500, 2000, 9000, 70000]) for _ in range(B)]
        append = rng.random() < 0.8
        q_tile = rng.choice([0, 0, 0, rng.randint(1, 256 // G)])
        lines.append(line([p + c for p, c in zip(prior, new)] if append else prior,
                          new if append else None, hkv * G, hkv, rng.choice([1, 2, 4, 8, 64, 256, 304]),
                          rng.choice([3, 3, 1, 2]), rng.choice([16, 1, 2]), rng.choice([64, 128, 3]),
                          q_tile))
    got = forms(driver, lines)
    assert {f["form"] for f in got} == {"none", "units", "halves", "listed", "tiles"}
    assert any(f["singles"] < f["table_singles"] for f in got)


def test_whole_tiles_in_many_waves_have_no_table(driver):
    """Short prompts run as halves of their units: nothing is built or uploaded for them
    beyond the plan's own tables.  Longer ones run as whole units, between them the form that
    is faster: 20 tokens to each of 128 requests, but not prompts of 64-2,048 tokens."""
    prompts = [64 + 61 * i for i in range(32)]
    short, long, few, mixed = forms(driver, [
        line([510] * 80, [510] * 80, 40, 8), line([40960], [40960], 40, 8),
        line([2020] * 128, [20] * 128, 32, 8), line(prompts, prompts, 40, 8)])
    assert few["form"] == "halves" and mixed["form"] == "units"
    assert short["form"] == "halves" and short["workspace"] == short["plain"]
    assert long["form"] == "units" and long["workspace"] == long["plain"]


def test_chunk_tiles_are_not_cut_where_decode_rows_fill_the_chip(driver):
    """Cutting a chunk's keys over all CUs delays the decode rows beside it, so it is done only
    where whole units would outlast them."""
    def form(chunks, tokens, prior, rows, length):
        lens = [prior + tokens] * chunks + [length] * rows
        return line(lens, [tokens] * chunks + [1] * rows, 32, 8)

    cases = [(1, 333, 4000, 0, 0, True), (1, 333, 4000, 16, 1000, True),
             (1, 333, 4000, 127, 1000, False), (1, 333, 16000, 127, 1000, True),
             (1, 333, 16000, 127, 4000, False), (1, 500, 4000, 16, 16000, False),
             (4, 64, 4000, 127, 1000, False), (4, 64, 16000, 16, 16000, True)]
    got = forms(driver, [form(*c[:5]) for c in cases])
    assert [f["parts"] > 1 for f in got] == [c[5] for c in cases]


def test_gpu_cases_take_the_forms_they_are_for(driver):
    """The GPU tests of the launched forms run what they say."""
    import test_gpu_fewer_units as fewer
    import test_gpu_fine_tiles as fine
    import test_gpu_softmax_range as moving

    got = forms(driver, [line(c[0], c[1], *c[2:5]) for c in fine.CASES])
    assert [(f["form"], f["parts"]) for f in got] == [c[5:] for c in fine.CASES]
    longest = [f["pages"] for c, f in zip(fine.CASES, got) if c[0][0] >= 66000]
    assert longest[0] < 4096 < min(longest[1:])        # pages of a workgroup against the staged row
    got = forms(driver, [line(c[0], None, *c[1:4]) for c in fewer.CASES])
    assert [f["singles"] for f in got] == [c[4] for c in fewer.CASES]
    assert [f["singles"] < f["table_singles"] for f in got] == [True] * 7 + [False] * 2
    lens = [p + c for p, c in zip(moving.PRIOR, moving.CHUNK)]
    got = forms(driver, [line(lens, moving.CHUNK, 16, 4, c) for c in (8, 256)])
    assert got[0]["form"] == "units" and got[1]["form"] == "tiles" and got[1]["parts"] > 1
