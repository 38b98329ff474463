"""The launch plan's rules, on both sides of each line (CPU only): api.cpp
built for the host, with the stand-ins of tests/host_fuzz for the launches."""

import json
import os
import subprocess

import pytest

from paper_2609_03430_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_03430_amd", "csrc")
FUZZ = os.path.join(ROOT, "tests", "host_fuzz")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CHRON, PAGED = B.RA_LAYOUT_CHRONOLOGICAL, B.RA_LAYOUT_PAGED

pytestmark = pytest.mark.skipif(
    not (os.path.exists(HIPCC) and os.path.isdir(FUZZ)), reason="hipcc or the stand-ins missing")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan_rules")
    objs = []
    for src in (os.path.join(CSRC, "api.cpp"), os.path.join(FUZZ, "stub_launchers.cpp"),
                os.path.join(FUZZ, "plan_rules.cpp")):
        objs.append(str(d / (os.path.basename(src) + ".o")))
        subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17",
                        "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-c", src, "-o",
                        objs[-1]], check=True, capture_output=True)
    exe = str(d / "plan_rules")
    subprocess.run(["g++", "-no-pie"] + objs + ["-o", exe], check=True, capture_output=True)

    def launches(lens, dtype=B.RA_BF16, layout=CHRON, q_heads=40, kv_heads=8, budget=64, recent=64,
                 every=64, forward=0, steps=1):
        args = [dtype, layout, q_heads, kv_heads, budget, recent, every, forward, steps] + lens
        r = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True,
                           timeout=60)
        assert r.returncode == 0, r.stderr
        return [json.loads(line) for line in r.stdout.splitlines()]
    return launches


def _ragged(n, mean, longest):
    """n caches of about the mean length, one of them the longest."""
    short = (mean * n - longest) // (n - 1)
    return [short] * (n - 1) + [longest]


@pytest.mark.parametrize("n,mean,longest,layout,wide", [
    (33, 1000, 4000, CHRON, 0), (33, 2080, 4000, CHRON, 0), (33, 3200, 9000, CHRON, 0),
    (33, 2570, 4000, CHRON, 1), (33, 5200, 9000, CHRON, 1), (33, 2570, 4000, PAGED, 0),
    (64, 1600, 9000, CHRON, 0), (64, 1530, 4000, CHRON, 0), (48, 3020, 4200, CHRON, 1), (64, 3010, 4200, CHRON, 0),
    (80, 940, 4000, CHRON, 0), (80, 1530, 4000, CHRON, 1), (80, 3070, 9000, CHRON, 1),
    (80, 1590, 9000, CHRON, 0), (95, 1530, 4000, PAGED, 0),
])
def test_wide_registers_by_mean_and_longest(plans, n, mean, longest, layout, wide):
    """One long prompt among short caches does not take the build for one
    wavefront per SIMD, which reads it more slowly."""
    a = plans(_ragged(n, mean, longest), layout=layout)[0]
    assert (a["waves"], a["splits"], a["wide"]) == (4, 1, wide)


@pytest.mark.parametrize("n,kv_heads,layout,splits", [
    (33, 8, CHRON, 2), (48, 8, CHRON, 2), (38, 10, PAGED, 2),
    (39, 10, CHRON, 1), (49, 8, CHRON, 1), (49, 8, PAGED, 1), (64, 8, CHRON, 1),
])
def test_heads_halved_while_all_items_are_resident(plans, n, kv_heads, layout, splits):
    """Two items per head up to 384 heads: three workgroups fit a CU."""
    a = plans([3200] * n, layout=layout, kv_heads=kv_heads)[0]
    assert (a["waves"], a["splits"], a["wide"]) == (4, splits, 0)


@pytest.mark.parametrize("n,prompt", [(48, 3200), (64, 3200), (33, 2000)])
def test_lockstep_events_leave_their_moves_to_the_next_step(plans, n, prompt):
    """Halved heads defer as whole ones do: the step after an event of every
    sequence moves the rows, one workgroup per head, and the next is halved again."""
    a = plans([prompt] * n, budget=64, recent=16, every=16, forward=95, steps=3)
    assert [x["evicted"] for x in a] == [n, 0, 0]
    assert [x["pending"] for x in a] == [1, 0, 0]
    halves = 2 if n == 48 else 1
    assert [(x["move"], x["splits"]) for x in a] == [(0, halves), (1, 1), (0, halves)]


@pytest.mark.parametrize("dtype,n,kv_heads,prompt,moved,every,layout,chunks", [
    # (moved: the candidates and recent rows of the event)
    # every row in the last-level cache
    (B.RA_BF16, 1, 8, 40, 832, 64, CHRON, 0), (B.RA_BF16, 1, 8, 40, 896, 64, PAGED, 0),
    (B.RA_BF16, 1, 8, 40, 960, 64, CHRON, 2), (B.RA_BF16, 1, 8, 40, 1280, 64, PAGED, 3),
    (B.RA_BF16, 1, 8, 40, 1152, 1, CHRON, 0), (B.RA_BF16, 1, 8, 40, 1153, 1, CHRON, 3),
    (B.RA_BF16, 4, 8, 40, 9000, 1, PAGED, 18), (B.RA_BF16, 12, 8, 40, 960, 64, CHRON, 2),
    (B.RA_BF16, 12, 8, 40, 1280, 64, CHRON, 0), (B.RA_BF16, 15, 8, 40, 3000, 1, PAGED, 0),
    (B.RA_BF16, 1, 8, 40, 10745, 1, CHRON, 21), (B.RA_BF16, 1, 8, 40, 10746, 1, CHRON, 0),
    (B.RA_F32, 1, 8, 40, 448, 1, CHRON, 0), (B.RA_F32, 1, 8, 40, 449, 1, PAGED, 2),
    (B.RA_F32, 12, 8, 40, 546, 1, CHRON, 0), (B.RA_F32, 15, 8, 40, 1050, 1, CHRON, 0),
    (B.RA_F32, 15, 8, 40, 1300, 1, CHRON, 6), (B.RA_F32, 16, 8, 40, 1300, 1, CHRON, 0),
    # more rows than it holds
    (B.RA_BF16, 8, 8, 6000, 768, 1, CHRON, 0), (B.RA_BF16, 8, 8, 6000, 769, 1, CHRON, 2),
    (B.RA_BF16, 12, 8, 6000, 1018, 1, PAGED, 0), (B.RA_BF16, 15, 8, 6000, 1529, 1, CHRON, 0),
    (B.RA_BF16, 15, 8, 6000, 1530, 1, CHRON, 4), (B.RA_BF16, 16, 8, 6000, 1530, 1, PAGED, 0),
    (B.RA_F32, 15, 8, 6000, 761, 1, CHRON, 0), (B.RA_F32, 15, 8, 6000, 762, 1, CHRON, 4),
])
def test_events_split_where_the_second_launch_pays(plans, dtype, n, kv_heads, prompt, moved, every,
                                                   layout, chunks):
    """The moves of an event get workgroups of their own where the rows past the
    first chunk pay for a second launch, and past 64 heads only while all of them
    run at once or the moves are long."""
    a = plans([prompt] * n, dtype=dtype, layout=layout, kv_heads=kv_heads,
              budget=moved - 16 - every, recent=16, every=every, forward=moved - 1)[0]
    assert a["evicted"] == n and a["len"] == prompt + moved - every
    assert a["chunks"] == chunks


@pytest.mark.parametrize("n,keys,waves,splits", [
    (65, 64, 1, 1), (65, 65, 4, 1), (64, 64, 4, 1), (300, 31, 1, 1),
])
def test_many_fp32_heads_of_few_keys_take_one_wavefront(plans, n, keys, waves, splits):
    a = plans([keys - 1] * n, dtype=B.RA_F32)[0]
    assert (a["waves"], a["splits"]) == (waves, splits)
