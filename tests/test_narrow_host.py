"""Host check of the narrow form's rule and masks (CPU only).

tests/narrow_check.cpp is compiled against the library's headers, host side only.  It says which
problems the launchers take the form for, and compares the masks of every query of those with its
neighbour lists.
"""
import os
import random
import shutil
import subprocess

import pytest

from tests.test_gpu_parity import HUGE_SCORE_CASES, NARROW_CASES, NARROW_EDGE_CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _line(ext, ks, ds, cs, wt, wg):
    cs = cs or (False,) * len(ext)
    cols = zip(ext, ks, ds, cs, wt, wg)
    return " ".join(map(str, [len(ext)] + [int(x) for col in cols for x in col]))


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    hipcc = shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("no hipcc")
    tmp = tmp_path_factory.mktemp("narrow")
    exe = str(tmp / "narrow_check")
    subprocess.check_call([hipcc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17",
                           "-I", os.path.join(ROOT, "paper_2403_04690_amd", "csrc"),
                           os.path.join(ROOT, "tests", "narrow_check.cpp"), "-o", exe])

    def run_(lines):
        res = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True,
                             timeout=300)
        assert res.returncode == 0, res.stdout[-500:] + res.stderr[-500:]
        out = [tuple(map(int, row.split())) for row in res.stdout.splitlines()[:-1]]
        return out, int(res.stdout.split()[-1])
    return run_


def test_gpu_cases_run_the_form_they_name(run):
    """The cases of the GPU tests of the narrow form are taken by it, the edge cases are not."""
    cases = [(c[0], c[1], c[2], c[3], c[6], c[7]) for c in NARROW_CASES]
    cases += [(c[0], c[1], (1,) * len(c[0]), c[2], c[4], c[5]) for c in HUGE_SCORE_CASES]
    taken, pairs = run([_line(*c) for c in cases])
    assert [t[0] for t in taken] == [1] * len(cases) and pairs > 10000
    edge = [(c[0], c[1], c[2], c[3], c[6], c[7]) for c in NARROW_EDGE_CASES]
    assert [t[0] for t in run([_line(*c) for c in edge])[0]] == [0] * len(edge)


def test_masks_are_the_neighbour_lists(run):
    """Random problems of every two-block tiling the library accepts, in the orders, windows,
    dilations and causal axes it accepts; enough of them are taken."""
    rng = random.Random(7)
    lines = []
    while len(lines) < 4000:
        rank = rng.choice((2, 3))
        wt = [1] * rank
        for _ in range(5):  # 32 queries per wave
            wt[rng.randrange(rank)] *= 2
        wg = [1] * rank
        for _ in range(2):
            wg[rng.randrange(rank)] *= 2
        if wt[-1] * wg[-1] > 16:  # (its halo rows hold more than one block)
            continue
        ds = [rng.choice((1, 1, 2, 3)) for _ in range(rank)]
        hi = 30 if rank == 2 else 14
        ext = [rng.randint(1, hi) * d + rng.randint(0, d - 1) for d in ds]
        ks = [min(rng.randint(1, 9 if a < rank - 1 else 7), e // d)
              for a, (e, d) in enumerate(zip(ext, ds))]
        cs = [rng.random() < 0.3 for _ in range(rank)]
        lines.append(_line(ext, ks, ds, cs, wt, wg))
    out, pairs = run(lines)
    taken = [t for t in out if t[0]]
    assert len(taken) > 300 and len({t[1:] for t in taken}) >= 6 and pairs > 10 ** 6
