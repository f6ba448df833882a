"""Which form a column subset takes, asked of the header that decides it (cols_plan_driver.cpp)."""
import os
import shutil
import subprocess

import pytest

import test_gpu_cols_lines
import test_gpu_cols_rounds
import test_gpu_cols_stream

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    """(threads, round, staged, store) for each (element bytes, rows, cols, values, columns asked, output address)."""
    exe = str(tmp_path_factory.mktemp("cols_plan") / "driver")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(ROOT, "paper_2406_11674_amd", "csrc"),
                    "-o", exe, os.path.join(ROOT, "tests", "cols_plan_driver.cpp")], check=True)

    def ask(calls):
        text = "".join(" ".join(str(int(v)) for v in c) + "\n" for c in calls)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=120)
        assert out.returncode == 0, out.stdout
        return [tuple(int(v) for v in line.split()) for line in out.stdout.splitlines()]
    return ask


# bytes, rows, cols, kept, columns asked: calls of which both forms were timed, and what they took, us, a workgroup per row /
# workgroups that stay
FASTER_BY_ROW = [(2, 16384, 16384, 0.5, 1147), (2, 16384, 16384, 0.5, 1638),      # 59 / 65, 62 / 66
                 (2, 6656, 12224, 0.62, 978), (2, 21312, 9920, 0.82, 1220),        # 22.0 / 27.2, 76 / 83
                 (2, 25408, 11840, 0.57, 912), (2, 35137, 9370, 0.78, 759),        # 78 / 86, 107 / 115
                 (2, 5824, 11712, 0.55, 2249), (2, 6016, 6656, 0.65, 2110),        # 22.0 / 25.4, 20.2 / 22.5
                 (2, 9088, 2624, 0.6, 1278), (1, 5718, 11811, 0.87, 1465),         # 18.4 / 22.1, 16.4 / 18.8
                 (2, 21632, 13248, 0.75, 2782), (2, 31040, 9920, 0.3, 1984),       # 106 / 116, 115 / 122
                 (2, 13120, 5120, 0.42, 1280)]                                     # 25.2 / 29.7
FASTER_STAYING = [(2, 8192, 28672, 0.5, 2867), (2, 8192, 28672, 0.5, 5734),        # 63 / 55, 93 / 71
                  (2, 16384, 16384, 0.5, 4915), (1, 36864, 9216, 0.5, 2765),       # 100 / 96, 113 / 87
                  (1, 28672, 8192, 0.5, 2867), (1, 25776, 4887, 0.5, 2443),        # 90 / 67, 76 / 58
                  (2, 6505, 9210, 0.71, 2745), (1, 6469, 12229, 0.88, 1810),       # 25.5 / 22.7, 20.0 / 16.9
                  (2, 16464, 5143, 0.64, 1193), (2, 12538, 3715, 0.79, 1523),      # 45 / 36, 36 / 28
                  (2, 9782, 8261, 0.32, 1239), (2, 6375, 3321, 0.5, 1577),        # 28.7 / 24.6, 19.3 / 17.6
                  (2, 17637, 4565, 0.53, 1233)]                                    # 45.2 / 37.2


def test_the_faster_form_is_taken(forms):
    got = forms([(b, r, c, r * c * keep, n, 0) for b, r, c, keep, n in FASTER_BY_ROW + FASTER_STAYING])
    assert [f[0] != 0 for f in got] == [False] * len(FASTER_BY_ROW) + [True] * len(FASTER_STAYING)


def _all(forms, calls, out=0):
    """The form of each call, the same for whatever its random mask keeps (five standard deviations either way)."""
    rows = [(b, r, c, r * c * keep, 5 * (r * c * keep * (1 - keep)) ** 0.5, n) for b, r, c, keep, n in calls]
    got = [forms([(b, r, c, max(0, min(r * c, nnz + z * spread)), n, out) for b, r, c, nnz, spread, n in rows]) for z in (0, -1, 1)]
    assert got[0] == got[1] == got[2]
    return got[0]


def test_the_calls_of_the_staying_form_take_it(forms):
    t = test_gpu_cols_stream
    calls = [(2 if wide else 1, r, c, keep, n) for r, c, keep, wide, n in t.CASES]
    got = _all(forms, calls)
    assert all(f[0] for f in got)
    assert {(c[0],) + f[:2] for c, f in zip(calls, got)} == {(b, 256, q) for b in (1, 2) for q in (6, 8, 12)} | {
        (b, 512, q) for b in (1, 2) for q in (4, 6, 8, 12)}
    r, c, n = t.NOT_STAGED
    others = [(b, *t.ANY_ORDER) for b in (1, 2)] + [(2, *t.OWN_ENTRY), (2, *t.IN_A_GRAPH), (2, r, c, 0.4, n), (1, r, c, 0.8, n)]
    assert all(f[0] for f in _all(forms, others))


PLAIN, STREAMED, LINES = 0, 1, 2


def test_the_calls_of_a_workgroup_per_row_take_that(forms):
    """Every form with a workgroup for each row that stores are tested for: gathered and staged, plain, streamed, in whole lines."""
    lines = [(2, r, c, keep, n) for r, c, n, keep in test_gpu_cols_lines.CASES]
    got = [f for off in (0, 1, 37, 64) for f in _all(forms, lines, 2 * off)]
    assert not any(f[0] for f in got)
    assert {f[2:] for f in got} >= {(0, STREAMED), (0, LINES), (1, STREAMED), (1, LINES)}
    # short rows staged and in whole lines
    assert _all(forms, [(2, 30000, 3000, 0.8, 1700)], 2 * 37)[0] == (0, 4, 1, LINES) and lines[-1] == (2, 30000, 3000, 0.8, 1700)
    rounds = [(b, r, c, keep, n) for b in (2, 1) for r, c, n, keep in test_gpu_cols_rounds.CASES]
    got = dict(zip(rounds, _all(forms, rounds)))
    assert {f[1:] for c, f in got.items() if f[0] == 0 and c[0] == 2} >= {(3, 0, PLAIN), (4, 0, PLAIN), (6, 0, PLAIN), (4, 0, STREAMED),
                                                                       (4, 1, PLAIN), (4, 1, LINES)}
    for b in (1, 2):  # short rows: gathered, staged, by workgroups that stay
        assert [got[(b,) + c][0::2] for c in ((12000, 2500, 0.8, 1100), (5400, 2000, 0.95, 1700))] == [(0, 0), (0, 1)]
        assert all(got[(b,) + c][0] for c in ((12000, 2500, 0.8, 1500), (12001, 2501, 0.7, 1701)))
