"""The strip width of a call that is not tuned, chosen from its own work.  The
rule is host arithmetic in a header of its own, compiled here by itself, and
its picks are compared with the width that was faster when calls of these
shapes were timed at both widths on the device (only shapes where the two
differ by 10% or more)."""
import os
import subprocess

import pytest

from paper_2210_08052_amd import workloads as W

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2210_08052_amd", "csrc")
CUS = 256

# residues, bases, pairs, and for score-only, traced, score-only without
# introns, traced without introns, 16-bit lanes: the faster width (0: within 10%)
SHAPES = [
    (1000, 10000, 1, (1, 1, 1, 1, 1)),
    (500, 20000, 1, (1, 1, 1, 1, 1)),
    (1000, 40000, 8, (1, 1, 1, 1, 1)),
    (300, 12000, 60, (1, 1, 1, 1, 1)),
    (600, 24000, 30, (1, 1, 1, 1, 1)),
    (100, 4000, 1000, (0, 1, 0, 1, 0)),
    (4000, 16000, 8, (0, 1, 0, 0, 0)),
    (2000, 1000, 1, (2, 2, 2, 2, 2)),
    (2000, 3000, 60, (2, 2, 2, 2, 2)),
    (1000, 1200, 250, (2, 2, 2, 2, 2)),
    (2000, 2400, 120, (2, 2, 2, 2, 2)),
    (4000, 4800, 60, (2, 2, 2, 2, 2)),
    (8000, 9600, 30, (2, 2, 2, 2, 2)),
]
# the batch recipe: pairs, the same
BATCHES = [(400, (1, 1, 0, 1, 1)), (1200, (1, 1, 1, 1, 1)), (3000, (2, 0, 2, 0, 0)),
           (6000, (2, 0, 2, 0, 0))]
# traced, introns, 16-bit lanes
KINDS = [(0, 1, 0), (1, 1, 0), (0, 0, 0), (1, 0, 0), (0, 1, 1)]

PROGRAM = r"""
#include <cstdio>
#include "mpg_width.h"
// calls on stdin: traced introns int16 pairs, then n m of each; the width of each call
int main() {
    int tb, introns, i16, pairs, n, m;
    while (scanf("%d %d %d %d", &tb, &introns, &i16, &pairs) == 4) {
        mpg::WidthWork w;
        for (int k = 0; k < pairs; ++k) {
            if (scanf("%d %d", &n, &m) != 2) return 1;
            if (i16) w.add16(n, m);
            else w.add(n, m, tb != 0, introns != 0);
        }
        printf("%d\n", w.width(CUS));
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    d = tmp_path_factory.mktemp("width")
    (d / "width.cpp").write_text(PROGRAM)
    exe = str(d / "width")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-DCUS=%d" % CUS, "-I", CSRC,
                           str(d / "width.cpp"), "-o", exe])

    def run(calls):
        text = "".join("%d %d %d %d\n" % (*kind, len(sizes)) +
                       "".join("%d %d\n" % s for s in sizes) for kind, sizes in calls)
        return [int(x) for x in subprocess.run([exe], input=text, capture_output=True, text=True,
                                               check=True).stdout.split()]
    return run


@pytest.mark.parametrize("kind", range(len(KINDS)))
def test_picks_the_faster_width(pick, kind):
    calls, want, label = [], [], []
    for m, n, pairs, best in SHAPES:
        calls.append((KINDS[kind], [(n, m)] * pairs))
        want.append(best[kind])
        label.append((m, n, pairs))
    sizes = [(len(p.dna), len(p.prot)) for p in W.batch_pairs(3000, seed=5)] * 2
    for pairs, best in BATCHES:
        calls.append((KINDS[kind], sizes[:pairs]))
        want.append(best[kind])
        label.append(pairs)
    wrong = [(s, got, w) for s, got, w in zip(label, pick(calls), want) if w and got != w]
    assert not wrong, wrong
