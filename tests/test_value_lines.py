"""Both sides of each line between the forms of the DP kernels' values: the last
length, penalty and depth that the exact fp32 form admits and the first beyond
it, against the oracle (whole numbers: equality).  The lines, with t = 16 with
traceback and 1 without: t * (largest score * (m + 1) + 2) below 2^23 (LOCAL)
or 2^22; t * 4 * largest penalty below 2^22 (LOCAL) or 2^21; and, without a
floor, t * the lowest value below 2^22."""
import numpy as np
import pytest

from oracle import params as oparams
from paper_2210_08052_amd import mpg
from tests._cases import compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with mpg.Context(0) as c:
        yield c


def _both(mode, flags=0, **kw):
    return (mpg.params(mode=mode, flags=flags, **kw),
            oparams.default_scoring(mode=mode, flags=flags, **kw))


@pytest.mark.parametrize("mode,m", [(0, 4127), (0, 4128), (1, 2063), (1, 2064), (2, 2063),
                                    (2, 2064), (3, 2063), (3, 2064)])
def test_largest_score(ctx, mode, m):
    """W^m against (TGG)^m with W:W = 127 reaches 127 m; traced, the last and the
    first beyond."""
    mat = np.full((24, 24), -5, np.int8)
    mat[17, 17] = 127
    g, o = _both(mode, mat=mat)
    left = b"" if mode in (1, 2) else b"ACGTTACA"
    right = b"" if mode in (2, 3) else b"ACGTTACA"
    print("case mode=%d m=%d" % (mode, m), flush=True)
    got = compare(ctx, [(b"W" * m, left + b"TGG" * m + right)], g, o, True,
                  label="largest m%d %d" % (mode, m))
    assert got[0]["score"] == 127 * m


@pytest.mark.parametrize("tb", [False, True])
@pytest.mark.parametrize("mode", [0, 1, 2, 3])
def test_largest_penalty(ctx, mode, tb):
    """A gap opening, then a frameshift, at the largest penalty and one more,
    where the gap or the shift must be taken (GLOBAL) or is offered; short
    sequences, since the score bound caps length times penalty."""
    line = (1 << 22 if mode == 0 else 1 << 21) // (4 * (16 if tb else 1))
    if mode in (1, 2) and 30 * line >= 1 << 24:
        line = ((1 << 24) - 1) // 30  # beyond the score bound: the largest that is accepted
    prot = b"MKWL"
    for top in (line - 1, line):
        for kw in (dict(q=top - 1, e=1, f=23), dict(q=11, e=1, f=top)):
            print("case mode=%d tb=%d penalties %s" % (mode, tb, kw), flush=True)
            g, o = _both(mode, **kw)
            pairs = [(prot, b"ATGAAATGGTTA"), (prot, b"ATGAAATGG"), (prot, b"ATGAAATGGATTA"),
                     (prot, b"ATGAAACCCTGGTTA"), (b"MW", b"ATGATGG")]
            compare(ctx, pairs, g, o, tb, label="penalty m%d %d" % (mode, top))


def _lowest(n, m, q, e, f, introns):
    """The depth below which no value of the modes without a floor lies, as the
    planner bounds it: the largest penalties of the default splice tables are
    30 each, a partial sum stays within 256."""
    intron = 0 + 30 + 30  # r = 0
    cell = (intron + q + e + e * (m + 1) if introns
            else f + 2 * (q + e) + e * ((n + 2) // 3 + m + 1))
    return cell + max(intron, q + e + e) + f + 256


@pytest.mark.parametrize("tb,flags,m,n,e", [(True, 3, 1400, None, 60), (True, 0, None, 3, 60),
                                            (False, 3, 100, None, 1000),
                                            (False, 0, None, 3, 400)])
@pytest.mark.parametrize("mode", [2, 1])
def test_lowest_value(ctx, mode, tb, flags, m, n, e):
    """End to end over sequences that share nothing: gaps all the way, as deep as
    the last size that the fp32 form admits, and one unit deeper."""
    q, f = 1, 0 if flags == 3 else 23
    mat = np.full((24, 24), -128, np.int8)
    line = (1 << 22) // (16 if tb else 1)
    g, o = _both(mode, flags, q=q, e=e, f=f, r=0, mat=mat)
    size = 1
    while _lowest(*((n, size) if m is None else (3 * size, m)), q, e, f, flags == 0) < line:
        size += 1
    for k in (size - 1, size):
        mm, nn = (k, n) if m is None else (m, 3 * k)
        assert (nn + mm + 4) * max(q + e, 128) < 1 << 24
        print("case mode=%d tb=%d flags=%d m=%d n=%d" % (mode, tb, flags, mm, nn), flush=True)
        got = compare(ctx, [(b"W" * mm, b"A" * nn)], g, o, tb, label="lowest %d %d" % (mm, nn))
        if mode == 2 and flags == 3 and tb:
            assert got[0]["score"] == -2 * q - e * (mm + nn // 3)
