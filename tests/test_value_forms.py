"""The two forms of the DP kernels' values: exact fp32 numbers where the score
bound proves that they fit, integers beyond.  Pairs that reach the largest
values on both sides of the line, penalties on both sides of it, and the
integer form of ordinary pairs, against the oracle (whole numbers: equality)."""
import numpy as np
import pytest

from oracle import params as oparams
from paper_2210_08052_amd import mpg
from paper_2210_08052_amd import workloads as W
from tests._cases import compare, scorings

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with mpg.Context(0) as c:
        yield c


def _pairs(seed, n, max_prot, max_dna):
    return [(p.prot, p.dna) for p in W.random_pairs(n, seed, max_prot=max_prot, max_dna=max_dna)]


def _both(mode, flags=0, **kw):
    return (mpg.params(mode=mode, flags=flags, **kw),
            oparams.default_scoring(mode=mode, flags=flags, **kw))


@pytest.mark.parametrize("K", [1, 2, 4])
def test_integer_form_of_ordinary_pairs(ctx, K, monkeypatch):
    monkeypatch.setenv("MPG_NO_F32", "1")
    monkeypatch.setenv("MPG_FORCE_K", str(K))
    for mode in range(4):
        for tb in (False, True):
            print("case K=%d mode=%d tb=%d" % (K, mode, tb), flush=True)
            for flags, rs in ((0, None), (1, 910 + mode), (2, 920 + mode), (3, None)):
                g, o = scorings(mode, flags, rand_seed=rs)
                compare(ctx, _pairs(900 + K, 12, 400, 700), g, o, tb,
                        label="int K%d m%d f%d" % (K, mode, flags))


@pytest.mark.parametrize("mode,m", [(0, 4126), (0, 4128), (1, 2062), (1, 2064), (2, 2062),
                                    (2, 2064), (3, 2062), (3, 2064)])
def test_largest_scores_at_the_line(ctx, mode, m):
    """W^m against (TGG)^m with W:W = 127, the largest score a protein of m
    residues can reach: with traceback the last fp32 length and the first
    integer one of the mode."""
    mat = np.full((24, 24), -5, np.int8)
    mat[17, 17] = 127
    g, o = _both(mode, mat=mat)
    pad = b"" if mode == 2 else b"ACGTTACA"
    left = b"" if mode in (1, 2) else pad
    right = b"" if mode in (2, 3) else pad
    pairs = [(b"W" * m, left + b"TGG" * m + right)]
    for tb in (True, False):
        print("case mode=%d m=%d tb=%d" % (mode, m, tb), flush=True)
        got = compare(ctx, pairs, g, o, tb, label="largest m%d %d" % (mode, m))
        assert got[0]["score"] == 127 * m


@pytest.mark.parametrize("tb", [False, True])
def test_penalties_on_both_sides_of_the_line(ctx, tb):
    """Penalties up to the limits of the two forms (traceback holds 16x, so
    its line is 16 times lower), in every mode; gaps long enough to reach the
    lowest values of the modes without a floor."""
    for mode in range(4):
        for q, e, f, r, flags in ((11, 100, 23, 29, 1), (11, 200, 23, 29, 1), (11, 1500, 23, 29, 3),
                                  (8000, 100, 8100, 8000, 0), (20000, 10, 32000, 32000, 0),
                                  (40000, 10, 60000, 60000, 0), (5, 1, 300000, 200000, 0)):
            print("case mode=%d tb=%d q=%d e=%d f=%d r=%d" % (mode, tb, q, e, f, r), flush=True)
            g, o = _both(mode, flags, q=q, e=e, f=f, r=r)
            pairs = _pairs(940 + mode, 6, 300, 1800)
            pairs = [(p, d[:len(d) // 3 * 3]) for p, d in pairs]
            n = max(len(d) for _, d in pairs) + max(len(p) for p, _ in pairs) + 4
            if mode in (1, 2) and n * max(q + e, f, r + 60) >= 1 << 24:
                pairs = [(p[:20], d[:60]) for p, d in pairs]  # within the library's bound
            if mode in (1, 2) and 90 * max(q + e, f, r + 60) >= 1 << 24:
                continue
            compare(ctx, pairs, g, o, tb, label="pen m%d q%d" % (mode, q))


def test_forms_mixed_in_one_call(ctx):
    """One traced call with pairs of both forms, in shapes that may share a
    wavefront's lanes with a pair of their own form only."""
    mat = np.full((24, 24), -5, np.int8)
    mat[17, 17] = 127
    g, o = _both(0, mat=mat)
    pairs = [(b"W" * m, b"ACG" + b"TGG" * 40 + b"A" * (120 + m % 3)) for m in
             (4120, 4126, 4128, 4130, 30, 95, 140)]
    print("case mixed forms", flush=True)
    compare(ctx, pairs, g, o, True, label="mixed forms")


@pytest.mark.parametrize("K16", [1, 2])
def test_int16_forms_at_the_line(ctx, K16, monkeypatch):
    """16-bit lanes: W^m against (TGG)^m at the last length of the three-input
    maximum's form (11 * (m + 1) <= 31,600) and the first beyond it, each in a
    call of its own (a call runs one form), with short and empty partners."""
    monkeypatch.setenv("MPG_FORCE_K16", str(K16))
    g, o = _both(0, flags=0)
    g.flags |= mpg.MPG_ALLOW_I16
    for m in (2871, 2872):
        print("case K16=%d m=%d" % (K16, m), flush=True)
        pairs = [(b"W" * m, b"ACGT" + b"TGG" * m + b"CA"), (b"", b"ACGTA"), (b"MKV", b""),
                 (b"M", b"AC"), (b"MKW", b"ATGAAATGG"), (b"W" * 70, b"TGG" * 70)]
        got = compare(ctx, pairs, g, o, False, label="int16 %d" % m)
        assert got[0]["score"] == 11 * m


@pytest.mark.parametrize("K16", [1, 2])
def test_int16_free_moves(ctx, K16, monkeypatch):
    """16-bit lanes with penalties of 0 (every move but a gap is free) and with
    positive scores for partial codons and stops: nothing may start outside
    the region or before a whole codon."""
    monkeypatch.setenv("MPG_FORCE_K16", str(K16))
    mat = np.full((24, 24), 3, np.int8)
    mat[22, :] = 40
    mat[:, 22] = 40
    zero = np.zeros(125, np.uint8)
    for flags in range(4):
        for kw in (dict(q=0, e=1, f=0, r=0, donor=zero, acceptor=zero),
                   dict(q=1, e=0, f=0, r=0, donor=zero, acceptor=zero, mat=mat),
                   dict(q=3, e=1, f=2, r=1, mat=mat)):
            print("case K16=%d flags=%d q=%d" % (K16, flags, kw["q"]), flush=True)
            g, o = _both(0, flags=flags, **kw)
            g.flags |= mpg.MPG_ALLOW_I16
            compare(ctx, _pairs(960 + flags, 14, 150, 300), g, o, False, label="free")
