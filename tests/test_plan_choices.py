"""What a call's plan may depend on: pairs that only get an error record do not
move the others' strip width, and a pair is refused for its direction bits
whatever else is in the call."""
import numpy as np
import pytest

from paper_2210_08052_amd import mpg

pytestmark = pytest.mark.gpu


def _run(ctx, prot, dna, segs):
    """Score-only records of segments of one protein and region, and the number
    of wavefronts that ran two pairs' last strips (it follows from the width)."""
    import torch
    d_prot = torch.frombuffer(bytearray(prot), dtype=torch.uint8).cuda()
    d_dna = torch.frombuffer(bytearray(dna), dtype=torch.uint8).cuda()
    arr = np.zeros(len(segs), mpg.SEG_DTYPE)
    for k, (m, n) in enumerate(segs):
        arr["plen"][k], arr["dlen"][k] = m, n
    d_out = torch.zeros(len(segs) * mpg.DEV_RESULT_DTYPE.itemsize, dtype=torch.uint8,
                        device="cuda")
    d_ops = torch.zeros(len(segs), dtype=torch.uint8, device="cuda")
    ctx.timing(reset=True)
    ctx.align_batch_dev(mpg.params(), d_prot.data_ptr(), d_dna.data_ptr(), arr,
                        d_out.data_ptr(), d_ops.data_ptr(), len(segs))
    ctx.sync()
    rec = np.frombuffer(d_out.cpu().numpy().tobytes(), dtype=mpg.DEV_RESULT_DTYPE)
    return rec, ctx.timing(reset=True)["seg_packs"]


@pytest.mark.parametrize("beyond", [(300, mpg.MPG_MAX_DNA + 1), (300, 2**31 - 1),
                                    (mpg.MPG_MAX_PROT + 1, 4000), (-1, 900), (300, -5)])
def test_refused_pairs_do_not_choose_the_width(beyond):
    """3,000 pairs of 300 residues run at width 2 (their last strips fill 23
    lanes and share wavefronts; at width 1 they fill 45 and cannot), whatever
    the lengths of a pair that is refused."""
    rng = np.random.default_rng(5)
    prot = bytes(rng.choice(list(b"ARNDCQEGHILKMFPSTWYV"), 300).astype(np.uint8))
    dna = bytes(rng.choice(list(b"ACGT"), 1000).astype(np.uint8))
    print("case refused pair %s" % (beyond,), flush=True)
    with mpg.Context(0) as ctx:
        ctx.enable_timing(True)
        segs = [(300, 1000)] * 3000
        ref, packs = _run(ctx, prot, dna, segs)
        got, packs2 = _run(ctx, prot, dna, segs + [beyond])
    assert packs > 1000
    assert packs2 == packs
    assert got["status"][-1] == mpg.MPG_E_RANGE
    assert (got["status"][:-1] == 0).all() and (got["score"][:-1] == ref["score"]).all()


@pytest.mark.parametrize("budget,status", [(313343, mpg.MPG_E_RANGE), (313344, 0)])
def test_budget_refusal_does_not_hang_on_the_call(budget, status):
    """A traced pair of 150 residues on 1,000 bases: 17 chunks of 4,608 bytes per
    column, 2 strips of width 2 (313,344 bytes) or 3 of width 1 (235,008).  Its
    refusal goes by width 2, alone (the call's work would choose width 1) and
    among 3,000 others (width 2)."""
    rng = np.random.default_rng(6)
    prot = bytes(rng.choice(list(b"ARNDCQEGHILKMFPSTWYV"), 300).astype(np.uint8))
    dna = bytes(rng.choice(list(b"ACGT"), 1000).astype(np.uint8))
    print("case budget %d" % budget, flush=True)
    with mpg.Context(0, tb_budget_bytes=budget) as ctx:
        one = (prot[:150], dna, True)
        alone = ctx.align_batch([one], mpg.params())
        among = ctx.align_batch([one] + [(prot, dna, False)] * 3000, mpg.params())
    assert alone[0]["status"] == status
    assert among[0] == dict(alone[0], job_id=among[0]["job_id"])
