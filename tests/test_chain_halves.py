"""Anchor-driven calls around the size from which they run in two halves, the
second on a stream forked from the context's: results, order on the context's
stream, memory and failures."""
import numpy as np
import pytest

from paper_2210_08052_amd import mpg
from paper_2210_08052_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def chains():
    """2,100 chains, half of them traced, and their results on the host entry."""
    cases = [(p.prot, p.dna, a, 6, k % 2 == 0)
             for k, (p, a) in enumerate(W.chain_jobs(2100, seed=92))]
    with mpg.Context(0) as c:
        return cases, c.align_chains(cases, mpg.params())


class _Call:
    """A call over the first n chains, its buffers on the device."""

    def __init__(self, chains, n):
        import torch
        self.cases, self.ref, self.n = chains[0][:n], chains[1][:n], n
        pb, db, self.segs = mpg.pack_chains(self.cases)
        self.prot = torch.frombuffer(bytearray(pb), dtype=torch.uint8).cuda()
        self.dna = torch.frombuffer(bytearray(db), dtype=torch.uint8).cuda()
        self.cap = self.segs.ops_capacity(mpg.params())
        self.ops = torch.zeros(self.cap, dtype=torch.uint8, device="cuda")
        self.out = torch.zeros(n * mpg.DEV_RESULT_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()

    def run(self, ctx):
        ctx.align_chains_dev(mpg.params(), self.prot.data_ptr(), self.dna.data_ptr(), self.segs,
                             self.out.data_ptr(), self.ops.data_ptr(), self.cap)

    def check(self, out=None, ops=None):
        rec = np.frombuffer((self.out if out is None else out).cpu().numpy().tobytes(),
                            dtype=mpg.DEV_RESULT_DTYPE)
        text = (self.ops if ops is None else ops).cpu().numpy().tobytes()
        for k, (r, c) in enumerate(zip(self.ref, self.cases)):
            got = tuple(rec[f][k] for f in ("status", "score", "g_end", "p_end"))
            assert got == tuple(r[f] for f in ("status", "score", "g_end", "p_end")), k
            if c[4]:
                at = int(rec["ops_off"][k])
                assert text[at:at + int(rec["ops_len"][k])].decode() == r["ops"], k


@pytest.mark.parametrize("n", [511, 512, 513, 1025])
def test_results_around_the_split(chains, n):
    print("case n=%d" % n, flush=True)
    call = _Call(chains, n)
    with mpg.Context(0) as ctx:
        for _ in range(2):
            call.run(ctx)
            ctx.sync()
            call.check()


@pytest.mark.parametrize("n", [511, 600, 2100])
def test_order_on_the_stream(chains, n):
    """The letters arrive by a copy queued on the context's stream just before
    the call, behind other work, and the results leave by a copy queued just
    after it; nothing waits on the host in between."""
    import torch
    print("case stream order n=%d" % n, flush=True)
    call = _Call(chains, n)
    prot, dna = call.prot.clone(), call.dna.clone()
    stream = torch.cuda.Stream()
    a = torch.randn(4096, 4096, device="cuda")
    with mpg.Context(0) as ctx:
        ctx.set_stream(stream.cuda_stream)
        call.run(ctx)  # workspaces are in place: the next call does not wait for them
        torch.cuda.synchronize()
        for _ in range(2):
            call.prot.zero_()
            call.dna.zero_()
            call.out.zero_()
            call.ops.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                for _ in range(20):
                    b = a @ a
                call.prot.copy_(prot)
                call.dna.copy_(dna)
            call.run(ctx)
            with torch.cuda.stream(stream):
                out, ops = call.out.clone(), call.ops.clone()
                call.out.zero_()
                call.ops.zero_()
            stream.synchronize()
            call.check(out, ops)
        del b


class _Pool:
    """Device memory for a context: bytes in use, and refusals on demand."""

    def __init__(self):
        self.live, self.calls, self.refuse = {}, 0, ()

    def alloc(self, n):
        import torch
        self.calls += 1
        if self.calls in self.refuse:
            return 0
        q = torch.cuda.caching_allocator_alloc(n, device=0)
        self.live[q] = n
        return q

    def release(self, q):
        import torch
        del self.live[q]
        torch.cuda.caching_allocator_delete(q)


def _used(chains, n, budget):
    """Bytes of workspace after a call of n chains."""
    pool = _Pool()
    call = _Call(chains, n)
    with mpg.Context(0, tb_budget_bytes=budget) as ctx:
        ctx.set_allocator(pool.alloc, pool.release)
        call.run(ctx)
        ctx.sync()
        used = sum(pool.live.values())
        call.check()
    assert not pool.live
    return used


def test_halves_share_the_budget(chains):
    """2,047 traced chains need more than 192 MiB of direction bits (at the width
    that needs most, by which they are split into waves): raising the budget
    from 96 to 192 MiB adds no more than that to the call's memory."""
    cases = [c[:4] + (True,) for c in chains[0][:2047]]
    with mpg.Context(0) as ctx:
        traced = (cases, ctx.align_chains(cases, mpg.params()))
    small, large = (_used(traced, 2047, b << 20) for b in (96, 192))
    print("case budget %d %d" % (small, large), flush=True)
    assert 32 << 20 < large - small <= 96 << 20


def test_a_chain_beyond_half_the_budget(chains):
    """A chain whose one piece needs most of the budget, among 600: accepted,
    as when it is alone."""
    rng = np.random.default_rng(7)
    prot = bytes(rng.choice(list(b"ARNDCQEGHILKMFPSTWYV"), 1200).astype(np.uint8))
    dna = bytes(rng.choice(list(b"ACGT"), 6000).astype(np.uint8))
    wide = (prot, dna, [(0, 0)], 6, True)
    # 19 strips of width 1 (10 of width 2, 5 of width 4), 95 chunks of 4,608 bytes a column
    budget = int(9.5e6)
    cases = chains[0][:599] + [wide]
    with mpg.Context(0) as ctx:
        ref = ctx.align_chains(cases, mpg.params())
    assert ref[-1]["status"] == 0
    call = _Call((cases, ref), 600)
    print("case wide piece", flush=True)
    with mpg.Context(0, tb_budget_bytes=budget) as ctx:
        call.run(ctx)
        ctx.sync()
        call.check()


@pytest.mark.parametrize("n", [600, 2100])
@pytest.mark.parametrize("half", [0, 1])
def test_a_half_without_memory(chains, n, half):
    """The allocator refuses a block of one half: below 2,048 chains the call
    runs as one batch; above, it fails, and the next call is whole."""
    print("case n=%d half=%d" % (n, half), flush=True)
    call = _Call(chains, n)
    pool = _Pool()
    with mpg.Context(0) as ctx:
        ctx.set_allocator(pool.alloc, pool.release)
        call.run(ctx)
        ctx.sync()
    per_half, rest = divmod(pool.calls, 2)
    assert rest == 0 and per_half >= 5
    pool.calls = 0
    first = half * per_half + 4
    pool.refuse = (first, first + 1)  # a buffer is asked for with room to grow, then without
    with mpg.Context(0) as ctx:
        ctx.set_allocator(pool.alloc, pool.release)
        if n < 2048:
            call.run(ctx)
        else:
            with pytest.raises(RuntimeError):
                call.run(ctx)
            ctx.sync()
            call.run(ctx)
        ctx.sync()
        call.check()
    assert not pool.live


@pytest.mark.parametrize("n", [511, 600, 2100])
def test_timing_counts_overlap_once(chains, n):
    """The device time of the DP kernels, added over calls that run one at a
    time, is less than the calls' own time, also where halves overlap."""
    import time
    call = _Call(chains, n)
    with mpg.Context(0) as ctx:
        call.run(ctx)
        ctx.sync()
        ctx.enable_timing(True)
        ctx.timing(reset=True)
        t0 = time.perf_counter()
        for _ in range(10):
            call.run(ctx)
            ctx.sync()
        wall = (time.perf_counter() - t0) * 1e3
        t = ctx.timing(reset=True)
    print("case timing n=%d wall %.3f dp %.3f prepass %.3f walk %.3f" %
          (n, wall, t["dp_ms"], t["prepass_ms"], t["walk_ms"]), flush=True)
    assert t["dp_spans"] == (10 if n < 512 else 20)
    assert 0.3 * wall < t["dp_ms"] < wall
    assert 0 < t["prepass_ms"] < wall and 0 < t["walk_ms"] < wall
