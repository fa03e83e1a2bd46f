"""GPU: batches large enough for the gather in bursts give the bits of the same arrivals in batches that are not.

The general path (checked against the CPU oracle elsewhere) is reached by handing the arrivals over in pieces, each a
range of sequence numbers and too small for bursts.  Sums are formed in worker order on both, so the mean is
compared bit for bit, and so are bitmap and counters; the norm, a double sum of about 1e7 terms whose order differs,
to 1e-12."""
import pytest

pytestmark = pytest.mark.gpu

SIGMA, ROUND = 1e-3, 5


def _sizes(kind, n, P):
    if kind == "one":
        return [n]
    if kind == "many":                       # more buckets than the on-chip table holds
        return [3 * P + 1] * (n // (3 * P + 1)) + [n % (3 * P + 1) or 1]
    sizes, k = [], 1                         # ragged: 1, 2, 3, 5 ... floats up, last packets of every remainder
    while sum(sizes) + k < n:
        sizes.append(k)
        k = k * 3 // 2 + 1
        if k > n // 7:
            k = 1 + len(sizes) % 9
    return sizes + [n - sum(sizes)]


class _Case:
    def __init__(self, W, P, n, kind, seed, **acc):
        import torch
        import paper_2605_01989_amd as dblp
        from paper_2605_01989_amd import binding
        self.dblp, self.binding, self.torch, self.W, self.P = dblp, binding, torch, W, P
        cnt = _sizes(kind, n, P)
        off = [0]
        for c in cnt:
            off.append(off[-1] + c)
        self.make = lambda: dblp.Aggregator(W, off[-1], P, off[:-1], cnt, **acc)
        self.n, self.gen = off[-1], torch.Generator(device="cuda").manual_seed(seed)
        self.grads = [torch.randn(self.n, generator=self.gen, device="cuda").mul_(SIGMA) for _ in range(W)]
        self.n_pkts = self.make().n_pkts

    def rand(self, *shape):
        return self.torch.rand(*shape, generator=self.gen, device="cuda")

    def batch(self, alive, dup=0.01):
        """Packets of the flagged (worker, seq) pairs at shuffled slots, a share of them arriving twice, as a queue."""
        t = self.torch
        w, seq = t.nonzero(alive, as_tuple=True)
        order = t.randperm(w.numel(), generator=self.gen, device="cuda")
        lst = ((w << 32) | seq)[order].contiguous()
        n = lst.numel()
        ctx = self.make()
        packets = t.empty(n * ctx.stride, dtype=t.uint8, device="cuda")
        src = t.empty(n, dtype=t.int16, device="cuda")
        ctx.packetize_list(ROUND, self.grads, lst, n, packets, src)
        slots = t.arange(n, device="cuda")
        slots = t.cat([slots, slots[t.randint(0, n, (max(1, int(n * dup)),), generator=self.gen, device="cuda")]])
        slots = slots[t.randperm(slots.numel(), generator=self.gen, device="cuda")]
        return dict(packets=packets, n=n, queue=slots | (src[slots].long() << 32), seq=(lst & 0xFFFFFFFF)[slots])

    def receive(self, batches, pieces, ctx=None, policy=None):
        t = self.torch
        agg = ctx or self.make()
        if policy is not None:
            agg.accumulator_policy(policy)
        agg.profile_enable(1 << self.binding.K_GATHER)
        agg.begin_round(ROUND)
        for b in batches:
            edge = [self.n_pkts * i // pieces for i in range(pieces + 1)]
            for lo, hi in zip(edge[:-1], edge[1:]):
                q = b["queue"] if pieces == 1 else b["queue"][(b["seq"] >= lo) & (b["seq"] < hi)].contiguous()
                if q.numel():
                    agg.apply_arrivals_queue(b["packets"], b["n"], q)
        out, bitmap = t.empty(self.n, device="cuda"), t.empty(agg.W * agg.words_pw, dtype=t.int64, device="cuda")
        agg.get_bitmap(bitmap)
        agg.finalize(out)
        norm = agg.phase_signal()[0]
        agg.profile_read(self.binding.K_GATHER)
        return out, bitmap, agg.get_counters(), norm, agg.profile_bursts()

    def check(self, batches, pieces, policy=None, bursts=1):
        """bursts: how many of the batches are to be gathered in bursts when they come whole."""
        got, ref = self.receive(batches, 1, policy=policy), self.receive(batches, pieces)
        assert (got[4], ref[4]) == (bursts, 0)
        assert self.torch.equal(got[0].view(self.torch.int32), ref[0].view(self.torch.int32))
        assert self.torch.equal(got[1], ref[1])
        assert got[2] == ref[2]
        assert abs(got[3] - ref[3]) <= 1e-12 * ref[3]


# W, P, elements, buckets: packets of up to 128 floats from 48 MB read on; units counted from the packet and from the
# payload; one to five passes, pieces; groups of a multiple of 8 packets, of fewer than 8, of one; bytes read from 150
# and 300 MB, written from 144 and 256 MB on
CASES = [
    (2, 128, 6_800_000, "ragged"), (2, 64, 6_100_003, "many"), (33, 100, 410_001, "ragged"), (64, 127, 420_000, "one"),
    (8, 255, 5_300_001, "ragged"), (8, 256, 4_900_001, "many"), (64, 512, 1_650_000, "ragged"), (8, 768, 6_000_001, "ragged"),
    (8, 1024, 6_000_001, "ragged"), (8, 366, 5_400_007, "ragged"), (64, 366, 1_100_001, "many"), (5, 700, 17_500_001, "ragged"),
    (8, 1000, 5_500_001, "ragged"), (8, 1200, 5_500_001, "ragged"), (16, 2243, 8_000_001, "ragged"), (8, 4097, 13_500_003, "ragged"),
    (8, 9000, 5_600_001, "ragged"), (8, 16374, 9_900_001, "one"), (8, 38000, 23_000_001, "one"), (3, 366, 41_000_001, "ragged"),
    (4, 2243, 41_000_001, "ragged"), (2, 1024, 72_000_001, "ragged"),
]


@pytest.mark.parametrize("W,P,n,kind", CASES)
def test_bursts_give_the_bits_of_the_general_path(W, P, n, kind):
    """Random loss, runs of packets that nobody delivered, duplicates; then what was lost, as a retransmission."""
    c = _Case(W, P, n, kind, seed=W * 1000 + P)
    alive = c.rand(W, c.n_pkts) >= 0.04
    for at in (0.1, 0.5, 0.93):
        alive[:, int(c.n_pkts * at):int(c.n_pkts * at) + 1 + c.n_pkts // 200] = False
    alive[:, -1] = False
    first = c.batch(alive)
    c.check([first], 12)
    late = ~alive & (c.rand(W, c.n_pkts) < 0.5)
    c.check([first, c.batch(late)], 12)


@pytest.mark.parametrize("copies", [1, 2])
@pytest.mark.parametrize("W,P,n,kind", [(4, 128, 11_000_000, "ragged"), (16, 256, 8_800_001, "ragged"), (16, 1200, 13_000_001, "ragged"),
                                        (16, 9000, 15_000_001, "ragged"), (8, 128, 51_000_001, "ragged")])
def test_bursts_add_to_spans_of_an_earlier_batch(W, P, n, kind, copies):
    """Half of the workers in one batch, the others in the next: spans are opened, updated, and, with two accumulator
    copies that take turns, updated in the copy they are in."""
    from paper_2605_01989_amd import binding
    acc = dict(accumulator_mode=binding.ACCMODE_PAIR) if copies == 2 else {}
    c = _Case(W, P, n, kind, seed=W + P, **acc)
    alive = c.rand(W, c.n_pkts) >= 0.3
    alive[: W // 2, c.n_pkts // 3: c.n_pkts // 2] = False
    a, b = alive.clone(), alive.clone()
    a[W // 2:] = False
    b[: W // 2] = False
    b[0] |= c.rand(c.n_pkts) < 0.5            # copies of what is there already
    c.check([c.batch(a), c.batch(b)], 16, policy=binding.ACC_ALTERNATE if copies == 2 else None,
            bursts=0 if W == 4 else 2)            # (of four workers two at a time are too few)


@pytest.mark.parametrize("spread", [False, True])
def test_launches_that_decide_on_the_device(spread):
    """A batch of 256 MB and less than an eighth of the round: a contiguous step goes in bursts, one spread over the
    round does not; both give the bits of the general path."""
    W, P = 16, 366
    c = _Case(W, P, 34_000_000, "ragged", seed=3)
    alive = c.torch.zeros(W, c.n_pkts, dtype=c.torch.bool, device="cuda")
    if spread:
        alive |= c.rand(W, c.n_pkts) < 0.12
    else:
        alive[:, c.n_pkts // 3 + 5: c.n_pkts // 3 + 5 + int(c.n_pkts * 0.124)] = True
        alive &= c.rand(W, c.n_pkts) >= 0.03
    c.check([c.batch(alive, dup=0.0)], 3 if spread else 40, bursts=0 if spread else 1)


def test_a_later_context_with_smaller_groups_leaves_an_earlier_one_its_own():
    """Two rounds whose bursts are the same kernel with images of different sizes; the smaller context is made second."""
    W, P = 8, 366
    c = _Case(W, P, 25_000_001, "ragged", seed=8)
    first = c.batch(c.rand(W, c.n_pkts) >= 0.02)
    ctx = c.make()
    small = _Case(W, P, 5_400_007, "ragged", seed=9)
    got, ref = c.receive([first], 1, ctx=ctx), c.receive([first], 40)
    small.check([small.batch(small.rand(W, small.n_pkts) >= 0.02)], 12)
    assert c.torch.equal(got[0].view(c.torch.int32), ref[0].view(c.torch.int32))
    assert c.torch.equal(got[1], ref[1]) and got[2] == ref[2] and (got[4], ref[4]) == (1, 0)


# (workers, floats, elements, share of the round) of thin batches over the round, of a share at which bursts pay, and at which
# they do not; more and fewer than seven turns, packets of one KB and in pieces; 256 MB and more, where the blocks decide,
# and less, where the number of arrivals does
@pytest.mark.parametrize("W,P,n,share,bursts", [(2, 366, 100_000_000, 0.5, 0), (2, 366, 150_000_000, 0.9, 1), (8, 366, 50_000_000, 0.16, 0),
                                                (8, 366, 80_000_000, 0.3, 1), (8, 128, 60_000_000, 0.15, 0), (8, 128, 60_000_000, 0.3, 1),
                                                (8, 366, 25_600_000, 0.25, 0), (8, 366, 25_600_000, 0.5, 1), (8, 2243, 120_000_000, 0.16, 1),
                                                (5, 700, 40_000_000, 0.6, 0)])
def test_thin_batches(W, P, n, share, bursts):
    c = _Case(W, P, n, "ragged", seed=W + n)
    c.check([c.batch(c.rand(W, c.n_pkts) < share, dup=0.001)], 30, bursts=bursts)


@pytest.mark.parametrize("share,bursts", [(0.03, 0), (0.98, 1)])
@pytest.mark.parametrize("W,P,n", [(8, 366, 30_000_001), (16, 1024, 20_000_001)])
def test_masked_batches(W, P, n, share, bursts):
    """The whole buffer with a mask: the number of slots says nothing of what is alive.  Against the same packets as a queue, in pieces."""
    c = _Case(W, P, n, "ragged", seed=n)
    t = c.torch
    b = c.batch(t.ones(W, c.n_pkts, dtype=t.bool, device="cuda"), dup=0.0)
    slot, worker = b["queue"] & 0xFFFFFFFF, b["queue"] >> 32
    alive = c.rand(b["n"]) < share                      # by slot
    src = t.empty(b["n"], dtype=t.int16, device="cuda")
    src[slot] = worker.to(t.int16)
    bits = t.zeros(-(-b["n"] // 64) * 64, dtype=t.uint8, device="cuda")
    bits[:b["n"]] = alive
    words = (bits.view(-1, 8) * t.tensor([1, 2, 4, 8, 16, 32, 64, 128], dtype=t.uint8, device="cuda")).sum(1, dtype=t.uint8).view(t.int64)
    agg = c.make()
    agg.profile_enable(1 << c.binding.K_GATHER)
    agg.begin_round(ROUND)
    agg.apply_arrivals(b["packets"], src, b["n"], words, slot.int())
    out = t.empty(c.n, device="cuda")
    agg.finalize(out)
    norm = agg.phase_signal()[0]
    agg.profile_read(c.binding.K_GATHER)
    keep = alive[slot]
    ref = c.receive([dict(b, queue=b["queue"][keep].contiguous(), seq=b["seq"][keep])], 30)
    assert (agg.profile_bursts(), ref[4]) == (bursts, 0)
    assert t.equal(out.view(t.int32), ref[0].view(t.int32)) and agg.get_counters() == ref[2]
    assert abs(norm - ref[3]) <= 1e-12 * ref[3]
