"""GPU: batches of few packets, which are gathered by a list of what arrived.

Every batch is restated in float32 with plain torch, in the order that the library documents: the workers' floats in worker
order onto zero, times 1 / W (W a power of two), onto what the span held.  The same additions give the same bits."""
import pytest

pytestmark = pytest.mark.gpu

ROUND = 9


class _Rx:
    def __init__(self, W, P, sizes, seed):
        import torch
        import paper_2605_01989_amd as dblp
        off = [sum(sizes[:i]) for i in range(len(sizes))]
        self.W, self.P, self.n = W, P, sum(sizes)
        self.agg = agg = dblp.Aggregator(W, self.n, P, off, sizes)
        self.gen = torch.Generator(device="cuda").manual_seed(seed)
        self.grads = [torch.randn(self.n, generator=self.gen, device="cuda") for _ in range(W)]
        lens = []
        for c in sizes:
            lens += [P] * (-(-c // P) - 1) + [c - (-(-c // P) - 1) * P]
        self.pkts = len(lens)
        assert self.pkts == agg.n_pkts
        self.packet = torch.repeat_interleave(torch.arange(self.pkts, device="cuda"), torch.tensor(lens, device="cuda"))
        self.got = torch.zeros(W, self.pkts, dtype=torch.bool, device="cuda")
        self.sum = torch.zeros(self.n, device="cuda")
        self.counts = dict(accepted=0, duplicate=0, stale=0, invalid=0)
        self.scale = 1.0 / W if W & (W - 1) == 0 else 1.0
        agg.begin_round(ROUND)

    def deliver(self, w, seq, queue, stale=False, broken=0):
        """Packets (w[i], seq[i]) in this order; a packet that occurs twice has two copies in the buffer, of different contents."""
        import torch
        agg, m = self.agg, w.numel()
        packets = torch.empty(m * agg.stride, dtype=torch.uint8, device="cuda")
        src = torch.empty(m, dtype=torch.int16, device="cuda")
        agg.packetize_list(ROUND + stale, self.grads, ((w << 32) | seq).contiguous(), m, packets, src)
        if broken:          # the length says one float less: invalid
            packets.view(m, -1)[:broken, 6:8].view(torch.int16).sub_(1)
        slots = torch.arange(m, device="cuda")
        # later copies of a packet of this batch are made to differ: they must not be looked at
        key = (w * self.pkts + seq)
        first = torch.full((self.W * self.pkts,), m, dtype=torch.int64, device="cuda").scatter_reduce_(0, key[broken:], slots[broken:], "amin")
        is_first = first[key] == slots
        later = ~is_first
        if broken:
            later[:broken] = False
        packets.view(m, -1)[later, 8:] = 0x41
        if queue:
            agg.apply_arrivals_queue(packets, m, (slots | (w << 32)).contiguous())
        else:
            agg.apply_arrivals(packets, src, m)
        if stale:
            self.counts["stale"] += m
            return
        flags = torch.zeros_like(self.got)
        flags[w[broken:], seq[broken:]] = True
        fresh = flags & ~self.got
        self.counts["accepted"] += int(fresh.sum())
        self.counts["duplicate"] += m - broken - int(fresh.sum())
        self.counts["invalid"] += broken
        a = torch.zeros(self.n, device="cuda")
        for i in range(self.W):
            a = a + torch.where(fresh[i][self.packet], self.grads[i], 0.0)
        a = a * self.scale
        had, new = self.got.any(0)[self.packet], fresh.any(0)[self.packet]
        self.sum = torch.where(new, torch.where(had, self.sum + a, a), self.sum)
        self.got |= flags

    def check(self):
        import torch
        agg = self.agg
        out = torch.empty(self.n, device="cuda")
        agg.finalize(out)
        want = self.sum if self.scale != 1.0 or self.W == 1 else self.sum / torch.full_like(self.sum, self.W)      # (a scalar divisor would be a multiplication)
        want = torch.where(self.got.any(0)[self.packet], want, 0.0)
        assert torch.equal(out.view(torch.int32), want.view(torch.int32))
        norm = float(want.double().square().sum().sqrt())
        # in double while spans are stored and updated, or (W no power of two) squares of float32 summed four at a time
        limit = (4.5 * self.n * 2.0 ** -53 if self.scale != 1.0 or self.W == 1 else 2 * 2.0 ** -24) * norm
        assert abs(agg.phase_signal()[0] - norm) <= limit
        assert agg.get_counters() == self.counts
        words = torch.empty(self.W * agg.words_pw, dtype=torch.int64, device="cuda")
        agg.get_bitmap(words)
        bits = ((words.view(self.W, -1, 1) >> torch.arange(64, device="cuda")) & 1).bool().view(self.W, -1)
        assert torch.equal(bits[:, :self.pkts], self.got) and not bool(bits[:, self.pkts:].any())


# one packet length for each instance: pieces of 1 to 4 KB counted from the payload and from the packet, packets of two
# pieces, packets that a block takes together; 16 waves where packets are heavy and few
SHAPES = [(1, 256, 9000), (3, 255, 40_000), (8, 200, 9000), (2, 512, 6000), (8, 366, 30_000), (5, 768, 3000), (4, 700, 3000), (16, 1024, 5000), (4, 1000, 2500),
          (4, 1200, 2000), (17, 366, 3000), (24, 200, 6000), (3, 1800, 1500), (2, 2243, 2400), (4, 16374, 240), (64, 366, 4000), (40, 1200, 200), (64, 300, 9000)]


@pytest.mark.parametrize("W,P,pkts", SHAPES)
@pytest.mark.parametrize("queue", [False, True])
def test_few_packets(W, P, pkts, queue):
    import torch
    # short buckets at both ends and in the middle, so that short packets of every remainder occur
    sizes = [1, 2, 3, 4, 5, P, P + 1, 2 * P + 2, (pkts // 2) * P + 3, P + 7, 6, (pkts // 2 - 30) * P - 1] + [P - 1] * 8 + [min(P, 7), 1]
    rx = _Rx(W, P, sizes, W * P)
    gen, n = rx.gen, rx.pkts
    def pick(m):
        return torch.randint(0, W, (m,), generator=gen, device="cuda"), torch.randint(0, n, (m,), generator=gen, device="cuda")
    some = torch.rand(W, n, generator=gen, device="cuda") < 0.6        # most spans have contents, some have none
    some[:, n // 4:n // 4 + n // 8] = False
    w, seq = torch.nonzero(some, as_tuple=True)
    order = torch.randperm(w.numel(), generator=gen, device="cuda")
    rx.deliver(w[order], seq[order], queue)
    rx.check()
    most = max(4, n // 4)
    for m in (1, 3, min(64, most), min(most, 384 * W, 1536), min(most, 1537 if W > 4 else 384 * W + 1), most, n // 2):      # (the last by groups)
        w, seq = pick(m)
        if m > 8:                                   # copies in the batch, one number from all workers, both ends
            w[1], seq[1] = w[0], seq[0]
            seq[m // 2:m // 2 + min(W, m // 4)] = n // 4 + 1
            w[m // 2:m // 2 + min(W, m // 4)] = torch.arange(min(W, m // 4), device="cuda")
            seq[2], seq[3] = 0, n - 1
        rx.deliver(w, seq, queue, broken=m // 9)
        rx.check()
    rx.deliver(*pick(5), queue, stale=True)         # nothing of this round
    rx.check()
    # dense: what is left of a window, all workers, in numbers that the list is made for; then all the rest
    for width in (1, max(2, most // W // 2), max(3, most // W)):
        lo = n // 4 + (3 if width < n // 9 else 0)
        w, seq = torch.nonzero(~rx.got[:, lo:lo + width], as_tuple=True)
        if w.numel():
            rx.deliver(w, seq + lo, queue)
            rx.check()
    w, seq = torch.nonzero(~rx.got, as_tuple=True)
    rx.deliver(w, seq, queue)
    rx.check()


def test_few_packets_in_a_recorded_round():
    """A small batch after a large one, recorded and told again: the list and its owners start over each time."""
    import torch
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        rx = _Rx(4, 366, [3_000_000], 5)
        agg, n = rx.agg, rx.pkts
        late = torch.rand(4, n, generator=rx.gen, device="cuda") < 0.01
        m = 4 * n
        packets = torch.empty(m * agg.stride, dtype=torch.uint8, device="cuda")
        src = torch.empty(m, dtype=torch.int16, device="cuda")
        for w in range(4):
            agg.packetize(w, ROUND, rx.grads[w], 0, 0, n, packets, src, slot_base=w * n)
        first, second = (torch.nonzero(f.reshape(-1)).flatten().int() for f in (~late, late))
        out = torch.empty(rx.n, device="cuda")

        def receive():
            agg.begin_round(ROUND)
            agg.apply_arrivals(packets, src, m, None, first)
            agg.apply_arrivals(packets, src, m, None, second)
            agg.finalize(out)
        receive()
        want, norm, counts = out.clone(), agg.phase_signal()[0], agg.get_counters()
        assert counts["accepted"] == m
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            receive()
        for _ in range(3):
            out.fill_(7.0)
            side.synchronize()
            graph.replay()
            assert agg.phase_signal()[0] == norm and agg.get_counters() == counts
            assert torch.equal(out.view(torch.int32), want.view(torch.int32))


def _apply_in_turn(rx, packets, batches):
    """A round of the given batches of (worker, number) pairs: the mean's bits and the norm."""
    import torch
    agg = rx.agg
    agg.begin_round(ROUND)
    for w, seq in batches:
        agg.apply_arrivals_queue(packets, rx.W * rx.pkts, ((w * rx.pkts + seq) | (w << 32)).contiguous())
    out = torch.empty(rx.n, device="cuda")
    agg.finalize(out)
    return out, agg.phase_signal()[0]


def _all_packets(rx):
    import torch
    agg = rx.agg
    packets = torch.empty(rx.W * rx.pkts * agg.stride, dtype=torch.uint8, device="cuda")
    src = torch.empty(rx.W * rx.pkts, dtype=torch.int16, device="cuda")
    for w in range(rx.W):
        agg.packetize(w, ROUND, rx.grads[w], 0, 0, rx.pkts, packets, src, slot_base=w * rx.pkts)
    return packets


# batches that a launch of their own takes, and larger ones; packets of a wave and of a block, blocks of 16 waves; many workers
@pytest.mark.parametrize("W,P,pkts,m", [(1, 256, 9000, 1400), (4, 366, 30_000, 1500), (4, 366, 30_000, 6000), (16, 64, 40_000, 10_000), (2, 2243, 6000, 700),
                                        (2, 2243, 9000, 2000), (4, 16374, 1200, 250), (32, 366, 12_000, 3000), (64, 1200, 240, 60)])
def test_order_of_arrival_changes_no_bit(W, P, pkts, m):
    """The mean and the norm, of a small batch onto a large one and of small batches alone, in several orders."""
    import torch
    rx = _Rx(W, P, [(pkts // 2) * P + 1, (pkts // 2 - 1) * P], W + m)
    gen, n = rx.gen, rx.pkts
    for wide in (False, True):
        if wide:            # packets of very different size, whose squares' last bits get lost one way or another
            size = torch.exp2(torch.randint(-20, 20, (n,), generator=gen, device="cuda").float())[rx.packet]
            rx.grads = [g * size for g in rx.grads]
        packets = _all_packets(rx)
        late = torch.zeros(W * n, dtype=torch.bool, device="cuda")
        late[torch.randperm(W * n, generator=gen, device="cuda")[:m]] = True
        late = late.view(W, n)
        first, (w, seq) = torch.nonzero(~late, as_tuple=True), torch.nonzero(late, as_tuple=True)
        for before in ([first], [], [(w[:m // 2], seq[:m // 2])]):
            rest = (w, seq) if not before or before[0] is first else (w[m // 2:], seq[m // 2:])
            k = rest[0].numel()
            want = None
            for order in (torch.arange(k, device="cuda"), torch.arange(k - 1, -1, -1, device="cuda"), *(torch.randperm(k, generator=gen, device="cuda") for _ in range(3))):
                out, norm = _apply_in_turn(rx, packets, before + [(rest[0][order], rest[1][order])])
                if want is None:
                    want = out, norm
                    exact = float(out.double().square().sum().sqrt())
                    # sums in double while the spans are stored, or (W no power of two, not here) in the copy
                    assert abs(norm - exact) <= 4.5 * rx.n * 2.0 ** -53 * exact
                assert torch.equal(out.view(torch.int32), want[0].view(torch.int32))
                assert norm == want[1]


@pytest.mark.parametrize("m", [300, 3000])
def test_norm_of_the_smallest_and_largest_floats(m):
    """A batch of few packets alone, of the smallest floats that there are to the largest; then with infinities and NaN."""
    import torch
    P, n = 200, 20_000
    rx = _Rx(1, P, [P * n], m)
    seq = torch.randperm(n, generator=rx.gen, device="cuda")[:m]
    w = torch.zeros_like(seq)
    plain = rx.grads[0]
    for scale in (2.0 ** -149, 2.0 ** -140, 2.0 ** -75, 1.0, 2.0 ** 100):
        rx.grads = [(plain * scale if scale > 2.0 ** -149 else plain.sign() * 2.0 ** -149)]
        out, norm = _apply_in_turn(rx, _all_packets(rx), [(w, seq)])
        exact = float(out.double().square().sum().sqrt())
        assert exact > 0 and abs(norm - exact) <= 4.5 * rx.n * 2.0 ** -53 * exact
    at = int(seq[m // 2]) * P + 3
    rx.grads = [torch.full_like(plain, -3.4028234663852886e38)]
    out, norm = _apply_in_turn(rx, _all_packets(rx), [(w, seq)])
    exact = 3.4028234663852886e38 * (m * P) ** 0.5
    assert abs(norm - exact) <= 4.5 * rx.n * 2.0 ** -53 * exact
    for odd in (float("inf"), float("-inf"), float("nan")):
        rx.grads = [plain.clone()]
        rx.grads[0][at] = odd
        norm = _apply_in_turn(rx, _all_packets(rx), [(w, seq)])[1]
        assert norm != norm if odd != odd else norm == float("inf")
    rx.grads = [plain]                  # and of the next round nothing is left
    out, norm = _apply_in_turn(rx, _all_packets(rx), [(w, seq)])
    exact = float(out.double().square().sum().sqrt())
    assert abs(norm - exact) <= 4.5 * rx.n * 2.0 ** -53 * exact
