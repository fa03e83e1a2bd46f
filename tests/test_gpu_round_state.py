"""GPU: what a round counts in is cleared by the round before, by begin_round, or, where calls were recorded into a graph, by
begin_round alone.  The gradient is the same for all workers, so the mean is gradient * arrivals / W: of small whole
numbers times a float over a power of two, exact but for the roundings of the additions (4 workers: 3 * 2**-24)."""
import pytest

pytestmark = pytest.mark.gpu

ROUND, W = 5, 4


class _Rx:
    def __init__(self, P, n):
        import torch
        import paper_2605_01989_amd as dblp
        self.n, self.P = n, P
        self.agg = agg = dblp.Aggregator(W, n, P, [0, n // 3], [n // 3, n - n // 3])
        self.gen = torch.Generator(device="cuda").manual_seed(n)
        self.grad = torch.randn(n, generator=self.gen, device="cuda")
        self.pkts = agg.n_pkts
        self.packets = torch.empty(W * self.pkts * agg.stride, dtype=torch.uint8, device="cuda")
        self.src = torch.empty(W * self.pkts, dtype=torch.int16, device="cuda")
        for w in range(W):
            agg.packetize(w, ROUND, self.grad, 0, 0, self.pkts, self.packets, self.src, slot_base=w * self.pkts)
        lens = torch.full((self.pkts,), P, dtype=torch.int64, device="cuda")
        first = -(-(n // 3) // P)
        lens[first - 1], lens[-1] = n // 3 - (first - 1) * P, n - n // 3 - (self.pkts - first - 1) * P
        self.lens = lens
        self.out = torch.empty(n, device="cuda")

    def alive(self, share):
        import torch
        return torch.rand(W, self.pkts, generator=self.gen, device="cuda") < share

    def order(self, flags):
        import torch
        return torch.nonzero(flags.reshape(-1)).flatten().int()

    def apply(self, order):
        self.agg.apply_arrivals(self.packets, self.src, W * self.pkts, None, order)

    def check(self, flags, scalars=True):
        got = flags.double().sum(0).repeat_interleave(self.lens)
        want = got * self.grad.double() / W
        assert bool(((self.out.double() - want).abs() <= 3 * 2.0 ** -24 * want.abs()).all())
        if scalars:     # the norm is kept in double while the spans are stored, as many additions as there are elements
            want = float(self.out.double().square().sum().sqrt())
            assert abs(self.agg.phase_signal()[0] - want) <= self.n * 2.0 ** -53 * want
        self.check_counts(flags, scalars)

    def check_counts(self, flags, scalars=True):
        import torch
        agg = self.agg
        assert not scalars or agg.get_counters() == dict(accepted=int(flags.sum()), duplicate=0, stale=0, invalid=0)
        words = torch.empty(W * agg.words_pw, dtype=torch.int64, device="cuda")
        agg.get_bitmap(words)
        bits = (words.view(W, -1, 1) >> torch.arange(64, device="cuda")) & 1
        assert bool((bits.view(W, -1)[:, :self.pkts].bool() == flags).all()) and int(bits.sum()) == int(flags.sum())


@pytest.mark.parametrize("P,n", [(64, 30_011), (366, 9_000_001)])
def test_no_round_sees_the_one_before(P, n):
    rx = _Rx(P, n)
    agg, nobody = rx.agg, rx.alive(-1)
    #  share that arrives, finalizes of the round, begin_rounds that open it
    for share, finalizes, begins in ((0.9, 1, 1), (0.1, 1, 1), (-1, 1, 1), (0.9, 0, 1), (0.02, 2, 1), (0.7, 1, 3), (1.0, 2, 2), (0.5, 0, 1), (-1, 1, 1), (0.3, 1, 1)):
        for _ in range(begins):
            agg.begin_round(ROUND)
        rx.check_counts(nobody)
        flags = rx.alive(share)
        if share > 0:
            rx.apply(rx.order(flags))
        for _ in range(finalizes):
            agg.finalize(rx.out)
        if finalizes:
            rx.check(flags)
        else:
            rx.check_counts(flags)


@pytest.mark.parametrize("what", ["begin and arrivals", "arrivals", "arrivals and finalize"])
def test_part_of_a_round_recorded(what):
    """The rest of each round is made as usual, before the replay and after it; two rounds as usual come before the recording."""
    import torch
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        rx = _Rx(366, 2_000_003)
        agg = rx.agg
        steps = {"begin": lambda: agg.begin_round(ROUND), "arrivals": lambda: rx.apply(order), "finalize": lambda: agg.finalize(rx.out)}
        for share in (0.8, 0.6):
            flags = rx.alive(share)
            order = rx.order(flags)
            for f in steps.values():
                f()
            rx.check(flags)
        recorded = [k for k in steps if k in what]
        flags = rx.alive(0.9)
        order = rx.order(flags)
        if "begin" not in recorded:
            steps["begin"]()
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            for k in recorded:
                steps[k]()
        for rep in range(3):
            rx.out.fill_(7.0)
            for k in steps:
                if k not in recorded:
                    if rep or k != "begin":
                        steps[k]()
                elif k == recorded[0]:
                    side.synchronize()
                    graph.replay()
            rx.check(flags, scalars=what == "begin and arrivals")     # (what the host keeps of a call, it keeps when that is recorded)
