"""GPU: batches of about half a round, where the gather stops asking the index pass which range was touched, and batches
of as many arrivals, of which few are valid, or none.

Against plain torch: the mean of at most four addends of a worker each, exact in float64 and rounded once per addition in
float32 (three additions, a scaling by a power of two that is exact): within 3 * 2**-24 of the addends' magnitudes."""
import pytest

pytestmark = pytest.mark.gpu

ROUND = 11


@pytest.mark.parametrize("W,P,n", [(4, 64, 40_000), (4, 366, 2_000_003), (2, 2243, 300_001), (4, 16374, 700_000), (4, 256, 38_000_001)])
@pytest.mark.parametrize("what", ["under half, one end", "half, other end", "half, spread", "no packet of this round"])
def test_half_a_round(W, P, n, what):
    import torch
    import paper_2605_01989_amd as dblp
    agg = dblp.Aggregator(W, n, P, [0, n // 3], [n // 3, n - n // 3])
    gen = torch.Generator(device="cuda").manual_seed(n)
    grads = [torch.randn(n, generator=gen, device="cuda") for _ in range(W)]
    pkts = agg.n_pkts
    half = (pkts + 1) // 2
    alive = torch.zeros(W, pkts, dtype=torch.bool, device="cuda")
    if what == "under half, one end":
        alive[:, :(pkts - 1) // 2] = True
    elif what == "half, other end":
        alive[:, pkts - half:] = True
    elif what == "half, spread":
        alive.flatten()[torch.randperm(W * pkts, generator=gen, device="cuda")[:W * half]] = True
    else:
        alive[:] = True
    agg.begin_round(ROUND)

    def deliver(flags, rnd):
        w, seq = torch.nonzero(flags, as_tuple=True)
        m = w.numel()
        order = torch.randperm(m, generator=gen, device="cuda")
        packets = torch.empty(m * agg.stride, dtype=torch.uint8, device="cuda")
        src = torch.empty(m, dtype=torch.int16, device="cuda")
        agg.packetize_list(rnd, grads, ((w << 32) | seq)[order].contiguous(), m, packets, src)
        agg.apply_arrivals(packets, src, m)

    def mean(flags):
        lens = torch.full((pkts,), P, dtype=torch.int64, device="cuda")
        first = -(-(n // 3) // P)
        lens[first - 1] = n // 3 - (first - 1) * P
        lens[-1] = n - n // 3 - (pkts - first - 1) * P
        got = flags.double().repeat_interleave(lens, dim=1)
        return sum(got[w] * grads[w].double() for w in range(W)) / W, sum(got[w] * grads[w].double().abs() for w in range(W)) / W

    out = torch.empty(n, device="cuda")
    stale = what == "no packet of this round"
    deliver(alive, ROUND + 1 if stale else ROUND)
    now = torch.zeros_like(alive) if stale else alive
    for flags in (now, torch.ones_like(alive)):
        if flags is not now:
            deliver(~now, ROUND)
        agg.finalize(out)
        want, size = mean(flags)
        assert bool(((out.double() - want).abs() <= 3 * 2.0 ** -24 * size).all())
        norm, want = agg.phase_signal()[0], float(out.double().square().sum().sqrt())
        # kept in double while the spans are stored, an updated one's old squares taken off: at most 3 n additions of terms
        # whose sizes add up to no more than three times the result, halved by the root
        assert abs(norm - want) <= 4.5 * n * 2.0 ** -53 * want
        c = agg.get_counters()
        assert c == dict(accepted=int(flags.sum()), duplicate=0, stale=int(alive.sum()) if stale else 0, invalid=0)

def _words(flags):
    import torch
    bits = torch.zeros(-(-flags.numel() // 64) * 64, dtype=torch.uint8, device="cuda")
    bits[:flags.numel()] = flags
    return (bits.view(-1, 8) * torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], dtype=torch.uint8, device="cuda")).sum(1, dtype=torch.uint8).view(torch.int64)


class _Buffer:
    """Every worker's packets of one gradient (the same for all: the mean then says how many arrived) at shuffled slots."""

    def __init__(self, W, P, n, rnd=ROUND):
        import torch
        import paper_2605_01989_amd as dblp
        self.agg = agg = dblp.Aggregator(W, n, P, [0], [n])
        gen = torch.Generator(device="cuda").manual_seed(W + n)
        self.grad = torch.randn(n, generator=gen, device="cuda")
        self.slots = W * agg.n_pkts
        self.slot_of = torch.randperm(self.slots, generator=gen, device="cuda").view(W, -1)
        self.u = torch.rand(W, agg.n_pkts, generator=gen, device="cuda")
        self.src = torch.empty(self.slots, dtype=torch.int16, device="cuda")
        self.fill(rnd)

    def fill(self, rnd):
        import torch
        self.packets = torch.empty(self.slots * self.agg.stride, dtype=torch.uint8, device="cuda")
        for w in range(self.agg.W):
            self.agg.packetize(w, rnd, self.grad, 0, 0, self.agg.n_pkts, self.packets, self.src, d_slot_map=self.slot_of[w].int())

    def mask(self, alive):
        import torch
        by_slot = torch.empty(self.slots, dtype=torch.bool, device="cuda")
        by_slot[self.slot_of.reshape(-1)] = alive.reshape(-1)
        return _words(by_slot)


@pytest.mark.parametrize("W,P,n", [(4, 256, 300_000), (3, 366, 5_000_003), (8, 366, 30_000_001), (4, 16374, 40_000_000)])
def test_few_of_many_slots(W, P, n):
    """Batches over the whole buffer whose masks leave nothing, a hundredth of the range, a hundredth of the packets, and
    nearly all; a round of another counter before the last."""
    import torch
    b = _Buffer(W, P, n)
    agg, pkts = b.agg, b.agg.n_pkts
    seq = torch.arange(pkts, device="cuda")
    alive = torch.zeros(W, pkts, dtype=torch.bool, device="cuda")
    copies = 0
    out = torch.empty(n, device="cuda")
    agg.begin_round(ROUND)
    for k, flags in enumerate((b.u < -1, ((seq >= pkts // 3) & (seq < pkts // 3 + 1 + pkts // 100)).expand(W, pkts), b.u < 0.01, b.u < 0.98)):
        if k == 3:
            b.fill(ROUND + 1)
            agg.apply_arrivals(b.packets, b.src, b.slots)
            agg.apply_arrivals(b.packets, b.src, b.slots)
            b.fill(ROUND)
        copies += int((flags & alive).sum())
        alive |= flags
        agg.apply_arrivals(b.packets, b.src, b.slots, b.mask(flags))
        agg.finalize(out)
        got = alive.double().sum(0).repeat_interleave(P)[:n]
        want = got * b.grad.double() / W
        assert bool(((out.double() - want).abs() <= 4 * 2.0 ** -24 * W * want.abs()).all())
        assert agg.get_counters() == dict(accepted=int(alive.sum()), duplicate=copies, stale=2 * b.slots if k == 3 else 0, invalid=0)


@pytest.mark.parametrize("masked", [False, True])
def test_what_arrived_is_asked_on_every_replay(masked):
    """A recorded round, told again on packets of this round, of another, and of this one again; masked: with the mask of
    nearly all, of a hundredth, of nothing, and of nearly all."""
    import torch
    W, P, n = 8, 366, 30_000_001
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        b = _Buffer(W, P, n)
        agg = b.agg
        shares = (0.98, 0.01, -1.0, 0.98) if masked else (2.0, 2.0, -1.0, 2.0)
        words = b.mask(b.u < 2)
        out = torch.empty(n, device="cuda")

        def receive():
            agg.begin_round(ROUND)
            agg.apply_arrivals(b.packets, b.src, b.slots, words if masked else None)
            agg.finalize(out)

        receive()
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        packets = b.packets
        with torch.cuda.graph(graph, stream=side):
            receive()
        for share in shares:
            alive = b.u < share
            if masked:
                words.copy_(b.mask(alive))
            else:
                b.fill(ROUND if share > 0 else ROUND + 1)
                packets.copy_(b.packets)
            out.fill_(7.0)
            side.synchronize()
            graph.replay()
            norm = agg.phase_signal()[0]
            want = alive.double().sum(0).repeat_interleave(P)[:n] * b.grad.double() / W
            assert bool(((out.double() - want).abs() <= 4 * 2.0 ** -24 * W * want.abs()).all())
            total = float(out.double().square().sum().sqrt())
            assert abs(norm - total) <= 4.5 * n * 2.0 ** -53 * total


def test_few_of_many_slots_take_few_slots_time():
    """What the gather of a whole buffer costs where a hundredth of the range is alive, or nothing of this round."""
    import torch
    from paper_2605_01989_amd import binding
    W, P, n = 8, 366, 124_000_000
    b = _Buffer(W, P, n)
    agg, pkts = b.agg, b.agg.n_pkts
    seq = torch.arange(pkts, device="cuda")
    some = b.mask(((seq >= pkts // 3) & (seq < pkts // 3 + pkts // 100)).expand(W, pkts))
    agg.profile_enable((1 << binding.K_GATHER) | (1 << binding.K_GATHER_DIRECT))

    def gather(rnd, mask):
        times = []
        for _ in range(9):
            agg.begin_round(rnd)
            agg.apply_arrivals(b.packets, b.src, b.slots, mask)
            times.append(agg.profile_read(binding.K_GATHER)[0] + agg.profile_read(binding.K_GATHER_DIRECT)[0])
        return sorted(times)[4]

    full = gather(ROUND, None)
    assert gather(ROUND, some) <= 0.06 * full
    assert gather(ROUND + 1, None) <= 0.03 * full
