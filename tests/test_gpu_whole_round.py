"""GPU: batches of about half a round, where the gather stops asking the index pass which range was touched.

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
