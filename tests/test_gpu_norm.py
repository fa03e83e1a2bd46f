"""GPU: sums of squares whose blocks are added up by the last block of their own launch.

Against float64: the four squares of a 16-byte unit are added in float32 (three roundings of at most 2**-24 each, relative
to a sum of positive terms), the rest in double, so the sum is within 3 * 2**-24 and the norm within half of that."""
import math

import pytest

pytestmark = pytest.mark.gpu

TOL = 1.5 * 2.0 ** -24 + 1e-12


# floats: less than a unit, around a run of 4096, around 512 runs (a block each), several runs a block with a remainder
@pytest.mark.parametrize("n", [1, 3, 4, 4095, 4097, 511 * 4096 + 5, 512 * 4096, 512 * 4096 + 1, 9_000_003])
def test_norm_of_a_vector(n):
    import torch
    import paper_2605_01989_amd as dblp
    agg = dblp.Aggregator(1, n, 366, [0], [n])
    gen = torch.Generator(device="cuda").manual_seed(n)
    for scale in (1e-3, 5.0, 1e-3):              # what an earlier call left in the context must not show
        v = torch.randn(n, generator=gen, device="cuda").mul_(scale)
        want = float(v.double().square().sum().sqrt())
        assert abs(agg.phase_signal(v)[0] - want) <= TOL * want
    v[n // 2] = math.inf
    assert math.isinf(agg.phase_signal(v)[0])
    v[n // 2] = math.nan
    assert math.isnan(agg.phase_signal(v)[0])


@pytest.mark.parametrize("W,n", [(3, 50), (5, 700_001), (3, 9_000_001)])
def test_norm_of_a_round_whose_worker_count_is_no_power_of_two(W, n):
    """Eager, with a vector's norm in between (the two share their words), and replayed from a graph three times."""
    import torch
    import paper_2605_01989_amd as dblp
    P, rnd = 366, 3
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        agg = dblp.Aggregator(W, n, P, [0], [n])
        gen = torch.Generator(device="cuda").manual_seed(n)
        packets = torch.empty(W * agg.n_pkts * agg.stride, dtype=torch.uint8, device="cuda")
        src = torch.empty(W * agg.n_pkts, dtype=torch.int16, device="cuda")
        out = torch.empty(n, device="cuda")

        def send(scale):
            for w in range(W):
                agg.packetize(w, rnd, torch.randn(n, generator=gen, device="cuda").mul_(scale), 0, 0, agg.n_pkts, packets, src, slot_base=w * agg.n_pkts)

        def receive():
            agg.begin_round(rnd)
            agg.apply_arrivals(packets, src, W * agg.n_pkts)
            agg.finalize(out)

        def check():
            norm = agg.phase_signal()[0]
            want = float(out.double().square().sum().sqrt())
            assert abs(norm - want) <= TOL * want
            assert agg.phase_signal()[0] == norm          # asked again: the same

        send(1e-3)
        receive()
        check()
        agg.phase_signal(out)
        receive()
        check()
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            receive()
        for scale in (1.0, 1e-4, 20.0):
            send(scale)
            side.synchronize()
            graph.replay()
            check()
