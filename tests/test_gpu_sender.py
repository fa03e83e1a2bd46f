"""GPU: the senders' packets, short ones of which a wave writes several at once and longer ones, against their bytes built by plain torch."""
import pytest

pytestmark = pytest.mark.gpu

ROUND = 70_003          # the header holds its low 16 bits


def _make(W, P, sizes, seed):
    import torch
    import paper_2605_01989_amd as dblp
    off = [sum(sizes[:i]) for i in range(len(sizes))]
    agg = dblp.Aggregator(W, sum(sizes), P, off, sizes)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    grads = [torch.randn(sum(sizes), generator=gen, device="cuda") for _ in range(W)]
    start, length = [], []
    for o, c in zip(off, sizes):
        k = -(-c // P)
        start += [o + i * P for i in range(k)]
        length += [P] * (k - 1) + [c - (k - 1) * P]
    assert len(start) == agg.n_pkts
    return agg, gen, grads, torch.tensor(start, device="cuda"), torch.tensor(length, device="cuda")


def _wire(agg, grads, start, length, w, seq):
    """The packets (w[i], seq[i]), a row each, as int32 words."""
    import torch
    words = agg.stride // 4
    i = torch.arange(words - 2, device="cuda")[None, :]
    n = length[seq][:, None]
    at = (start[seq][:, None] + i).clamp(max=grads[0].numel() - 1)
    rows = torch.zeros(seq.numel(), words, dtype=torch.int32, device="cuda")
    for k, g in enumerate(grads):
        mine = (w == k)[:, None]
        rows[:, 2:] = torch.where(mine & (i < n), g.view(torch.int32)[at], rows[:, 2:])
    rows[:, 0] = seq.to(torch.int32)
    head = (ROUND & 0xFFFF) | (length[seq] << 16)
    rows[:, 1] = torch.where(head >= 2**31, head - 2**32, head).to(torch.int32)
    return rows


def _sizes(P, pkts, many):
    """About pkts packets: whole ones, a bucket of one float, odd offsets; the last bucket ends in a packet of one float."""
    sizes = [P * (pkts // 2) + 1, 1, P, 2 * P + 3]
    if many:
        sizes += [7] * 5000               # more buckets than the boundaries kept in LDS
    return sizes + [P * (pkts // 2 - 3) + 1]


# payload floats: 2 units (64 packets of a wave) .. 127, 128 (the last with two), 129 and more (one)
SHORT = [1, 2, 3, 14, 62, 63, 126, 127, 254, 255, 300, 366, 505, 506, 507, 510, 511, 514, 1100, 2001]


@pytest.mark.parametrize("pkts", [300, 8_191, 8_300, 41_003])
@pytest.mark.parametrize("P", SHORT)
def test_range_of_packets(P, pkts):
    import torch
    many = pkts == 41_003 and P in (1, 14, 254, 511)
    agg, gen, grads, start, length = _make(2, P, _sizes(P, pkts, many), P + pkts)
    n = agg.n_pkts
    for first, count, by_map in ((0, n, False), (3, n - 3, True), (n - 1, 1, True), (5, n // 2, False)):
        seq = torch.arange(first, first + count, device="cuda")
        slots = count + 9
        to = torch.randperm(slots, generator=gen, device="cuda")[:count] if by_map else torch.arange(count, device="cuda") + 4
        packets = torch.full((slots * agg.stride,), 0x5A, dtype=torch.uint8, device="cuda")
        src = torch.full((slots,), 777, dtype=torch.int16, device="cuda")
        base = int(start[first])                      # the gradient handed over begins at the first packet
        agg.packetize(1, ROUND, grads[1][base:].clone(), base, first, count, packets, src,
                      d_slot_map=to.to(torch.int32) if by_map else None, slot_base=0 if by_map else 4)
        want = torch.full((slots, agg.stride // 4), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        want[to] = _wire(agg, grads, start, length, torch.ones_like(seq), seq)
        want_src = torch.full((slots,), 777, dtype=torch.int16, device="cuda")
        want_src[to] = 1
        assert torch.equal(packets.view(torch.int32).view(slots, -1), want), (first, count)
        assert torch.equal(src, want_src)


@pytest.mark.parametrize("entries", [1, 8_192, 20_011])
@pytest.mark.parametrize("P", [1, 14, 63, 127, 254, 366, 506, 511, 1100])
def test_list_of_packets(P, entries):
    import torch
    W = 3
    agg, gen, grads, start, length = _make(W, P, _sizes(P, 9_000, P in (14, 366)), P + entries)
    w = torch.randint(0, W, (entries,), generator=gen, device="cuda")
    seq = torch.randint(0, agg.n_pkts, (entries,), generator=gen, device="cuda")
    packets = torch.full(((entries + 2) * agg.stride,), 0x5A, dtype=torch.uint8, device="cuda")
    src = torch.full((entries + 2,), 777, dtype=torch.int16, device="cuda")
    agg.packetize_list(ROUND, grads, ((w << 32) | seq).contiguous(), entries, packets, src, slot_base=1)
    rows = packets.view(torch.int32).view(entries + 2, -1)
    assert torch.equal(rows[1:-1], _wire(agg, grads, start, length, w, seq))
    assert bool((rows[0] == 0x5A5A5A5A).all()) and bool((rows[-1] == 0x5A5A5A5A).all())
    assert torch.equal(src[1:-1].long(), w) and int(src[0]) == int(src[-1]) == 777


def test_entries_out_of_range_are_refused_and_the_others_written():
    import torch
    import paper_2605_01989_amd as dblp
    P, W = 20, 2
    agg, gen, grads, start, length = _make(W, P, _sizes(P, 17_000, False), 5)
    n = agg.n_pkts
    bad = torch.tensor([0, 4_001, n - 1], device="cuda")
    good = torch.ones(n, dtype=torch.bool, device="cuda")
    good[bad] = False
    seq, one = torch.arange(n, device="cuda"), torch.ones(n, dtype=torch.int64, device="cuda")
    want = _wire(agg, grads, start, length, one, seq)
    want[bad] = 0x5A5A5A5A
    fresh = lambda: (torch.full((n * agg.stride,), 0x5A, dtype=torch.uint8, device="cuda"), torch.full((n,), 777, dtype=torch.int16, device="cuda"))

    packets, src = fresh()
    to = seq.clone()
    to[bad] = n
    with pytest.raises(dblp.DblpError):
        agg.packetize(1, ROUND, grads[1], 0, 0, n, packets, src, d_slot_map=to.to(torch.int32))
    assert torch.equal(packets.view(torch.int32).view(n, -1), want) and torch.equal(src == 1, good)

    packets, src = fresh()
    entry = (one << 32) | seq
    entry[bad] = torch.tensor([W << 32, (1 << 32) | n, -1], device="cuda")
    with pytest.raises(dblp.DblpError):
        agg.packetize_list(ROUND, grads, entry, n, packets, src)
    assert torch.equal(packets.view(torch.int32).view(n, -1), want) and torch.equal(src == 1, good)
