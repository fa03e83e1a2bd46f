"""GPU: a probe's counts, list and verdict at the edges of its launches, against plain torch on the flags of what arrived.

Short rounds (at most 2048 bitmap words and 8192 pairs) are probed in one launch whose blocks count all pairs for themselves.  In
longer ones the list is written in one launch by blocks that add up each other's lengths while there are at most seven blocks per
four CUs (1792 pairs on 256 CUs, 448 where a block takes a pair), in two launches while there are at most 4096 blocks, and
in three beyond.  All values are integers and compared exactly."""
import pytest

pytestmark = pytest.mark.gpu

P, ROUND = 4, 9


def _context(W, packets):
    """Buckets of the given numbers of packets, the last packet of each a float short."""
    import paper_2605_01989_amd as dblp
    cnt = [n * P - 1 for n in packets]
    off = [0]
    for c in cnt:
        off.append(off[-1] + c)
    return dblp.Aggregator(W, off[-1], P, off[:-1], cnt)


def _expect(alive, first, n_b, bound):
    import torch
    lost = torch.zeros(alive.shape[0], alive.shape[1] + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(~alive, 1, out=lost[:, 1:])
    missing = lost[:, first[1:]] - lost[:, first[:-1]]
    fails = missing > bound * n_b // 1_000_000
    w, seq = torch.nonzero(~alive & fails.repeat_interleave(n_b, dim=1), as_tuple=True)
    return missing.int().flatten(), (w << 32) | seq


# short rounds: one pair; a few; many
SHORT = [(1, [1]), (3, [5, 70, 1, 64, 65, 129]), (3, [2] * 598), (32, [2] * 256)]
# longer ones: one pair, a block's, and 64, a wave's each; a block's remainder; as many pairs as one launch takes, and more; one pair a
# wave and two; 64 a wave, and more blocks than are added up without a scan; long buckets of which a block takes one, in one launch and in two
LONG = [(1, [131_073]), (64, [2100]), (33, [5, 70, 1, 64, 65, 4000]), (7, [1, 300] * 128), (3, [74] * 598), (32, [17] * 256), (33, [2] * 249), (64, [3, 1] * 4096),
        (64, [1] * 8193), (64, [1] * 16400), (5, [40_000, 3, 33_000, 1]), (64, [33_000, 3, 1, 70, 500, 9, 2, 64]), (56, [33_000] + [2] * 7), (50, [33_000] + [2] * 8)]
CASES = SHORT + LONG


def _is_short(agg):
    return agg.W * agg.words_pw <= 2048 and agg.W * agg.B <= 8192


@pytest.mark.parametrize("W,packets", CASES)
def test_probe_lists_what_is_missing(W, packets):
    agg = _context(W, packets)
    assert _is_short(agg) == ((W, packets) in SHORT)
    _probes(W, packets, agg)


@pytest.mark.parametrize("polls", [0, 1])
@pytest.mark.parametrize("W,packets", [c for c in CASES if c[0] * len(c[1]) <= 1792])
def test_probe_whose_blocks_do_not_wait_is_made_again(W, packets, polls):
    """With no look allowed every block that needs the ones before it gives up; with one, some may.  The answers are the
    same, also of a probe that may wait and follows one that gave up (its words in the totals carry no tag).  In a short round
    nobody waits, whatever is allowed."""
    agg = _context(W, packets)
    agg.probe_polls(polls)
    _probes(W, packets, agg, lambda k: agg.probe_polls(16384 if k % 3 == 2 else polls))


def _probes(W, packets, agg, before=None):
    import torch
    n_b = torch.tensor(packets, device="cuda")
    first = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), n_b.cumsum(0)])
    gen = torch.Generator(device="cuda").manual_seed(W + len(packets))
    grads = [torch.ones(agg.N, device="cuda") for _ in range(W)]
    alive = torch.zeros(W, agg.n_pkts, dtype=torch.bool, device="cuda")
    agg.begin_round(ROUND)
    missing = torch.empty(W * agg.B, dtype=torch.int32, device="cuda")
    out = torch.empty(W * agg.n_pkts + 1, dtype=torch.int64, device="cuda")
    for more in (0.0, 0.5, 0.9, 1.0):            # what has arrived before each probe; every packet before the last
        new = ~alive & (torch.rand(W, agg.n_pkts, generator=gen, device="cuda") < more)
        w, seq = torch.nonzero(new, as_tuple=True)
        n = w.numel()
        if n:
            packets_buf = torch.empty(n * agg.stride, dtype=torch.uint8, device="cuda")
            src = torch.empty(n, dtype=torch.int16, device="cuda")
            agg.packetize_list(ROUND, grads, (w << 32) | seq, n, packets_buf, src)
            agg.apply_arrivals(packets_buf, src, n)
        alive |= new
        for bound in (0, 200_000, 1_000_000):
            want_missing, want = _expect(alive, first, n_b, bound)
            for k, cap in enumerate((out.numel(), want.numel() // 2, 0)):
                if before is not None:
                    before(k)
                missing.fill_(-1)
                out.fill_(-1)
                count, met, truncated = agg.loss_account(bound, missing, out, cap)
                assert (count, met, truncated) == (want.numel(), want.numel() == 0, want.numel() > cap)
                assert torch.equal(missing, want_missing)
                k = min(cap, count)
                assert torch.equal(out[:k], want[:k]) and bool((out[k:] == -1).all())
    assert bool(alive.all())


# short rounds, which every block counts for itself: as many words and pairs as that takes, and more; whole words; buckets that
# end with a word, inside it, and many in one
@pytest.mark.parametrize("W,packets", [(1, [64]), (1, [63, 1]), (2, [64, 128, 64]), (3, [1] * 130), (32, [4096]), (32, [4000, 1, 95]), (33, [4000]),
                                       (32, [8] * 256), (64, [1] * 129), (5, [200, 1, 1, 1, 3000, 62, 64, 7]), (64, [2040, 8])])
def test_probe_of_a_short_round(W, packets):
    _probes(W, packets, _context(W, packets))


def test_probes_of_several_contexts_at_once():
    """Four contexts, each on a stream and in a thread of its own, of as many blocks as one launch takes."""
    import threading

    import torch
    W, packets, found = 32, [80] * 56, [None] * 4
    want = _expect(torch.zeros(W, 80 * 56, dtype=torch.bool, device="cuda"), torch.arange(57, device="cuda") * 80,
                   torch.full((56,), 80, device="cuda"), 0)

    def work(k):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            agg = _context(W, packets)
            agg.begin_round(ROUND)
            missing = torch.empty(W * agg.B, dtype=torch.int32, device="cuda")
            out = torch.empty(W * agg.n_pkts, dtype=torch.int64, device="cuda")
            ok = not _is_short(agg)         # its blocks wait for each other
            for _ in range(100):
                out.fill_(-1)
                ok = ok and agg.loss_account(0, missing, out) == (out.numel(), False, False)
                ok = ok and torch.equal(missing, want[0]) and torch.equal(out, want[1])
            found[k] = ok

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    torch.cuda.synchronize()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert found == [True] * 4
