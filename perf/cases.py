"""The receiver's and the sender's work on one GPU, as cases that can be timed and compared.

A case is a dict of plain values.  There are four kinds:

  round    one communication round as a parameter server runs it: begin_round, the arrivals of the
           first transmission (one batch, or one per chunk step), a probe, the retransmission batch
           and a second probe when the bound is not met, finalize, phase_signal, counters
  send     the sender's packetisation of one worker's gradient
  resend   the sender's answer to a retransmit list, all workers
  norm     the phase signal of a vector that the caller holds

Keys of a round: W workers, N floats, P floats per packet; `buckets` names the bucket table (see
`_sizes`); `form` how arrivals are handed over ("queue": descriptors; "tables": order + mask + worker
per slot); `place` where the packets lie in the receive buffer and `order` the order in which they
arrive; `loss`, `p` the loss process and its mean rate; `bound` the tolerance in ppm; `chunk` buckets
per arrival batch (0: the whole round is one batch); `dup` share of datagrams that arrive twice;
`out` "place" (the accumulator is the caller's buffer and the result stays in it) or "copy" (the
accumulator is the library's, the result is written to the caller's buffer).
"""
import math

import torch

import paper_2605_01989_amd as dblp

DEV = "cuda"
SIGMA = 1e-3            # standard deviation of the gradients' entries
ROUND = 7               # round counter carried in the headers
MAX_BYTES = 26 * 10**9  # packets of the largest listed round
MAX_SLOTS = 17_400_000


def listed():
    """Sizes: the workloads of this repository's benchmark and studies (1 M elements; ResNet-50;
    GPT-2 small and medium; 1.3 B in chunks, of which three steps are taken here; EfficientNet-B0;
    AlexNet) with the packet sizes of an MTU of 1500, of one-page payloads, of jumbo frames (9000)
    and of the largest UDP datagram."""
    def rnd(name, W, N, P, buckets, **k):
        c = dict(name=name, kind="round", W=W, N=N, P=P, buckets=buckets, form="queue", place="shuffle", order="shuffle",
                 loss="iid", p=0.02, bound=50_000, chunk=0, dup=0.0, out="place")
        c.update(k)
        return c
    return [
        # the smallest round in use: launches and host round trips count
        rnd("small_w4", 4, 1 << 20, 256, "fixed64", place="worker_major", p=0.01),
        # three workers and one accounting unit per worker, the mean written to the caller's buffer: a
        # worker count that is no power of two, and a loss above the tolerance, so that one
        # retransmission round follows
        rnd("effnetb0_w3", 3, 5_288_548, 366, "one", form="tables", place="interleave", bound=8_000, out="copy"),
        # an ordinary round over per-tensor buckets of very different sizes
        rnd("resnet50_w8", 8, 25_600_000, 366, "log161"),
        # bursty loss against a tight bound: many buckets fail and are sent again
        rnd("gpt2s_w8", 8, 124_439_808, 366, "gpt2_768_12", loss="burst", p=0.007, bound=10_000),
        # 4 KB packets that arrive nearly in order, contiguous loss windows
        rnd("gpt2m_w16_4k", 16, 354_823_168, 1024, "gpt2_1024_24", place="interleave", order="identity", loss="window", p=0.02,
            bound=80_000),
        # many workers, arrivals in chunk steps, heavy bursts; the largest round
        rnd("chunked_w32", 32, 3 * 44 * 4096 * 366, 366, "fixed4096", loss="burst", p=0.032, bound=20_000, chunk=44),
        # jumbo frames
        rnd("jumbo_w8", 8, 124_439_808, 2243, "gpt2_768_12", p=0.01, dup=0.002),
        # the largest UDP datagrams
        rnd("datagram64k_w4", 4, 61_100_840, 16374, "log16", place="interleave", p=0.005),
        # the broadcast leg: one sender's packets received by a worker, loss within the tolerance
        rnd("broadcast_w1", 1, 25_600_000, 366, "log161", place="interleave", order="identity", p=0.005),
        # the sender's side of an ordinary round, of its retransmission, and Eq. 1 on a held vector
        dict(name="send_resnet50", kind="send", N=25_600_000, P=366, buckets="log161", map=False),
        dict(name="resend_gpt2s_w8", kind="resend", W=8, N=124_439_808, P=366, buckets="gpt2_768_12", p=0.03),
        dict(name="norm_gpt2s", kind="norm", N=124_439_808),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["round", "send", "resend", "norm"], [8, 1, 1, 1])[0]
    if kind == "norm":
        return dict(kind=kind, N=_log(rng, 10_000, 1_300_000_000))
    P = rng.choice([366, 256, 1024, 2243, 16374, _log(rng, 64, 1100), _log(rng, 64, 16374)])
    buckets = rng.choice(["one", "fixed64", "fixed4096", "log16", "log161", "log%d" % _log(rng, 2, 3000), "gpt2_768_12", "gpt2_1024_24"])
    if kind == "send":
        return dict(kind=kind, N=_log(rng, 200_000, 355_000_000), P=P, buckets=buckets, map=rng.random() < 0.5)
    W = rng.choice([1, 2, 3, 4, 8, 8, 16, 32, rng.randint(2, 64), rng.randint(2, 64)])
    # the largest gradient whose packets stay below the largest listed round's
    top = min(355_000_000, MAX_BYTES * P // (W * ((8 + 4 * P + 15) // 16 * 16)), MAX_SLOTS * P // W - 4096 * P)
    if kind == "resend":
        return dict(kind=kind, W=W, N=_log(rng, 200_000, min(top, 1_000_000_000 // W)), P=P, buckets=buckets,
                    p=round(rng.uniform(0.002, 0.1), 4))
    loss = rng.choice(["iid", "burst", "window"])
    return dict(kind=kind, W=W, N=_log(rng, 200_000, top), P=P, buckets=buckets, form=rng.choice(["queue", "queue", "tables"]),
                place=rng.choice(["shuffle", "interleave", "worker_major"]), order=rng.choice(["shuffle", "identity"]),
                loss=loss, p=round(rng.uniform(0.007, 0.05), 4), bound=rng.choice([8_000, 20_000, 50_000, 150_000]),
                chunk=44 if buckets == "fixed4096" else 0, dup=rng.choice([0.0, 0.0, 0.002]),
                out="place" if W & (W - 1) == 0 and rng.random() < 0.6 else "copy")


# ---------------------------------------------------------------------------------------------
# geometry
# ---------------------------------------------------------------------------------------------
def _sizes(case):
    """Elements per bucket: "one"; "fixedK" buckets of K packets; "logK" K sizes spread evenly over the
    logarithm from 1 to 2400, scaled; "gpt2_D_L" the tensors of a GPT-2 of width D with L layers, scaled."""
    N, P, kind = case["N"], case["P"], case["buckets"]
    if kind == "one":
        return [N]
    if kind.startswith("fixed"):
        per = int(kind[5:]) * P
        return [per] * (N // per) + ([N % per] if N % per else [])
    if kind.startswith("log"):
        n = int(kind[3:])
        raw = [math.exp(math.log(2400.0) * ((i * 0.6180339887498949) % 1.0)) for i in range(n)]
    else:
        d, layers = (int(v) for v in kind.split("_")[1:])
        raw = [50257 * d, 1024 * d] + [d, d, 3 * d * d, 3 * d, d * d, d, d, d, 4 * d * d, 4 * d, 4 * d * d, d] * layers + [d, d]
    total = sum(raw)
    sizes = [max(1, int(v * N / total)) for v in raw]
    sizes[sizes.index(max(sizes))] += N - sum(sizes)
    return sizes


class _Geo:
    def __init__(self, case):
        self.W, self.N, self.P = case.get("W", 1), case["N"], case["P"]
        self.cnt = _sizes(case)
        self.off = [0]
        for c in self.cnt:
            self.off.append(self.off[-1] + c)
        self.off.pop()
        self.n_b = [-(-c // self.P) for c in self.cnt]
        self.first = [0]
        for n in self.n_b:
            self.first.append(self.first[-1] + n)
        self.n_pkts, self.B = self.first[-1], len(self.cnt)
        self.stride = (8 + 4 * self.P + 15) // 16 * 16

    def steps(self, chunk):
        """Sequence ranges of the arrival batches."""
        if not chunk:
            return [(0, self.n_pkts)]
        return [(self.first[b], self.first[min(b + chunk, self.B)]) for b in range(0, self.B, chunk)]

    def context(self, accumulator=None):
        return dblp.Aggregator(self.W, self.N, self.P, self.off, self.cnt, d_accumulator=(accumulator, None))


def _gen(seed, stream):
    return torch.Generator(device=DEV).manual_seed((seed * 1_000_003 + stream * 7919 + 17) & (2**62 - 1))


def _grad(case, seed, w):
    return torch.randn(case["N"], generator=_gen(seed, 1000 + w), device=DEV).mul_(SIGMA)


# ---------------------------------------------------------------------------------------------
# the network: loss, placement, order of arrival
# ---------------------------------------------------------------------------------------------
def _bursts(n, rate, mean_len, g):
    """Flags of `n` positions that lie inside bursts: starts at `rate`, geometric lengths."""
    edge = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    start = torch.nonzero(torch.rand(n, generator=g, device=DEV) < rate).flatten()
    u = torch.rand(start.numel(), generator=g, device=DEV).clamp_min(1e-7)
    end = (start + 1 + (u.log() / math.log(1 - 1 / mean_len)).long()).clamp_max(n)
    edge.index_add_(0, start, torch.ones_like(start, dtype=torch.int32))
    edge.index_add_(0, end, -torch.ones_like(end, dtype=torch.int32))
    return edge[:n].cumsum(0) > 0


def _survive(case, geo, slot_of, seed):
    """[W, n_pkts] flags: the first transmission of the packet arrived."""
    g, p, n = _gen(seed, 1), case["p"], geo.W * geo.n_pkts
    u = torch.rand(n, generator=g, device=DEV)
    if case["loss"] == "iid":
        alive = u >= p
    elif case["loss"] == "burst":       # 30 % loss inside bursts of 40 packets on average
        alive = u >= torch.where(_bursts(n, p / 0.3 / 40 * 0.9, 40, g), 0.3, 0.1 * p)
    else:                               # three windows of the wire sequence, and background loss
        alive = u >= p / 4
        size = max(1, int(n * p / 4))
        seg = n // 3
        at = (torch.rand(3, generator=g, device=DEV) * max(1, seg - size)).long().tolist()
        slot = slot_of.reshape(-1)
        for j in range(3):
            alive &= (slot < j * seg + at[j]) | (slot >= j * seg + at[j] + size)
    return alive.view(geo.W, geo.n_pkts)


def _placement(case, geo, seed):
    """[W, n_pkts] slots; the packets of one arrival batch lie together."""
    g = _gen(seed, 2)
    slot_of = torch.empty(geo.W, geo.n_pkts, dtype=torch.int64, device=DEV)
    for s0, s1 in geo.steps(case["chunk"]):
        n, m = geo.W * (s1 - s0), s1 - s0
        if case["place"] == "worker_major":
            local = torch.arange(n, device=DEV)
        elif case["place"] == "shuffle":
            local = torch.randperm(n, generator=g, device=DEV)
        else:   # each worker's packets in order, the workers' streams merged with jitter
            key = torch.arange(m, device=DEV).repeat(geo.W) * geo.W * 4 + torch.randint(0, geo.W * 16, (n,), generator=g, device=DEV)
            key = key.view(geo.W, m).cummax(1).values.reshape(-1)
            local = torch.empty(n, dtype=torch.int64, device=DEV)
            local[torch.argsort(key, stable=True)] = torch.arange(n, device=DEV)
        slot_of[:, s0:s1] = local.view(geo.W, m) + geo.W * s0
    return slot_of


def _missing(geo, alive):
    """[W, B] packets of each bucket that have not arrived."""
    c = torch.zeros(geo.W, geo.n_pkts + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(~alive, 1, out=c[:, 1:])
    first = torch.tensor(geo.first, device=DEV)
    return c[:, first[1:]] - c[:, first[:-1]]


def _to_resend(geo, alive, bound):
    """[W, n_pkts] flags of the packets that a sender sends again: the missing ones of each (worker, bucket) above the bound."""
    n_b = torch.tensor(geo.n_b, device=DEV)
    fails = _missing(geo, alive) > bound * n_b // 1_000_000
    return ~alive & fails.repeat_interleave(n_b, dim=1)


def _words(flags):
    """Mask words: bit s % 64 of word s / 64."""
    n = flags.numel()
    bits = torch.zeros(-(-n // 64) * 64, dtype=torch.uint8, device=DEV)
    bits[:n] = flags
    weights = torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], dtype=torch.uint8, device=DEV)
    return (bits.view(-1, 8) * weights).sum(1, dtype=torch.uint8).view(torch.int64)


# ---------------------------------------------------------------------------------------------
# what a program holds before the call
# ---------------------------------------------------------------------------------------------
def prepare(case, seed):
    return {"round": _prepare_round, "send": _prepare_send, "resend": _prepare_resend, "norm": _prepare_norm}[case["kind"]](case, seed)


def _prepare_round(case, seed):
    geo = _Geo(case)
    out = torch.empty(geo.N, device=DEV)
    agg = geo.context(out if case["out"] == "place" else None)
    n_slots = geo.W * geo.n_pkts
    slot_of = _placement(case, geo, seed)
    alive = _survive(case, geo, slot_of, seed)
    packets = torch.empty(n_slots * geo.stride, dtype=torch.uint8, device=DEV)
    src = torch.empty(n_slots, dtype=torch.int16, device=DEV)
    for w in range(geo.W):
        agg.packetize(w, ROUND, _grad(case, seed, w), 0, 0, geo.n_pkts, packets, src, d_slot_map=slot_of[w].int())
    by_slot = torch.empty(n_slots, dtype=torch.bool, device=DEV)
    by_slot[slot_of.reshape(-1)] = alive.reshape(-1)
    g = _gen(seed, 3)
    batches = []
    for s0, s1 in geo.steps(case["chunk"]):
        base, n = geo.W * s0, geo.W * (s1 - s0)
        slots = torch.randperm(n, generator=g, device=DEV) if case["order"] == "shuffle" else torch.arange(n, device=DEV)
        if case["dup"]:
            slots = torch.cat([slots, slots[torch.randint(0, n, (max(1, int(n * case["dup"])),), generator=g, device=DEV)]])
        here, sent_by = by_slot[base:base + n], src[base:base + n]
        b = dict(packets=packets[base * geo.stride:(base + n) * geo.stride], n=n)
        if case["form"] == "queue":
            slots = slots[here[slots]]
            b["queue"] = slots | (sent_by[slots].long() << 32)
        else:
            b.update(src=sent_by, mask=_words(here), order=None if case["order"] == "identity" and not case["dup"] else slots.int())
        batches.append(b)
    again = _to_resend(geo, alive, case["bound"])
    w, seq = torch.nonzero(again, as_tuple=True)
    slots = slot_of[w, seq]
    resent = dict(packets=packets, n=n_slots)
    if case["form"] == "queue":
        resent["queue"] = slots | (w << 32)
    else:
        resent.update(src=src, mask=None, order=slots.int())
    return dict(kind="round", agg=agg, batches=batches, resent=resent, bound=case["bound"],
                lists=torch.zeros(n_slots // 2 + 64, dtype=torch.int64, device=DEV),
                missing=torch.empty(geo.W * geo.B, dtype=torch.int32, device=DEV), prev=1.25 * SIGMA * math.sqrt(geo.N / geo.W),
                out=out)


def _prepare_send(case, seed):
    geo = _Geo(case)
    g = _gen(seed, 2)
    return dict(kind="send", agg=geo.context(), grad=_grad(case, seed, 0), n=geo.n_pkts,
                map=torch.randperm(geo.n_pkts, generator=g, device=DEV).int() if case["map"] else None,
                packets=torch.empty(geo.n_pkts * geo.stride, dtype=torch.uint8, device=DEV),
                src=torch.empty(geo.n_pkts, dtype=torch.int16, device=DEV))


def _lost(case, geo):
    """Entries of the list of a "resend" case."""
    return max(1, int(geo.W * geo.n_pkts * case["p"]))


def _prepare_resend(case, seed):
    geo = _Geo(case)
    n = _lost(case, geo)
    at = torch.randperm(geo.W * geo.n_pkts, generator=_gen(seed, 1), device=DEV)[:n].sort().values
    return dict(kind="resend", agg=geo.context(), grads=[_grad(case, seed, i) for i in range(geo.W)], n=n,
                list=((at // geo.n_pkts) << 32) | (at % geo.n_pkts),
                packets=torch.empty(n * geo.stride, dtype=torch.uint8, device=DEV), src=torch.empty(n, dtype=torch.int16, device=DEV))


def _prepare_norm(case, seed):
    agg = dblp.Aggregator(1, case["N"], 366, [0], [case["N"]])
    return dict(kind="norm", agg=agg, vec=_grad(case, seed, 0), prev=1.25 * SIGMA * math.sqrt(case["N"]))


# ---------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------
def _apply(agg, b):
    if "queue" in b:
        agg.apply_arrivals_queue(b["packets"], b["n"], b["queue"])
    else:
        agg.apply_arrivals(b["packets"], b["src"], b["n"], b["mask"], b["order"])


def run(s):
    agg = s["agg"]
    if s["kind"] == "send":
        agg.packetize(0, ROUND, s["grad"], 0, 0, s["n"], s["packets"], s["src"], d_slot_map=s["map"])
        return dict(packets=s["packets"].view(torch.int32), src=s["src"])
    if s["kind"] == "resend":
        agg.packetize_list(ROUND, s["grads"], s["list"], s["n"], s["packets"], s["src"])
        return dict(packets=s["packets"].view(torch.int32), src=s["src"])
    if s["kind"] == "norm":
        agg.set_prev_norm(s["prev"])
        norm, delta, critical = agg.phase_signal(s["vec"])
        return dict(norm=norm, delta=delta, critical=critical)
    agg.begin_round(ROUND)
    for b in s["batches"]:
        _apply(agg, b)
    count, met, _ = agg.loss_account(s["bound"], s["missing"], s["lists"])
    if not met:
        _apply(agg, s["resent"])
        _, met, _ = agg.loss_account(s["bound"], s["missing"], s["lists"][count:])
    agg.finalize(s["out"])
    agg.set_prev_norm(s["prev"])
    norm, delta, critical = agg.phase_signal()
    return dict(mean=s["out"], missing=s["missing"], resend=s["lists"], met=met,
                norm=norm, delta=delta, critical=critical, counters=agg.get_counters())


# ---------------------------------------------------------------------------------------------
# what it has to move, how exact it is, and the result in 64 bits
# ---------------------------------------------------------------------------------------------
def work(case):
    """Bytes: every packet that arrives read once, its descriptor (or table entries) once, the mean
    written once; a sender reads the gradient and writes the packets; a norm reads its vector."""
    if case["kind"] == "norm":
        return dict(bytes=4 * case["N"], flops=2 * case["N"])
    geo = _Geo(case)
    if case["kind"] == "send":
        return dict(bytes=4 * geo.N + geo.n_pkts * (geo.stride + 2 + (4 if case["map"] else 0)), flops=0)
    if case["kind"] == "resend":
        return dict(bytes=_lost(case, geo) * (8 + 4 * geo.N / geo.n_pkts + geo.stride + 2), flops=0)
    sent = geo.W * geo.n_pkts
    got = sent * (1 - case["p"])
    per = 8 if case["form"] == "queue" else 6 + 1 / 8
    return dict(bytes=got * geo.stride + (got if case["form"] == "queue" else sent) * per + 4 * geo.N + 4 * geo.W * geo.B,
                flops=(geo.W * (1 - case["p"]) + 1) * geo.N)


def tolerance(case):
    """Wire bytes and counts are exact.  The mean: a 32-bit sum of up to 64 addends, measured against the
    64-bit sum at 3e-8 (2 workers) to 1e-7 (32) of the 2-norm, the norms below 1e-7; `rel` is about four
    times what 64 addends give, `max` is for elements whose addends cancel."""
    if case["kind"] in ("send", "resend"):
        return "exact"
    return dict(rel=6e-7, max=1e-5, differ=0.0)


def exact(case, seed):
    """The mean of what arrived and its norm in 64 bits, with plain torch; counts and lists have no
    rounding and are compared as they are."""
    if case["kind"] in ("send", "resend"):
        return None
    if case["kind"] == "norm":
        norm = float(_grad(case, seed, 0).double().square().sum().sqrt())
        prev = 1.25 * SIGMA * math.sqrt(case["N"])
        return dict(norm=norm, delta=abs(prev - norm) / prev, critical=None)
    geo = _Geo(case)
    slot_of = _placement(case, geo, seed)
    alive = _survive(case, geo, slot_of, seed)
    alive |= _to_resend(geo, alive, case["bound"])
    lens = torch.full((geo.n_pkts,), geo.P, dtype=torch.int64, device=DEV)
    lens[torch.tensor(geo.first[1:], device=DEV) - 1] = torch.tensor([c - (n - 1) * geo.P for c, n in zip(geo.cnt, geo.n_b)], device=DEV)
    packet = torch.repeat_interleave(torch.arange(geo.n_pkts, device=DEV, dtype=torch.int32), lens)
    mean = torch.zeros(geo.N, dtype=torch.float64, device=DEV)
    for w in range(geo.W):
        got = alive[w].float().index_select(0, packet)      # 0 or 1: the product below is exact
        mean += got.mul_(_grad(case, seed, w))
    mean /= geo.W
    norm = float(mean.square().sum().sqrt())
    prev = 1.25 * SIGMA * math.sqrt(geo.N / geo.W)
    return dict(mean=mean, missing=None, resend=None, met=None, norm=norm, delta=abs(prev - norm) / prev, critical=None, counters=None)
