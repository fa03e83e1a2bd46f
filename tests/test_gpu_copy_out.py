"""GPU: the mean copied into another buffer, below and above the sizes at which the copy's pieces and its way change: runs of
missing and of delivered packets, bit for bit against the float32 additions in worker order and the division."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,P,n", [(1, 366, 3_999_999), (3, 366, 4_000_000), (3, 2243, 1_000_003), (1, 16374, 300_001), (2, 64, 70_007), (3, 5, 3001),
                                   (3, 281, 19_999_999), (1, 281, 20_000_000), (3, 2243, 20_000_003), (2, 16374, 25_000_001), (5, 65535, 20_400_000)])
def test_copied_out(W, P, n):
    import torch
    from test_gpu_few import _Rx
    rx = _Rx(W, P, [1, n // 3, 2, n - n // 3 - 3], n)
    seq = torch.arange(rx.pkts, device="cuda")
    gone = (seq % 97 < 11) | (seq < 3) | (seq == rx.pkts - 1)           # nobody delivers these yet
    some = (torch.rand(W, rx.pkts, generator=rx.gen, device="cuda") < 0.7) & ~gone
    for flags in (some, ~some & ~gone, (seq < 2).expand(W, -1), (gone & (seq >= 2)).expand(W, -1)):
        w, s = torch.nonzero(flags, as_tuple=True)
        rx.deliver(w, s, True)
        rx.check()
