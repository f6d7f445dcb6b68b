"""Row divergences at the edges of a block's batches and of its two sizes,
against 64 bits: 1e-4 relative (plus 1e-6), the tolerance of the signals."""
import pytest
import torch

import paper_2607_24434_amd as de

from gpu_support import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 257, 2047, 2048, 2049, 2560, 2561, 8191, 8193, 12288, 12289,
                               16383, 16384, 16385, 24577])
@pytest.mark.parametrize("sigmoid", [False, True])
def test_row_kl(n, sigmoid):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(n)
    rows, ld, tau = 3, n + 5, 1.0 if sigmoid else 1.7
    a = torch.randn(rows, ld, generator=g, device="cuda") * 3
    b = a + torch.randn(rows, ld, generator=g, device="cuda")
    kl, ce = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    de.de_row_kl(rows, n, a, ld, b, ld, None, sigmoid, tau, kl, None if sigmoid else ce)
    x, y = a[:, :n].double(), b[:, :n].double()
    if sigmoid:
        p, q = torch.sigmoid(x), torch.sigmoid(y)
        p, q = p / p.sum(1, keepdim=True), q / q.sum(1, keepdim=True)
        lp, lq = p.log(), q.log()
    else:
        lp, lq = torch.log_softmax(x / tau, 1), torch.log_softmax(y / tau, 1)
        want = -torch.log_softmax(y, 1).gather(1, x.argmax(1, keepdim=True))[:, 0]
        assert ((ce - want).abs() <= 1e-6 + 1e-4 * want.abs()).all()
    want = tau * tau * (lp.exp() * (lp - lq)).sum(1)
    assert ((kl - want).abs() <= 1e-6 + 1e-4 * want.abs()).all()


@pytest.mark.parametrize("n", [1, 300, 2500, 9000, 20000])
def test_token_ce_of_masked_rows(n):
    """Logits of -inf (masked tokens) add nothing to the sum, wherever they are."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(n)
    rows = 4
    a = torch.randn(rows, n, generator=g, device="cuda") * 3
    b = a + torch.randn(rows, n, generator=g, device="cuda")
    masked = torch.rand(rows, n, generator=g, device="cuda") < 0.5
    masked[:, : n // 2] |= torch.tensor([[True], [False], [True], [False]], device="cuda")
    masked[:, -1] = False
    a[masked], b[masked] = float("-inf"), float("-inf")
    kl, ce = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    de.de_row_kl(rows, n, a, n, b, n, None, False, 1.0, kl, ce)
    want = -torch.log_softmax(b.double(), 1).gather(1, a.argmax(1, keepdim=True))[:, 0]
    assert ((ce - want).abs() <= 1e-6 + 1e-4 * want.abs()).all()
