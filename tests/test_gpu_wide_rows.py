"""Rows of more than 2048 columns, which the matrix-core passes do not take: the
vector-ALU passes of bf16 and Q4_0 layers and dense layers over blocks of
positions, and the LM head's own matrix-core kernel (5 to 12 positions whose
parts fit a CU's LDS) with the row-dot around it, on the GPU.

Against the same weights held as fp32: the products are the same but for the
rounding of an fp32 FMA, so the two differ by the order of the sums, a 2-norm
error of at most 2 sqrt(terms) 2^-24 per pass.
"""
import pytest
import torch

import paper_2607_24434_amd as de

from gpu_support import require_gpu
from test_gpu_grouped_mfma import inputs, layer, q4_blocks, rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def tol(terms):
    return 2 * 2.0 ** -24 * terms ** 0.5


# Wide inputs, wide intermediates, both, and a wide shared block alone.
WIDE = [(2080, 6, 3, 160, 320), (512, 5, 2, 2080, 0), (4096, 4, 2, 2560, 2560), (544, 4, 4, 96, 8224)]


@pytest.mark.parametrize("T", [2, 9, 17, 64])
@pytest.mark.parametrize("H,N,k,I,Is", WIDE)
@pytest.mark.parametrize("kind", ["verify", "draft"])
@pytest.mark.parametrize("dt", [de.DE_BF16, de.DE_Q4_0], ids=["bf16", "q4"])
def test_layer(T, H, N, k, I, Is, kind, dt):
    x, w, router = inputs(T, H, N, I, Is, T + H)
    if dt == de.DE_Q4_0:
        q, f = zip(*[q4_blocks(t.view(n, -1), n, i, H) if t is not None else (None, None)
                     for t, n, i in ((w[0], N, I), (w[1], 1, Is), (w[2], 1, I))])
    else:
        q = f = w
    a = layer(T, H, N, k, I, Is, x, q, router, dt, kind)
    b = layer(T, H, N, k, I, Is, x, f, router, de.DE_F32, kind)
    assert torch.equal(a[2], b[2]) and a[3] == b[3] == 0
    terms = max(H, I, Is)
    assert rel(a[0], b[0]) < 2 * tol(terms) and rel(a[1], b[1]) < 2 * tol(terms)


@pytest.mark.parametrize("T,H,I", [(1, 2056, 1000), (9, 4096, 1024), (17, 2056, 6000), (64, 2560, 520)])
def test_dense_layer(T, H, I):
    x, w, _ = inputs(T, H, 1, I, 0, T + I)
    out = []
    for dt, wt in ((de.DE_BF16, torch.bfloat16), (de.DE_F32, torch.float32)):
        y = torch.empty_like(x)
        ws = torch.empty(de.de_dense_workspace_bytes(T, H, I), dtype=torch.uint8, device="cuda")
        de.de_dense_swiglu(T, H, I, dt, x, w[0][0].to(wt), y, ws)
        out.append(y)
    assert rel(out[0], out[1]) < 2 * tol(max(H, I))


@pytest.mark.parametrize("H,V", [(2080, 1003), (4096, 333), (2056, 4100), (8192, 17)])
@pytest.mark.parametrize("T", [1, 4, 5, 6, 8, 12, 13, 64])
def test_lm_head(T, H, V):
    g = torch.Generator(device="cuda").manual_seed(T + H)
    # Whole numbers: every product and sum is exact, whichever kernel runs (the
    # matrix cores' for T = 5 to 12 of whole 32-column steps: all four lengths at
    # H = 2080, 5 and 6 at 4096).
    x = torch.randint(-256, 257, (T, H), generator=g, device="cuda").float()
    w = torch.randint(-4, 5, (V, H), generator=g, device="cuda").bfloat16()
    out = torch.full((T, V), float("nan"), device="cuda")
    de.de_lm_head(T, H, V, x, w, out)
    assert torch.equal(out.double(), x.double() @ w.double().t())


@pytest.mark.parametrize("T,H", [(5, 2080), (12, 2080), (6, 4096)])
def test_lm_head_parts(T, H):
    """Activations whose three bf16 parts all matter."""
    V = 515
    x, _, w = inputs(T, H, V, 8, 0, T)
    w = w.bfloat16()
    out = torch.empty(T, V, device="cuda")
    de.de_lm_head(T, H, V, x, w, out)
    assert rel(out, x.double() @ w.double().t()) < tol(H)
