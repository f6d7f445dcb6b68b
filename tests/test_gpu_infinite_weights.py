"""Infinite and NaN bf16 weights, on the GPU: an output is what plain fp32 gives.

The matrix cores meet every weight with the three bf16 parts of an activation, of
which the lower two are zero here (activations exact in bf16), and infinity times
zero is NaN; plain fp32 gives an infinity there.  The outputs of other rows are
those of finite weights, bit for bit.
"""
import pytest
import torch

import paper_2607_24434_amd as de

from gpu_support import require_gpu
from test_gpu_grouped_mfma import TOL, inputs, layer, rel

pytestmark = pytest.mark.gpu

INF, NAN = float("inf"), float("nan")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def same_kind(a, b):
    """The same NaNs and infinities."""
    return torch.equal(a.isnan(), b.isnan()) and torch.equal(a == INF, b == INF) and \
        torch.equal(a == -INF, b == -INF)


@pytest.mark.parametrize("T,H,V", [(1, 264, 5000), (9, 264, 5000), (17, 264, 5000),
                                   (64, 2048, 40961), (3, 8, 50)])
def test_lm_head(T, H, V):
    g = torch.Generator(device="cuda").manual_seed(T)
    # Whole numbers: every product and sum is exact.
    x = torch.randint(1, 9, (T, H), generator=g, device="cuda").float()
    x[0, 0] = 0.0  # ... times infinity is NaN in fp32 too
    w = torch.randint(-8, 9, (V, H), generator=g, device="cuda").bfloat16()
    w[7, 3], w[V - 1, H - 1], w[40, 0] = INF, -INF, NAN
    w[21, 0], w[22, 1], w[22, 2] = INF, INF, -INF
    out = torch.empty(T, V, device="cuda")
    de.de_lm_head(T, H, V, x, w, out)
    rows = [7, V - 1, 40, 21, 22]
    clean = w.clone()
    clean[rows] = 0
    want = x.double() @ clean.double().t()
    want[:, 7], want[:, V - 1], want[:, 40], want[:, 21], want[:, 22] = INF, -INF, NAN, INF, NAN
    want[0, 21] = NAN
    assert same_kind(out, want)
    fin = want.isfinite()
    assert torch.equal(out.double()[fin], want[fin])


def bf16_exact(x):
    return x.bfloat16().float()


@pytest.mark.parametrize("T,H,N,k,I,Is", [(2, 72, 5, 3, 24, 40), (9, 512, 8, 2, 136, 296),
                                          (17, 264, 6, 6, 136, 264), (64, 520, 4, 4, 128, 256)])
@pytest.mark.parametrize("kind", ["verify", "draft"])
@pytest.mark.parametrize("where", ["gate", "up", "down"])
def test_layer(T, H, N, k, I, Is, kind, where):
    x, w, router = inputs(T, H, N, I, Is, T + H)
    x = bf16_exact(x)
    m = {"gate": 0, "up": 1, "down": 2}[where]
    # An infinite weight in one routed expert and one in the shared block.  (Not in
    # the last rows of G and U: the fp32 passes multiply those outputs with the zeros
    # past a row's end.)
    w[0].view(N, 3, I * H)[1, m, 5] = INF
    w[1].view(3, Is * H)[m, Is * H // 2 + 3] = -INF
    a = layer(T, H, N, k, I, Is, x, w, router, de.DE_BF16, kind)
    b = layer(T, H, N, k, I, Is, x, w, router, de.DE_F32, kind)
    assert torch.equal(a[2], b[2])
    if where == "down":
        # Finite activations meet the infinite weights: each makes one column infinite.
        assert same_kind(a[0], b[0])
        fin = b[0].isfinite()
        assert not fin.all() and fin.any()
        assert rel(a[0][fin], b[0][fin]) < TOL
    else:
        # An infinite gate or up output of some position: whole rows of infinities
        # and NaN.
        assert same_kind(a[0], b[0])


@pytest.mark.parametrize("T", [1, 9, 33])
@pytest.mark.parametrize("where", ["gate", "up", "down"])
def test_dense_layer(T, where):
    H, I = 520, 1000
    x, w, _ = inputs(T, H, 1, I, 0, T)
    x = bf16_exact(x)
    wt = w[0][0]
    wt.view(3, I * H)[{"gate": 0, "up": 1, "down": 2}[where], 3] = INF
    out = []
    for dt, t in ((de.DE_BF16, torch.bfloat16), (de.DE_F32, torch.float32)):
        y = torch.empty_like(x)
        ws = torch.empty(de.de_dense_workspace_bytes(T, H, I), dtype=torch.uint8, device="cuda")
        de.de_dense_swiglu(T, H, I, dt, x, wt.to(t), y, ws)
        out.append(y)
    assert same_kind(out[0], out[1])
    if where == "down":
        fin = out[1].isfinite()
        assert rel(out[0][fin], out[1][fin]) < 3 * TOL


def test_infinite_logit_wins_the_acceptance():
    T, H, V = 3, 256, 5000
    x = torch.ones(T, H, device="cuda")
    w = torch.zeros(V, H, device="cuda").bfloat16()
    w[4321, 17] = INF
    logits = torch.empty(T, V, device="cuda")
    de.de_lm_head(T, H, V, x, w, logits)
    amax = torch.empty(T, dtype=torch.int32, device="cuda")
    out = torch.empty(2, dtype=torch.int32, device="cuda")
    drafts = torch.tensor([4321, 4321], dtype=torch.int32, device="cuda")
    de.de_accept_len(T - 1, V, logits, drafts, amax, out, de.accept_workspace(T - 1, V))
    assert amax.tolist() == [4321] * T and out.tolist() == [2, 4321]


@pytest.mark.parametrize("T,H,V", [(3, 264, 5000), (18, 2048, 4099)])
def test_a_position_with_a_nan_beside_infinite_weights(T, H, V):
    """A NaN activation makes all outputs of its position NaN, and no others."""
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randint(1, 9, (T, H), generator=g, device="cuda").float()
    w = torch.randint(-8, 9, (V, H), generator=g, device="cuda").bfloat16()
    w[9, 5], w[V - 1, 0] = INF, -INF
    x[1, H - 1] = NAN
    out = torch.empty(T, V, device="cuda")
    de.de_lm_head(T, H, V, x, w, out)
    clean = w.clone()
    clean[[9, V - 1]] = 0
    want = x.double() @ clean.double().t()
    want[:, 9], want[:, V - 1], want[1] = INF, -INF, NAN
    assert same_kind(out, want)
    fin = want.isfinite()
    assert torch.equal(out.double()[fin], want[fin])


def test_the_single_launch_layer(monkeypatch):
    """The same in the single-launch verify layer, whose blocks read each other's
    outputs: the bits of the separate launches."""
    T, H, N, k, I, Is = 9, 512, 8, 2, 136, 296
    x, w, router = inputs(T, H, N, I, Is, 1)
    x = bf16_exact(x)
    w[0].view(N, 3, I * H)[1, 1, 5] = INF
    w[0].view(N, 3, I * H)[2, 2, 7] = -INF
    w[1].view(3, Is * H)[2, 9] = INF
    out = []
    for fused in ("0", "1"):
        monkeypatch.setenv("DE_VERIFY_FUSED", fused)
        out.append(layer(T, H, N, k, I, Is, x, w, router, de.DE_BF16))
    assert out[0][0].isinf().any() and out[0][0].isfinite().any()
    assert torch.equal(out[0][0].nan_to_num(1e30, 2e30, -2e30),
                       out[1][0].nan_to_num(1e30, 2e30, -2e30))
