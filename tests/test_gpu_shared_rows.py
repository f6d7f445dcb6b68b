"""Launches of one dense source (dense layer, LM head) over several position
groups: the blocks of two and four groups are cut into runs that read the same
rows together; three groups, and fewer tiles than the chip has CUs, take the
plain order.  Whole numbers: every product and sum is exact."""
import pytest
import torch

import paper_2607_24434_amd as de

from gpu_support import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [4096 - 31, 8191, 10240, 25001])
@pytest.mark.parametrize("T,H", [(17, 2048), (32, 1000), (33, 264), (48, 520), (49, 2048), (64, 72)])
def test_lm_head(T, H, V):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(V + T)
    x = torch.randint(-512, 513, (T, H), generator=g, device="cuda").float()
    w = torch.randint(-8, 9, (V, H), generator=g, device="cuda").bfloat16()
    out = torch.full((T, V), float("nan"), device="cuda")
    de.de_lm_head(T, H, V, x, w, out)
    assert torch.equal(out.double(), x.double() @ w.double().t())


@pytest.mark.parametrize("T,H,I", [(17, 2048, 10944), (32, 1032, 5000), (64, 2048, 10944)])
def test_dense_layer(T, H, I):
    """bf16 weights against the same weights in fp32 on the vector ALU: sums of
    up to I terms in another order, 2^-24 sqrt(I) relative each way."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(T + H)
    x = torch.randn(T, H, generator=g, device="cuda")
    w = (torch.randn(3 * I * H, generator=g, device="cuda") * 0.02).bfloat16()
    out = []
    for dt, wt in ((de.DE_BF16, torch.bfloat16), (de.DE_F32, torch.float32)):
        y = torch.full_like(x, float("nan"))
        ws = torch.empty(de.de_dense_workspace_bytes(T, H, I), dtype=torch.uint8, device="cuda")
        de.de_dense_swiglu(T, H, I, dt, x, w.to(wt), y, ws)
        out.append(y.double())
    assert (out[0] - out[1]).norm() / out[1].norm() < 2 * 2.0 ** -24 * I ** 0.5
