"""Layer calls with a scratch of just the bytes they use, on the GPU."""
import pytest
import torch

import paper_2607_24434_amd as de

from gpu_support import require_gpu
from test_workspace import desc, plain, up256

pytestmark = pytest.mark.gpu


def weights(d, slots, g):
    def block(n, inter):
        return torch.randn(n, 3 * inter * d.hidden, generator=g, device="cuda").mul_(0.05).bfloat16() \
            if inter else None

    return block(slots, d.inter), block(1, d.shared_inter), block(1, d.draft_inter)


@pytest.mark.parametrize("T", [1, 9, 64])
def test_the_plain_buffers_are_enough(T):
    require_gpu()
    d = desc(H=520, N=16, k=4, I=136, Is=264, Id=136)
    g = torch.Generator(device="cuda").manual_seed(T)
    routed, shared, draft = weights(d, d.n_experts, g)
    tab = de.make_table(routed, de.expert_bytes(de.DE_BF16, d.inter, d.hidden), None, d.n_experts)
    x = torch.randn(T, d.hidden, generator=g, device="cuda")
    router = torch.randn(d.n_experts, d.hidden, generator=g, device="cuda")
    full = de.workspace(d, T)
    need = plain(d, T)
    # What follows the scratch stays untouched.
    store = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    ws = store[:need]
    de.de_workspace_init(ws)

    def both(w):
        y = [torch.empty_like(x) for _ in range(2)]
        de.de_verify_layer(d, T, x, router, None, tab, shared, y[0], ws=w)
        de.de_draft_layer(d, T, x, router, None, tab, shared, draft, 0.5, y[1], None, None, w)
        return y

    want, got = both(full), both(ws)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    assert (store[need:] == 0x5A).all()
    with pytest.raises(de.DEError) as e:
        both(store[:need - 256])
    assert e.value.code == -4


def test_noalloc_serves_what_its_scratch_holds():
    """A shape whose scratch with the words that a drafted position's launch once
    kept there (2 H + 2 N + Is + Id + I four-byte words) just fits the array."""
    require_gpu()
    T, room = 64, de.de_noalloc_scratch_bytes()

    def with_words(Is):
        d = desc(H=64, N=32, k=32, I=1888, Is=Is, Id=0)
        return d, plain(d, T) + up256((d.shared_inter + d.inter) * 4 + (d.hidden + d.n_experts) * 8)

    Is = max(i for i in range(8, 4096, 8) if with_words(i)[1] <= room)
    d, size = with_words(Is)
    assert room - size < 4096
    g = torch.Generator(device="cuda").manual_seed(1)
    routed, shared, _ = weights(d, 1, g)
    slots = torch.zeros(d.n_experts, dtype=torch.int32, device="cuda")
    tab = de.make_table(routed, de.expert_bytes(de.DE_BF16, d.inter, d.hidden), slots, 1)
    x = torch.randn(T, d.hidden, generator=g, device="cuda")
    router = torch.randn(d.n_experts, d.hidden, generator=g, device="cuda")
    y = [torch.empty_like(x) for _ in range(2)]
    de.de_verify_layer(d, T, x, router, None, tab, shared, y[0], ws=de.workspace(d, T))
    de.de_verify_layer_noalloc(d, T, x, router, None, tab, shared, y[1])
    torch.cuda.synchronize()
    assert torch.isfinite(y[0]).all() and torch.equal(y[0], y[1])


@pytest.mark.parametrize("T,H,I", [(1, 8, 8), (9, 520, 10944), (17, 2048, 10944), (3, 64, 16384),
                                   (2, 2056, 1000)])
def test_dense_layer_with_three_partials(T, H, I):
    """Scratch for three partials gives the bits of scratch for all of them."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(T + I)
    x = torch.randn(T, H, generator=g, device="cuda")
    w = (torch.randn(3 * I * H, generator=g, device="cuda") * 0.05).bfloat16()
    least = up256(4 * T * I) + 3 * up256(4 * T * H)
    full = de.de_dense_workspace_bytes(T, H, I)
    assert full >= least
    out = []
    for n in (full, least, least + up256(4 * T * H)):
        store = torch.full((n + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        y, normed = torch.empty_like(x), torch.empty_like(x)
        de.de_dense_swiglu(T, H, I, de.DE_BF16, x, w, y, store[:n],
                           epi=de.make_epilogue(x, normed, 1e-6))
        torch.cuda.synchronize()
        assert (store[n:] == 0x5A).all()
        out.append((y, normed))
    assert torch.isfinite(out[0][0]).all()
    for o in out[1:]:
        assert torch.equal(o[0], out[0][0]) and torch.equal(o[1], out[0][1])
    with pytest.raises(de.DEError) as e:
        de.de_dense_swiglu(T, H, I, de.DE_BF16, x, w, y, store[:least - 256])
    assert e.value.code == -4
