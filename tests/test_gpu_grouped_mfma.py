"""The grouped passes on the matrix cores (bf16 and Q4_0 weights) against the
vector-ALU passes of the same layer with the same weights held as fp32, on the
GPU.

The matrix-core layer splits each fp32 activation exactly into three bf16
parts, so both layers form the same exact products (Q4_0: of codes, scaled once
per block) and differ only in the order of fp32 sums: a 2-norm error of sqrt(terms) 2^-24 per pass, 2.7e-6 at 2048 terms.
Sizes: the edges of the 16-position slices and of the 16-row tiles, columns
that are not whole steps of 32, fewer rows than a tile, shared and dense
reductions whose last chunk is narrower, a single column unit.
"""
import pytest
import torch

import paper_2607_24434_amd as de

from gpu_support import require_gpu

pytestmark = pytest.mark.gpu

TOL = 3e-6


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def rel(a, b):
    return ((a.double() - b.double()).norm() / b.double().norm()).item()


def layer(T, H, N, k, I, Is, x, w, router, dt, kind="verify", slots=None):
    """One layer call; w: (routed [N, 3 I H], shared, draft) in bf16, or their
    Q4_0 blocks."""
    d = de.make_desc(H, N, k, I, Is, I, de.DE_SOFTMAX, True, 1.0, dt)
    routed, shared, draft = [t.float() if t is not None and dt == de.DE_F32 else t for t in w]
    tab = de.make_table(routed, de.expert_bytes(dt, I, H), slots, N)
    y, normed = torch.empty_like(x), torch.empty_like(x)
    epi = de.make_epilogue(x, normed, 1e-6)
    idx = torch.empty(T, k, dtype=torch.int32, device="cuda")
    ws = de.workspace(d, T)
    if kind == "verify":
        de.de_verify_layer(d, T, x, router, None, tab, shared, y, topk_idx=idx, ws=ws, epi=epi)
    else:
        de.de_draft_layer_topr(d, T, x, router, None, tab, shared, draft, 0.5, 1, y, idx, None, ws,
                               epi=epi)
    return y - x, normed, idx, de.de_layer_status(ws)


def inputs(T, H, N, I, Is, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def r(*s):
        return torch.randn(*s, generator=g, device="cuda")

    w = ((0.05 * r(N, 3 * I * H)).bfloat16(),
         (0.05 * r(3 * Is * H)).bfloat16() if Is else None, (0.05 * r(3 * I * H)).bfloat16())
    # A wide spread of magnitudes, so that all three parts of the split matter.
    x = r(T, H) * torch.exp2(8 * torch.rand(T, H, generator=g, device="cuda") - 4)
    return x, w, 0.1 * r(N, H)


@pytest.mark.parametrize("T,H,N,k,I,Is", [
    (2, 8, 4, 2, 8, 8), (16, 72, 5, 3, 24, 40), (17, 264, 6, 6, 136, 0), (5, 520, 8, 2, 16, 296),
    (33, 1000, 3, 2, 72, 144), (64, 512, 4, 4, 128, 256), (9, 2048, 16, 6, 1408, 2816),
    (32, 2048, 4, 1, 40, 2048 + 1032), (64, 2048, 256, 32, 16, 0)])
@pytest.mark.parametrize("kind", ["verify", "draft"])
def test_layer_matches_the_vector_alu_path(T, H, N, k, I, Is, kind):
    x, w, router = inputs(T, H, N, I, Is, T + H)
    print(kind, T, H, N, k, I, Is, flush=True)
    a = layer(T, H, N, k, I, Is, x, w, router, de.DE_BF16, kind)
    b = layer(T, H, N, k, I, Is, x, w, router, de.DE_F32, kind)
    assert torch.equal(a[2], b[2]) and a[3] == b[3] == 0
    assert rel(a[0], b[0]) < TOL and rel(a[1], b[1]) < TOL


def q4_blocks(w, n, inter, hidden):
    """The Q4_0 block [G|U|D] of each of the n experts in w, and the same weights
    as fp32."""
    out, back = [], []
    for m in w.float().view(n, 3, inter * hidden).unbind(1):
        b = m.view(n, -1, 32)
        d = (b.gather(2, b.abs().argmax(dim=2, keepdim=True)) / -8.0).half()
        q = (b / d.float() + 8.5).floor().clamp(0, 15)
        c = q.to(torch.uint8)
        codes = (c[:, :, :16] | (c[:, :, 16:] << 4)).reshape(n, -1)
        out += [codes, d.reshape(n, -1).view(torch.uint8)]
        back.append(((q - 8.0) * d.float()).view(n, -1))
    return torch.cat(out, 1).contiguous(), torch.cat(back, 1).contiguous()


@pytest.mark.parametrize("T,H,N,k,I,Is", [
    (2, 32, 4, 2, 32, 32), (16, 96, 5, 3, 64, 160), (17, 288, 6, 6, 160, 0), (5, 544, 8, 2, 32, 608),
    (64, 512, 4, 4, 128, 256), (9, 2048, 16, 6, 1408, 2816), (33, 1024, 3, 2, 64, 2048 + 1056),
    (2, 2048, 16, 6, 1408, 2816), (2, 1056, 8, 1, 64, 0), (2, 2048, 8, 7, 96, 64),
    (2, 1024, 8, 2, 96, 64)])
@pytest.mark.parametrize("kind", ["verify", "draft"])
def test_q4_layer_matches_the_vector_alu_path(T, H, N, k, I, Is, kind):
    x, w, router = inputs(T, H, N, I, Is, T + H)
    print(kind, T, H, N, k, I, Is, flush=True)
    q, f = [], []
    for t, n, i in ((w[0], N, I), (w[1], 1, Is), (w[2], 1, I)):
        b = q4_blocks(t.view(n, -1), n, i, H) if t is not None else (None, None)
        q.append(b[0])
        f.append(b[1])
    a = layer(T, H, N, k, I, Is, x, q, router, de.DE_Q4_0, kind)
    b = layer(T, H, N, k, I, Is, x, f, router, de.DE_F32, kind)
    assert torch.equal(a[2], b[2]) and a[3] == b[3] == 0
    assert rel(a[0], b[0]) < TOL and rel(a[1], b[1]) < TOL


def test_a_position_that_is_not_finite_stays_alone():
    T, H, N, k, I = 18, 136, 4, 4, 40
    x, w, router = inputs(T, H, N, I, I, 3)
    clean = layer(T, H, N, k, I, I, x, w, router, de.DE_BF16)[0]
    x2 = x.clone()
    x2[1, 5] = float("inf")
    x2[17, 100] = float("nan")
    got = layer(T, H, N, k, I, I, x2, w, router, de.DE_BF16)[0]
    rest = [t for t in range(T) if t not in (1, 17)]
    assert torch.equal(got[rest], clean[rest])
    assert not torch.isfinite(got[[1, 17]]).any()


def test_missing_expert_drops_out_and_is_reported():
    T, H, N, k, I = 20, 264, 4, 4, 40
    x, w, router = inputs(T, H, N, I, I, 4)
    slots = torch.tensor([0, 1, -1, 3], dtype=torch.int32, device="cuda")
    a = layer(T, H, N, k, I, I, x, w, router, de.DE_BF16, slots=slots)
    b = layer(T, H, N, k, I, I, x, w, router, de.DE_F32, slots=slots)
    assert a[3] == b[3] == -5
    assert rel(a[0], b[0]) < TOL


@pytest.mark.parametrize("T,H,I", [(1, 8, 8), (9, 520, 1000), (17, 2048, 10944), (40, 256, 16384),
                                   (3, 64, 16392)])
def test_dense_layer(T, H, I):
    x, w, _ = inputs(T, H, 1, I, 0, T + I)
    out = []
    for dt, wt in ((de.DE_BF16, torch.bfloat16), (de.DE_F32, torch.float32)):
        y = torch.empty_like(x)
        ws = torch.empty(de.de_dense_workspace_bytes(T, H, I), dtype=torch.uint8, device="cuda")
        de.de_dense_swiglu(T, H, I, dt, x, w[0][0].to(wt), y, ws)
        out.append(y)
    assert rel(out[0], out[1]) < 3 * TOL  # the down pass sums up to 16392 terms


@pytest.mark.parametrize("T,H,V", [(1, 8, 1), (2, 40, 17), (16, 1000, 1003), (17, 2048, 33),
                                   (64, 264, 8193)])
def test_lm_head(T, H, V):
    g = torch.Generator(device="cuda").manual_seed(V)
    # Whole numbers: every product and sum is exact.
    x = torch.randint(-512, 513, (T, H), generator=g, device="cuda").float()
    w = torch.randint(-8, 9, (V, H), generator=g, device="cuda").bfloat16()
    out = torch.empty(T, V, device="cuda")
    de.de_lm_head(T, H, V, x, w, out)
    assert torch.equal(out.double(), x.double() @ w.double().t())


@pytest.mark.parametrize("dt", [de.DE_BF16, de.DE_Q4_0], ids=["bf16", "q4"])
def test_lists_that_overlap_stay_in_bounds(dt):
    """Offsets that no union has (every second member owns all T k entries) make
    eight times the slices a block has room for: those past it are dropped.  With
    equal experts the members that remain write what one member would."""
    T, H, N, k, I = 64, 288, 64, 6, 160
    x, w, _ = inputs(T, H, 1, I, 0, 9)
    blk = w[0] if dt == de.DE_BF16 else q4_blocks(w[0], 1, I, H)[0]
    d = de.make_desc(H, N, k, I, 0, 0, de.DE_SOFTMAX, False, 1.0, dt)
    tab = de.make_table(blk.expand(N, -1).contiguous(), de.expert_bytes(dt, I, H), None, N)

    def i32(*v):
        return torch.tensor(v, dtype=torch.int32, device="cuda")

    pos = torch.arange(T * k, dtype=torch.int32, device="cuda")
    tok, ppos = (pos // k).contiguous(), pos.view(T, k)
    gate = torch.rand(T * k, generator=torch.Generator().manual_seed(1)).cuda()
    ws = de.workspace(d, T)
    out = []
    for n, offs in ((1, [0] + [T * k] * N), (N, [0, T * k] * (N // 2) + [0])):
        y = torch.empty_like(x)
        de.de_grouped_swiglu(d, T, x, tab, i32(n), i32(*range(N)), i32(*offs), tok, gate, ppos,
                             None, y, ws)
        torch.cuda.synchronize()
        assert de.de_layer_status(ws) == 0
        out.append(y)
    assert torch.isfinite(out[0]).all() and torch.equal(out[0], out[1])
