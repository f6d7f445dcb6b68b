"""Top-k selection and the block union at the edges of the lanes' candidate
counts (64 experts per candidate), with tied, infinite and NaN keys, on the GPU:
the routing call and the lists that a layer call's prologue builds.

x is one-hot, so a router column is the position's logits exactly.
"""
import numpy as np
import pytest
import torch

import paper_2607_24434_amd as de

from gpu_support import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def logits(T, N, seed):
    z = np.random.default_rng(seed).integers(-6, 7, size=(T, N)).astype(np.float32) / 2
    z[0, :] = 1.0  # all tied
    return z       # many ties elsewhere


def ordered(z, k):
    return np.argsort(-z, axis=1, kind="stable")[:, :k]


@pytest.mark.parametrize("T,N,k,wdtype", [
    (1, 1, 1, "bf16"), (2, 63, 6, "f32"), (8, 64, 32, "bf16"), (9, 65, 8, "bf16"),
    (17, 64, 6, "bf16"), (33, 200, 7, "f32"), (64, 256, 32, "bf16"), (64, 256, 32, "f32")])
@pytest.mark.parametrize("norm", [False, True])
def test_lists_follow_the_stable_order(T, N, k, wdtype, norm):
    H = I = 64
    z = logits(T, N, T + N)
    want = ordered(z, k)
    x = torch.zeros(T, H)
    x[torch.arange(T), torch.arange(T) % H] = 1.0
    router = torch.zeros(N, H)
    router[:, :T] = torch.from_numpy(z).t()
    x, w = x.cuda(), router.cuda()
    d = de.make_desc(H, N, k, I, 0, 0, de.DE_SOFTMAX, norm, 1.0,
                     de.DE_F32 if wdtype == "f32" else de.DE_BF16)
    idx = torch.empty(T, k, dtype=torch.int32, device="cuda")
    gate = torch.empty(T, k, device="cuda")
    ws = de.workspace(d, T)
    de.de_route_topk(d, T, x, w, None, idx, gate, ws)
    np.testing.assert_array_equal(idx.cpu().numpy(), want)
    e = np.exp(z.astype(np.float64) - z.max(1, keepdims=True))
    p = np.take_along_axis(e / e.sum(1, keepdims=True), want, 1)
    if norm:
        p = p / p.sum(1, keepdims=True)
    np.testing.assert_allclose(gate.cpu().numpy(), p, rtol=2e-6)  # sums of up to 256 fp32 terms
    # The layer call's own selection, union and lists.
    dt = torch.float32 if wdtype == "f32" else torch.bfloat16
    blocks = torch.zeros(N, 3 * I * H, dtype=dt, device="cuda")
    tab = de.make_table(blocks, 3 * I * H * blocks.element_size(), None, N)
    y = torch.empty_like(x)

    def i32(*s):
        return torch.empty(*s, dtype=torch.int32, device="cuda")

    idx2, gate2, nu, uids, offs = i32(T, k), torch.empty_like(gate), i32(1), i32(N), i32(N + 1)
    tok, gl, pp = i32(T * k), torch.empty(T * k, device="cuda"), i32(T, k)
    de.de_verify_layer(d, T, x, w, None, tab, None, y, idx2, gate2, nu, uids, offs, tok, gl, pp,
                       ws=ws)
    assert torch.equal(idx2, idx) and torch.equal(gate2, gate)
    members = np.unique(want)
    n = int(nu.item())
    assert n == len(members)
    np.testing.assert_array_equal(uids.cpu().numpy()[:n], members)
    np.testing.assert_array_equal(uids.cpu().numpy()[n:], -1)
    lists = [np.nonzero((want == m).any(1))[0] for m in members]
    np.testing.assert_array_equal(tok.cpu().numpy(), np.concatenate(lists))
    np.testing.assert_array_equal(offs.cpu().numpy()[:n + 1],
                                  np.cumsum([0] + [len(v) for v in lists]))
    g, q = gate.cpu().numpy(), pp.cpu().numpy()
    for t in range(T):
        for j in range(k):
            assert gl[q[t, j]].item() == g[t, j] and tok[q[t, j]].item() == t


def test_infinite_and_nan_keys():
    """Keys through the selection bias: NaN counts as -inf, ties go to the
    lower id, also among infinities."""
    N, k = 70, 8
    b = np.zeros(N, np.float32)
    b[[3, 66]] = np.inf
    b[[0, 5]] = np.nan
    b[[1, 69]] = -np.inf
    b[10] = -0.0
    d = de.make_desc(8, N, k, 8, 0, 0, de.DE_SIGMOID, False, 1.0, de.DE_BF16)
    x, w = torch.zeros(1, 8, device="cuda"), torch.zeros(N, 8, device="cuda")
    idx = torch.empty(1, k, dtype=torch.int32, device="cuda")
    gate = torch.empty(1, k, device="cuda")
    de.de_route_topk(d, 1, x, w, torch.from_numpy(b).cuda(), idx, gate, de.workspace(d, 1))
    assert idx[0].cpu().tolist() == [3, 66, 2, 4, 6, 7, 8, 9]
    assert torch.equal(gate, torch.full_like(gate, 0.5))
