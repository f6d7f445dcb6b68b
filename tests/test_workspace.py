"""What the scratch of a layer call holds (host only)."""
import pytest

import paper_2607_24434_amd as de


def up256(v):
    return (v + 255) & ~255


def desc(H=2048, N=64, k=6, I=1408, Is=2816, Id=1408, dt=de.DE_BF16):
    return de.make_desc(H, N, k, I, Is, Id, de.DE_SOFTMAX, 0, 1.0, dt)


SHAPES = dict(v2_lite=dict(), no_draft=dict(Id=0), no_shared=dict(Is=0), q4=dict(dt=de.DE_Q4_0),
              small=dict(H=520, N=256, k=2, I=128, Is=0, Id=128), f32=dict(dt=de.DE_F32),
              many=dict(N=256, k=32, Is=0, Id=0), wide=dict(H=4096, I=2560))


def plain(d, T):
    """The control area and the plain buffers of a layer call."""
    H, N, k, I, Is, Id = (d.hidden, d.n_experts, d.top_k, d.inter, d.shared_inter, d.draft_inter)
    buffers = [T * N * 4, T * k * 4, T * k * 4, 4, N * 4, (N + 1) * 4, T * k * 4, T * k * 4,
               T * k * 4, T * k * I * 4, T * Is * 4, T * Id * 4, T * k * H * 4, 3 * T * H * 4,
               T * H * 4]
    return 4096 + sum(up256(b) for b in buffers)


def tagged(d, T):
    """Room for a single-launch verify layer's values as words of eight bytes."""
    k = T * d.top_k
    return up256((k * (d.inter + d.hidden) + T * d.shared_inter + 3 * T * d.hidden) * 8)


@pytest.mark.parametrize("kw", SHAPES.values(), ids=SHAPES.keys())
def test_a_layer_call_holds_its_own_values_and_no_polled_words(kw):
    """The words that the blocks of a drafted position's launch poll (arrival
    flags, tagged logits and rows) are not in the workspace, where the buffers of
    a call of another shape or without the draft block could lie over them and
    pass for them: its bytes are the control area and the plain buffers, and for
    the shapes of the single-launch verify layer the room that is reported with
    them."""
    d = desc(**kw)
    for T in (1, 2, 9, 10, 64):
        one_launch = d.wdtype == de.DE_BF16 and 2 <= T <= 9 and max(d.hidden, d.inter) <= 2048
        want = plain(d, T) + (tagged(d, T) if one_launch else 0)
        assert de.de_workspace_bytes(d, T) == want, T


FAKE = 0x10000


@pytest.mark.parametrize("kw", SHAPES.values(), ids=SHAPES.keys())
@pytest.mark.parametrize("dense", [0, 10944])
def test_a_model_workspace_is_no_larger_than_with_a_scratch_for_each_layer(kw, dense):
    """A workspace that held the dense layer's scratch (three partials) beside the
    MoE layers' (with the words that a drafted position's launch polled) serves."""
    d = desc(**kw)
    V, H = 102400, d.hidden
    layer = dict(w_router=FAKE, bias=None, table=de.make_table(FAKE, 1 << 28, None, d.n_experts),
                 shared_w=FAKE if d.shared_inter else None,
                 draft_w=FAKE if d.draft_inter else None, gamma=1.0)
    m = de.make_model(d, [dict(layer) for _ in range(3)], vocab=V, emb=FAKE, lm_head=FAKE,
                      dense_w=FAKE if dense else None, dense_inter=dense)
    words = (d.shared_inter + d.draft_inter + d.inter) * 4 + (H + d.n_experts) * 8
    for T in (1, 2, 9, 64):
        old = [de.de_accept_workspace_bytes(63, V), plain(d, T) + up256(words),
               up256(T * dense * 4) + 3 * up256(T * H * 4) if dense else 0, 8, 64 * d.top_k * 4,
               64 * d.top_k * 4, T * H * 4, T * H * 4, T * H * 4, T * H * 4, T * V * 4,
               3 * ((d.n_experts + 63) // 64) * 8, 20, 3 * T * d.n_experts * 4,
               3 * T * d.n_experts * 4, T * V * 4]
        assert 0 < de.de_model_workspace_bytes(m, T) <= sum(up256(b) for b in old), T
