"""What the scratch of a layer call holds (host only)."""
import pytest

import paper_2607_24434_amd as de


def up256(v):
    return (v + 255) & ~255


def desc(H=2048, N=64, k=6, I=1408, Is=2816, Id=1408, dt=de.DE_BF16):
    return de.make_desc(H, N, k, I, Is, Id, de.DE_SOFTMAX, 0, 1.0, dt)


@pytest.mark.parametrize("kw", [dict(), dict(Id=0), dict(Is=0), dict(dt=de.DE_Q4_0),
                                dict(H=520, N=256, k=2, I=128, Is=0, Id=128), dict(dt=de.DE_F32)],
                         ids=["v2-lite", "no-draft", "no-shared", "q4", "small", "f32"])
def test_one_position_holds_its_own_values_and_no_polled_words(kw):
    """The words that the blocks of a drafted position's launch poll (arrival
    flags, tagged logits and rows) are not in the workspace, where the buffers of
    a call of another shape or without the draft block could lie over them and
    pass for them: its bytes are the control area and the plain buffers."""
    d = desc(**kw)
    H, N, k, I, Is, Id = (d.hidden, d.n_experts, d.top_k, d.inter, d.shared_inter, d.draft_inter)
    buffers = [N * 4, k * 4, k * 4, 4, N * 4, (N + 1) * 4, k * 4, k * 4, k * 4,  # routing, union
               k * I * 4, Is * 4, Id * 4, k * H * 4, 3 * H * 4, H * 4]           # A, partials
    assert de.de_workspace_bytes(d, 1) == 4096 + sum(up256(b) for b in buffers)
