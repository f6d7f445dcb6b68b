"""One drafted position in the single launch, over the shapes it accepts: bf16
and Q4_0 expert weights, hidden sizes that do not fill the lanes, with and
without shared and draft experts.  The separate launches (DE_PD_SINGLE=0) do
the same fp32 operations in the same order, so every output is identical bit
for bit.  Launches on two streams at once, and under stream capture."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2607_24434_amd as de

from gpu_support import require_gpu

pytestmark = pytest.mark.gpu

# dtype, hidden, experts, top_k, inter, shared, draft, score, norm_topk
SHAPES = [
    (de.DE_Q4_0, 2048, 64, 6, 1408, 2816, 1408, de.DE_SOFTMAX, 0),
    (de.DE_Q4_0, 512, 8, 2, 32, 0, 32, de.DE_SIGMOID, 1),
    (de.DE_Q4_0, 1056, 33, 4, 160, 320, 0, de.DE_SOFTMAX, 1),
    (de.DE_Q4_0, 2016, 128, 8, 704, 1408, 704, de.DE_SIGMOID, 0),
    (de.DE_BF16, 520, 16, 2, 128, 256, 128, de.DE_SOFTMAX, 0),
    (de.DE_BF16, 1304, 60, 4, 136, 136, 0, de.DE_SIGMOID, 1),
    (de.DE_BF16, 2040, 64, 6, 1408, 2816, 1408, de.DE_SOFTMAX, 1),
]


class Layer:
    def __init__(self, shape, seed):
        require_gpu()
        dt, H, N, k, I, Is, Id, score, norm = shape
        g = torch.Generator(device="cuda").manual_seed(seed)
        self.H, self.k = H, k
        self.desc = de.make_desc(H, N, k, I, Is, Id, score, norm, 1.0, dt)

        def block(n, inter):
            if inter == 0:
                return None
            m = inter * H
            if dt == de.DE_BF16:
                return torch.randn(n, 3 * m, generator=g, device="cuda").mul_(0.02).bfloat16()
            w = torch.randint(0, 256, (n, 3, m * 9 // 16), generator=g, device="cuda",
                              dtype=torch.uint8)
            d = torch.randn(n, 3, m // 32, generator=g, device="cuda").mul_(0.005).half()
            w[:, :, m // 2:] = d.view(torch.uint8)
            return w.view(n, -1)

        self.router = torch.randn(N, H, generator=g, device="cuda") * 0.1
        self.bias = torch.randn(N, generator=g, device="cuda") * 0.1
        self.routed, self.shared, self.draft = block(N, I), block(1, Is), block(1, Id)
        self.table = de.make_table(self.routed, de.expert_bytes(dt, I, H), None, N)
        self.x = torch.randn(1, H, generator=g, device="cuda")
        self.residual = torch.randn(1, H, generator=g, device="cuda")
        self.ws = de.workspace(self.desc, 1)

    def outputs(self):
        f = dict(device="cuda")
        return [torch.zeros(1, self.H, **f), torch.zeros(1, self.H, **f),
                torch.zeros(1, self.k, dtype=torch.int32, **f), torch.zeros(1, self.k, **f)]

    def run(self, out, stream=None):
        y, normed, idx, gate = out
        de.de_draft_layer(self.desc, 1, self.x, self.router, self.bias, self.table, self.shared,
                          self.draft, 0.5, y, idx, gate, self.ws,
                          epi=de.make_epilogue(self.residual, normed, 1e-6), stream=stream)


def separate(layer, monkeypatch):
    monkeypatch.setenv("DE_PD_SINGLE", "0")
    want = layer.outputs()
    layer.run(want)
    torch.cuda.synchronize()
    monkeypatch.setenv("DE_PD_SINGLE", "1")
    return want


def same(got, want):
    return all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s[:7])))
def test_single_launch_equals_separate_launches(shape, monkeypatch):
    layer = Layer(shape, 1)
    want = separate(layer, monkeypatch)
    assert torch.isfinite(want[0]).all()
    for _ in range(3):  # later launches find the words of earlier ones
        got = layer.outputs()
        layer.run(got)
        torch.cuda.synchronize()
        assert de.de_layer_status(layer.ws) == 0
        assert same(got, want)


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[6]], ids=["q4", "bf16"])
def test_two_streams(shape, monkeypatch):
    """Calls on two streams at once: a launch never shares the chip with
    another stream's, and the outputs are the same."""
    layers = [Layer(shape, s) for s in (2, 3)]
    want = [separate(l, monkeypatch) for l in layers]
    streams = [torch.cuda.Stream() for _ in layers]
    got = [[l.outputs() for _ in range(20)] for l in layers]
    torch.cuda.synchronize()
    for i in range(20):
        for l, s, g in zip(layers, streams, got):
            l.run(g[i], stream=s)
    torch.cuda.synchronize()
    for l, g, w in zip(layers, got, want):
        assert de.de_layer_status(l.ws) == 0
        assert all(same(o, w) for o in g)


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[6]], ids=["q4", "bf16"])
def test_captured(shape, monkeypatch):
    """A captured call replays on changed inputs, with eager calls between."""
    layer = Layer(shape, 4)
    separate(layer, monkeypatch)
    graph, out, s = torch.cuda.CUDAGraph(), layer.outputs(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=s):
        layer.run(out, stream=s)
    for i in range(4):
        layer.x.normal_()
        graph.replay()
        torch.cuda.synchronize()
        want = layer.outputs()
        layer.run(want)
        torch.cuda.synchronize()
        assert same(out, want)


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[6]], ids=["q4", "bf16"])
def test_with_and_without_the_draft_block_on_one_workspace(shape, monkeypatch):
    """Calls with and without the draft block, and verify calls, in turn on one
    workspace: none finds another's values in place of a word it waits for."""
    layer = Layer(shape, 5)
    verify = layer.outputs()

    def call(draft, out):
        keep, layer.draft = layer.draft, layer.draft if draft else None
        layer.run(out)
        layer.draft = keep

    want = {}
    for draft in (True, False):
        monkeypatch.setenv("DE_PD_SINGLE", "0")
        want[draft] = layer.outputs()
        call(draft, want[draft])
        torch.cuda.synchronize()
        monkeypatch.setenv("DE_PD_SINGLE", "1")
    assert not torch.equal(want[True][0], want[False][0])
    for i in range(70):
        got = layer.outputs()
        call(i % 2 == 0, got)
        if i % 5 == 0:
            de.de_verify_layer(layer.desc, 1, layer.x, layer.router, layer.bias, layer.table,
                               layer.shared, verify[0], ws=layer.ws)
        torch.cuda.synchronize()
        assert same(got, want[i % 2 == 0]), i
    assert de.de_layer_status(layer.ws) == 0


@pytest.mark.parametrize("dt", [de.DE_Q4_0, de.DE_BF16], ids=["q4", "bf16"])
def test_blocks_without_rows_on_two_streams(dt, monkeypatch):
    """A hidden size whose rows do not reach every block (544 rows, three a block),
    on two streams at once."""
    shape = (dt, 544, 64, 4, 1408, 2816, 1408, de.DE_SOFTMAX, 0)
    layers = [Layer(shape, s) for s in (6, 7)]
    want = [separate(l, monkeypatch) for l in layers]
    streams = [torch.cuda.Stream() for _ in layers]
    got = [[l.outputs() for _ in range(40)] for l in layers]
    torch.cuda.synchronize()
    for i in range(40):
        for l, s, g in zip(layers, streams, got):
            l.run(g[i], stream=s)
            if i % 4 == 3:
                s.synchronize()  # the next call, on the other stream, may follow
    torch.cuda.synchronize()
    for l, g, w in zip(layers, got, want):
        assert de.de_layer_status(l.ws) == 0
        assert all(same(o, w) for o in g)


FIRST_CALL = """
import sys
sys.path.insert(0, "tests")
import torch
import paper_2607_24434_amd as de
from test_gpu_draft_single_launch import SHAPES, Layer

layer, out, s = Layer(SHAPES[0], 8), None, torch.cuda.Stream()
out, ev = layer.outputs(), [torch.cuda.Event(enable_timing=True) for _ in range(2)]
a, b = torch.ones(8, device="cuda"), torch.zeros(8, device="cuda")
b.copy_(a + a)
graph = torch.cuda.CUDAGraph()


def single():
    # Ran as one launch: its phase timer brackets it (the events are else in
    # reverse order).
    ev[1].record(s)
    ev[0].record(s)
    de.de_time_next_phase(de.DE_PHASE_DRAFT_PASS, ev[0], ev[1])
    layer.run(out, stream=s)


torch.cuda.synchronize()
with torch.cuda.graph(graph):
    b.copy_(a)
    single()
torch.cuda.synchronize()
assert ev[0].elapsed_time(ev[1]) > 0.002, "first call, another stream under capture"
single()
torch.cuda.synchronize()
assert ev[0].elapsed_time(ev[1]) > 0.002, "second call"
a.fill_(3.0)
graph.replay()
torch.cuda.synchronize()
assert b.tolist() == [3.0] * 8 and de.de_layer_status(layer.ws) == 0
print("ok")
"""


def test_first_call_while_another_stream_is_captured():
    """A process's first single launch, while another stream is under capture: the
    capture stays whole and the launch is not given up (a process of its own,
    since what it needs is allocated once)."""
    require_gpu()
    r = subprocess.run([sys.executable, "-c", FIRST_CALL], capture_output=True, text=True,
                       cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
