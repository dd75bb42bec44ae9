"""Items of the bf16 attention that are cut into 2, 4 and 8 key chunks, and the arrival counters behind them: several problems alternate on
one context, half of the launches beside a stream of HBM traffic, and each result must be the bits of the problem's first run."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2410_12876_amd as ag
import workloads as W
from gpu_util import DEV, dev, ensure_built, make_ctx, new_cache

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


class Traffic:
    """A side stream that reads and writes 64 MiB over and over while the call under test runs."""

    def __init__(self):
        self.side = torch.cuda.Stream()
        self.junk = torch.empty(64 << 20, dtype=torch.uint8, device=DEV)

    def beside(self, fn, load):
        if load:
            self.side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(self.side):
                for _ in range(4):
                    self.junk.add_(1)
        fn()
        torch.cuda.current_stream().wait_stream(self.side)
        torch.cuda.synchronize()


@pytest.mark.parametrize("Hq,Hkv,L,D,n_recent", [(4, 4, 4096, 128, 1), (1, 1, 4500, 128, 1), (2, 2, 4500, 128, 1), (8, 2, 4096, 128, 1),
                                                 (4, 4, 4096, 64, 1), (2, 2, 4500, 64, 1), (2, 2, 4500, 64, 16), (4, 4, 4096, 128, 10)])
def test_items_of_4_and_8_chunks_are_reproducible_beside_traffic(Hq, Hkv, L, D, n_recent):
    g = np.random.default_rng(L + Hq + D)
    sets = []
    for s in range(2):
        q, k, v = (dev(W.store(g.standard_normal((1, h, L, D)).astype(np.float32) * (1.0 + s), "bf16")) for h in (Hq, Hkv, Hkv))
        keep = np.linspace(0.95, 0.6, Hkv)[None, :, None]
        sets.append((q, k, v, dev((g.random((1, Hkv, L)) < keep).astype(np.uint8))))
    ro = oracle.slab_row_off(Hkv, L)
    ctx = make_ctx(1, L, Hq, Hkv, D, ag.AG_BF16)
    traffic = Traffic()

    def run(s, load):
        q, k, v, flags = sets[s]
        cache = new_cache(1, Hkv, D, torch.bfloat16, ro)
        out = torch.full_like(q, float("nan"))
        traffic.beside(lambda: ag.ag_compact_prefill_attn(ctx, q, k, v, flags, 1.0 / math.sqrt(D), 0, cache, out, n_recent=n_recent), load)
        return out

    base = [run(0, False), run(1, False)]
    assert all(torch.isfinite(b).all() for b in base)
    for it in range(24):
        assert torch.equal(run(it % 2, it % 4 >= 2), base[it % 2]), it
    ctx.poll_error()
    ctx.close()


class GateModule:
    def __init__(self, B, L, hp, seed):
        g = np.random.default_rng(seed)
        d, H = 64, 8
        self.hp, self.bytes = hp, ag.gate_mha_workspace_bytes(B, L, d, hp, 128, H)
        self.x = dev(W.store(g.standard_normal((B, L, d)).astype(np.float32), "bf16"))
        self.w = dev(W.store((g.standard_normal((d, 3 * hp * 128)) / 4.0).astype(np.float32), "bf16"))
        self.w_o = dev(W.store((g.standard_normal((hp * 128, H)) / math.sqrt(hp * 128)).astype(np.float32), "bf16"))
        self.bias = torch.zeros(H, device=DEV)
        self.logits = torch.empty(B, L, H, device=DEV)
        self.flags = torch.empty(B, H, L, dtype=torch.uint8, device=DEV)

    def call(self, ctx):
        ag.ag_gate_mha(ctx, self.x, self.w, self.hp, 128, self.w_o, self.bias, 0.5, 0, self.logits, self.flags)

    def clear(self):
        self.logits.fill_(float("nan"))
        self.flags.fill_(255)

    def result(self):
        return self.logits.clone(), self.flags.clone()


def _alone(p):
    """the bits of the problem's first call, on a context of its own"""
    ctx = ag.Context(0, p.bytes)
    p.call(ctx)
    torch.cuda.synchronize()
    ctx.poll_error()
    ctx.close()
    want = p.result()
    assert torch.isfinite(want[0]).all()
    return want


def _modules():
    # uncut; 2 chunks an item; 4; 8; two sequences in 4; another one in 8, whose items have the counters of the others
    return [GateModule(B, L, hp, 7 + i) for i, (B, L, hp) in
            enumerate([(1, 1000, 4), (1, 1500, 8), (1, 4096, 4), (1, 4500, 1), (2, 2900, 2), (1, 8000, 1)])]


def test_gate_module_leaves_its_arrival_counters_at_zero():
    """The counters of the cut items live in the context and each launch has to find them at zero: calls of different sizes, whose items share
    counters, follow each other on one context."""
    modules = _modules()
    want = [_alone(p) for p in modules]
    ctx = ag.Context(0, max(p.bytes for p in modules))
    traffic = Traffic()
    order = np.random.default_rng(5)
    for it in range(10):
        for i in order.permutation(len(modules)):
            p = modules[i]
            p.clear()
            traffic.beside(lambda: p.call(ctx), it % 2 == 1)
            got = p.result()
            assert torch.equal(got[0], want[i][0]) and torch.equal(got[1], want[i][1]), (it, int(i))
    ctx.poll_error()
    ctx.close()


def test_gate_module_replayed_from_a_graph_among_eager_calls():
    modules = _modules()
    want = [_alone(p) for p in modules]
    ctx = ag.Context(0, max(p.bytes for p in modules))
    in_graph = modules[2]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        in_graph.call(ctx)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            in_graph.call(ctx)
        for it in range(8):
            in_graph.clear()
            graph.replay()
            stream.synchronize()
            got = in_graph.result()
            assert torch.equal(got[0], want[2][0]) and torch.equal(got[1], want[2][1]), it
            i = (1, 3, 4, 5)[it % 4]
            modules[i].clear()
            modules[i].call(ctx)
            stream.synchronize()
            got = modules[i].result()
            assert torch.equal(got[0], want[i][0]) and torch.equal(got[1], want[i][1]), (it, i)
    ctx.poll_error()
    ctx.close()
