"""GPU chunk importance where several workgroups share a chunk: vector counts
at the least a split chunk has, not divisible by the workgroups, the most
workgroups a chunk is given, chunk counts on both sides of the rule, and repeated
calls (each starts on what the last one left in the meeting place) on one and
on two streams at once.  Against the oracle at relative 1e-12 (64-bit sums in
another order); repeated calls, and calls with other chunks beside, give the
same bits."""
import sys

import numpy as np
import pytest
import torch

from oracle import importance as oimp

pytestmark = pytest.mark.gpu

SHAPES = [  # (chunks, layers, kv heads, head dim, dtype): a round of 128 vectors per layer and head
    (1, 8, 1, 64, np.float32),     # 8 rounds: one workgroup
    (1, 15, 1, 128, np.float64),   # the most that are never split
    (1, 16, 1, 64, np.float32),    # 4 workgroups of 4 rounds
    (1, 36, 2, 64, np.float32),    # 16 workgroups of 4 or 5 rounds
    (3, 17, 1, 128, np.float64),   # 17 rounds over 4 workgroups
    (40, 17, 1, 128, np.float64),  # 17 rounds over 2 workgroups
    (3, 11, 1, 128, np.float64),
    (40, 7, 2, 64, np.float32),
    (256, 4, 2, 64, np.float32),
    (257, 4, 2, 64, np.float32),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"P{s[0]}_L{s[1]}_H{s[2]}_d{s[3]}_{np.dtype(s[4]).name}")
def test_importance_split(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    P, L, H, d, dt = shape
    print(f"[importance-split] P={P} L={L} H={H} d={d} {np.dtype(dt).name}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(P * 1000 + L * 10 + H)
    keys = [(rng.standard_normal((P, L, H, 128, d)) * (1 + i)).astype(dt) for i in range(2)]
    kin = [torch.from_numpy(k).cuda() for k in keys]
    pool = kvb.pool_layout(L, H, d, 8, 128, d)
    kdt = kvb.KVB_F64 if dt == np.float64 else kvb.KVB_F32
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    out = [torch.zeros((4, P + (P & 1)), dtype=torch.float64, device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    for i in range(4):                      # interleaved on two streams
        for j, st in enumerate(streams):
            kvb.kvb_chunk_importance(pool, P, L, kdt, kin[j], out[j][i], st.cuda_stream)
    torch.cuda.synchronize()
    for j in range(2):
        g = out[j].cpu().numpy()[:, :P]
        np.testing.assert_allclose(g[0], oimp.chunk_importance(keys[j]), rtol=1e-12, atol=0)
        for i in range(1, 4):
            assert np.array_equal(g[i].view(np.uint64), g[0].view(np.uint64)), "not deterministic"
    # a call adds its share to what is there
    kvb.kvb_chunk_importance(pool, P, L, kdt, kin[1], out[0][0])
    torch.cuda.synchronize()
    got, a, b = (x.cpu().numpy()[:P] for x in (out[0][0], out[0][1], out[1][1]))
    assert np.array_equal(got, a + b)


@pytest.mark.parametrize("dt", [np.float32, np.float64], ids=lambda t: np.dtype(t).name)
def test_importance_same_bits_in_any_batch(dt):
    """A chunk's importance does not depend on the chunks beside it: alone, and in
    launches that give a chunk nine workgroups and fewer, down to one."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    L, H, d, P = 36, 1, 64, 257
    print(f"[importance-batch] {np.dtype(dt).name}", file=sys.stderr, flush=True)
    g = torch.Generator("cuda").manual_seed(3)
    keys = torch.randn((P, L, H, 128, d), generator=g, device="cuda", dtype=torch.float64)
    keys = (keys * torch.exp(torch.randn((P, 1, 1, 1, d), generator=g, device="cuda"))).to(
        torch.float64 if dt == np.float64 else torch.float32)
    pool = kvb.pool_layout(L, H, d, 8, 128, d)
    kdt = kvb.KVB_F64 if dt == np.float64 else kvb.KVB_F32

    def run(n):
        out = torch.zeros(n + (n & 1), dtype=torch.float64, device="cuda")
        kvb.kvb_chunk_importance(pool, n, L, kdt, keys[:n].contiguous(), out)
        torch.cuda.synchronize()
        return out.cpu().numpy()[:n]

    alone = run(1)
    whole = run(P)
    np.testing.assert_allclose(whole[:2], oimp.chunk_importance(keys[:2].cpu().numpy()), rtol=1e-12)
    for n in (1, 2, 5, 10, 20, 30, 42, 73, 256):
        assert np.array_equal(run(n).view(np.uint64), whole[:n].view(np.uint64)), n
    assert alone[0] == whole[0]


def test_importance_after_unordered_calls():
    """Calls that add to one address at the same time may lose a share, but leave
    nothing behind: the ordered calls that follow are exact, also after more of
    them than a chunk index has meeting places."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    L, H, d = 36, 1, 64
    print("[importance-unordered] 2 streams", file=sys.stderr, flush=True)
    rng = np.random.default_rng(5)
    k = rng.standard_normal((1, L, H, 128, d)).astype(np.float32)
    few = [torch.from_numpy(np.ascontiguousarray(k[:, :n])).cuda() for n in (36, 16, 20)]
    pool = kvb.pool_layout(L, H, d, 8, 128, d)
    out = torch.zeros(2, dtype=torch.float64, device="cuda")
    ref = torch.zeros(2, dtype=torch.float64, device="cuda")
    kvb.kvb_chunk_importance(pool, 1, L, kvb.KVB_F32, few[0], ref)
    streams = [torch.cuda.Stream() for _ in few]
    torch.cuda.synchronize()
    for _ in range(100):  # 9, 4 and 5 workgroups a chunk
        for t, st in zip(few, streams):
            kvb.kvb_chunk_importance(pool, 1, t.shape[1], kvb.KVB_F32, t, out, st.cuda_stream)
    torch.cuda.synchronize()
    for t in few:
        out.zero_()
        kvb.kvb_chunk_importance(pool, 1, t.shape[1], kvb.KVB_F32, t, out)
        torch.cuda.synchronize()
        n = t.shape[1]
        want = oimp.chunk_importance(k[:, :n])[0] * n / L
        np.testing.assert_allclose(out.cpu().numpy()[0], want, rtol=1e-12, atol=0)
        if n == L:
            assert out[0] == ref[0]


def test_importance_graph_replays():
    """Captured calls with chunks dealt to several workgroups, replayed one after
    another and two graphs at once on two streams, give the eager bits."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    P, L, H, d = 6, 36, 1, 64
    print("[importance-graph] 2 graphs", file=sys.stderr, flush=True)
    pool = kvb.pool_layout(L, H, d, 8, 128, d)
    g = torch.Generator("cuda").manual_seed(11)
    keys = [torch.randn((P, L, H, 128, d), generator=g, device="cuda") for _ in range(2)]
    outs = [torch.zeros(P, dtype=torch.float64, device="cuda") for _ in range(2)]
    refs = [torch.zeros(P, dtype=torch.float64, device="cuda") for _ in range(2)]
    for k, r in zip(keys, refs):
        kvb.kvb_chunk_importance(pool, P, L, kvb.KVB_F32, k, r)
    torch.cuda.synchronize()
    graphs, streams = [], [torch.cuda.Stream(), torch.cuda.Stream()]
    for k, o in zip(keys, outs):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            o.zero_()
            kvb.kvb_chunk_importance(pool, P, L, kvb.KVB_F32, k, o)
        graphs.append(graph)
    torch.cuda.synchronize()
    for r in range(5):
        for graph, st in zip(graphs, streams):
            with torch.cuda.stream(st):
                for _ in range(1 + r):
                    graph.replay()
        torch.cuda.synchronize()
        for o, ref in zip(outs, refs):
            assert torch.equal(o, ref), r
            o.fill_(-1.0)
        torch.cuda.synchronize()
