"""GPU chunk importance where several workgroups share a chunk: vector counts
at the least a slice takes, not divisible by the slices, the most slices a
chunk is given, chunk counts around the splitting rule's edges, and repeated
calls (each starts on what the last one left in the meeting place) on one and
on two streams at once.  Against the oracle at relative 1e-12 (64-bit sums in
another order); repeated calls give the same bits."""
import sys

import numpy as np
import pytest
import torch

from oracle import importance as oimp

pytestmark = pytest.mark.gpu

SHAPES = [  # (chunks, layers, kv heads, head dim, dtype): 128 * layers * heads vectors a chunk
    (1, 8, 1, 64, np.float32),     # 2 slices
    (1, 36, 2, 64, np.float32),    # 16 slices of 4 or 5 rounds
    (3, 11, 1, 128, np.float64),   # 11 rounds over 2 slices
    (40, 7, 2, 64, np.float32),    # 3 slices of 4 or 5 rounds
    (256, 4, 2, 64, np.float32),   # 2 slices, the most chunks that are split
    (257, 4, 2, 64, np.float32),   # one workgroup a chunk
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
