"""GPU stitch: a launch that fills the chip (four tokens a thread) and launches
of a few chunks (one token a thread, a chunk split over workgroups) write the
same bits: caches and deviations of one call over every chunk equal those of
calls over groups of chunks, at both sides of the launch rule, for both head
sizes and widths, key groups inside and across a workgroup's tokens, and chunks
at rows that are not multiples of four.  The small launches are pinned to the
oracle by the parity tests."""
import sys

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [  # (layers, kv heads, chunks, d, bits, Gk, Gv, first row, fused, out)
    (48, 1, 33, 128, 4, 32, 32, 0, True, "bf16"),    # 1584 workgroups against 48 to 336
    (24, 2, 64, 64, 8, 128, 64, 3, True, "bf16"),    # 1536: the first that is not split
    (40, 2, 39, 128, 8, 4, 16, 1, True, "bf16"),
    (48, 2, 33, 64, 4, 16, 32, 2, True, "bf16"),
    (8, 2, 8, 128, 4, 64, 32, 1, False, "bf16"),     # 128: the first that is not split
    (16, 2, 9, 64, 8, 32, 16, 0, False, "f32"),
    (9, 2, 11, 128, 8, 8, 128, 5, False, "f32"),
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: "L%d_H%d_P%d_d%d_b%d_k%d_%s_%s" % (
    *c[:6], "fused" if c[8] else "plain", c[9]))
def test_split_launches_same_bits(c):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    L, H, P, d, bits, gk, gv, row0, fused, out = c
    print(f"[stitch-split] {c}", file=sys.stderr, flush=True)
    g = torch.Generator("cuda").manual_seed(P + d)
    T = row0 + 128 * P + 2
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    codes = [torch.randint(0, 256, (P, L, H, 128, d * bits // 8), generator=g, device="cuda",
                           dtype=torch.uint8) for _ in range(2)]
    ks, kz = rnd(P, L, H, 128 // gk, d).abs() / 64, rnd(P, L, H, 128 // gk, d)
    vs, vz = rnd(P, L, H, 128, d // gv).abs() / 64, rnd(P, L, H, 128, d // gv)
    desc = np.stack([np.arange(P), np.zeros(P), row0 + 128 * np.arange(P),
                     row0 + 128 * np.arange(P)], 1).astype(np.int32)
    chunks = torch.from_numpy(desc).cuda()
    cos, sin = (torch.from_numpy(t).cuda() for t in kvb.kvb_rope_delta_table(1e4, d, desc[:, 3]))
    fresh = rnd(L, H, T, d).bfloat16()
    pool = kvb.pool_layout(L, H, d, bits, gk, gv)
    dt, code = (torch.float32, kvb.KVB_F32) if out == "f32" else (torch.bfloat16, kvb.KVB_BF16)

    def run(groups):
        k, v = (torch.full((L, H, T, d), 7.0, dtype=dt, device="cuda") for _ in range(2))
        delta = torch.full((L, T), -7.0, device="cuda")
        for lo, hi in groups:
            a = (pool, P, codes[0], ks, kz, codes[1], vs, vz, chunks[lo:hi], hi - lo, cos[lo:hi],
                 sin[lo:hi], T)
            if fused:
                kvb.kvb_stitch_deviation(*a, k, v, fresh, delta)
            else:
                kvb.kvb_stitch(*a, code, k, v)
        torch.cuda.synchronize()
        return k, v, delta

    whole = run([(0, P)])
    parts = run([(i, min(i + 7, P)) for i in range(0, P, 7)] if fused else [(i, i + 1) for i in range(P)])
    for name, a, b in zip(("k", "v", "delta"), whole, parts):
        assert torch.equal(a, b), name
    for t in whole[:2]:
        assert torch.all(t[:, :, :row0] == 7) and torch.all(t[:, :, row0 + 128 * P:] == 7)
        assert torch.all(torch.isfinite(t))
    if fused:
        d2 = whole[2]
        assert torch.all(d2[:, :row0] == -7) and torch.all(d2[:, row0 + 128 * P:] == -7)
        assert torch.all((d2[:, row0:row0 + 128 * P] >= -1e-6) & (d2[:, row0:row0 + 128 * P] <= 2))
