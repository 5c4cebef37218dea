"""GPU attention where the launch shape is decided by size: prompts whose rows
fill, end inside or just pass a 32-query tile, key counts at the edges of a
block and of a round of four blocks (waves with no block at all), every number
of query heads per kv head, both head sizes and output types, several prompts
(empty ones, one-row ones, more than one wave-wide lookup of them), and row
counts that reach whole tiles and balanced ranges.  Against the float64 oracle
within the bound of attn_check; rows outside the list stay untouched.  The
per-layer call equals the combined call bit for bit."""
import sys

import numpy as np
import pytest
import torch

from attn_check import REL, worst_rel
from oracle import attention as oatt
from oracle import numerics

pytestmark = pytest.mark.gpu

CASES = [  # (prompt lengths, rows per prompt, q heads, kv heads, d, f32 out)
    ([1], [1], 16, 2, 128, False),
    ([32], [32], 16, 2, 128, False),
    ([33], [4], 16, 2, 128, True),
    ([128], [5], 16, 2, 128, False),
    ([129], [129], 8, 8, 64, False),
    ([257], [31], 32, 1, 128, False),
    ([500], [33], 4, 2, 64, True),
    ([40, 0, 1, 300, 97], [7, 0, 1, 64, 0], 16, 2, 128, False),
    ([3] * 70 + [64] * 3, [1] * 70 + [20] * 3, 8, 2, 64, False),
    ([2100], [300], 16, 2, 128, False),
    ([4200], [90], 16, 2, 128, False),
    ([300, 200], [300, 200], 16, 8, 128, False),
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: "T%d_B%d_hq%d_hkv%d_d%d" % (
    sum(c[0]), len(c[0]), *c[2:5]))
def test_attention_launch_shapes(c):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    lens, picks, hq, hkv, d, f32 = c
    print(f"[attn-shapes] {sum(lens)} rows, {len(lens)} prompts, {hq}/{hkv} heads, d={d}",
          file=sys.stderr, flush=True)
    rng = np.random.default_rng(sum(lens) + hq)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, B = int(cu[-1]), len(lens)
    rows, cr = [], [0]
    for b, n in enumerate(picks):
        # the last row always, so that the tiles reach every key block
        r = rng.choice(max(lens[b] - 1, 0), max(n - 1, 0), replace=False)
        rows += sorted(int(cu[b] + i) for i in list(r) + ([lens[b] - 1] if n else []))
        cr.append(len(rows))
    bf = lambda *s: numerics.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))  # noqa: E731
    q, kf, vf = bf(1, T, hq, d), bf(1, hkv, T, d), bf(1, hkv, T, d)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()  # noqa: E731
    all_rows = np.full((1, T), -1, np.int32)
    all_rows[0, :len(rows)] = rows
    d_rows, d_cr = torch.from_numpy(all_rows).cuda(), torch.from_numpy(np.array([cr], np.int32)).cuda()
    d_cu, q_d, k_d, v_d = torch.from_numpy(cu).cuda(), dev(q), dev(kf), dev(vf)
    out_t, out_k = (torch.float32, kvb.KVB_F32) if f32 else (torch.int16, kvb.KVB_BF16)
    size = (hq, hkv, d, T, B, max(lens), len(rows))
    status = torch.zeros(4, dtype=torch.int32, device="cuda")
    outs = []
    for split in (False, True):
        out = torch.full((1, T, hq, d), -1, dtype=out_t, device="cuda")
        kc, vc = k_d.clone(), v_d.clone()
        v16 = torch.zeros((1, hkv, T, d), dtype=torch.int16, device="cuda")
        need = kvb.kvb_sparse_attn_workspace_bytes(1, *size, 1)
        ws = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
        args = (d_cu, B, max(lens), d_rows, d_cr, 1, len(rows))
        if split:
            pb = kvb.kvb_attn_plans_bytes(1, *size)
            plans = torch.empty(max(pb, 16), dtype=torch.uint8, device="cuda")
            kvb.kvb_patch(1, hq, hkv, d, T, *args, k_d, v_d, kc, vc, v16, plans, pb, v_status=status)
            kvb.kvb_sparse_attn_layer(0, 1, hq, hkv, d, T, *args, q_d, kc, v16, plans, pb, d ** -0.5,
                                      out_k, out, ws, need)
        else:
            kvb.kvb_sparse_attn(1, hq, hkv, d, T, *args, q_d, k_d, v_d, kc, vc, v16, d ** -0.5, out_k,
                                out, ws, need, v_status=status)
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy())
    assert np.array_equal(outs[0].view(np.uint8), outs[1].view(np.uint8))
    got = outs[0][0] if f32 else numerics.bf16_bits_to_f32(outs[0][0].view(np.uint16))
    ref = oatt.attend_rows(q[0], kf[0], vf[0], rows, cu)
    err = worst_rel(got[rows], ref)
    print(f"[attn-shapes] worst relative error {err:.2e}", file=sys.stderr, flush=True)
    assert err <= REL["f32" if f32 else "bf16"], err
    others = np.setdiff1d(np.arange(T), rows)
    assert np.all(outs[0][0][others] == -1), "a row outside the list was written"
