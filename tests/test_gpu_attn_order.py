"""GPU attention of batches whose tiles outnumber the resident workgroups (512
on 256 CUs): launches of one layer, and those of several with at most 128 tiles a
prompt, then take their tile slots in an order built on the device.  512 tiles (no
order) and 516, prompts of one length and of falling and rising ones, empty
prompts, one prompt more than the order takes, more slots than the builder
handles in one round (1024; long tiles in both rounds), several layers with few
and with many tiles a prompt, and row sets that differ between layers (the order
comes from the first).  Against the float64 oracle within the bound of
attn_check; rows outside the lists stay untouched.  Both the combined call, whose
workspace shows whether an order was built and that it is a permutation, and the
per-layer calls (which may take another launch shape)."""
import sys

import numpy as np
import pytest
import torch

from attn_check import REL, worst_rel
from oracle import attention as oatt
from oracle import numerics

pytestmark = pytest.mark.gpu

CASES = [  # (prompt lengths, rows per prompt of layer 0, layers, q heads, kv heads, d, ordered)
    ([300] * 2, [300] * 2, 8, 32, 8, 128, False),                        # 672 tiles a prompt
    ([700, 0, 300, 90, 33, 1], [700, 0, 300, 90, 33, 1], 2, 64, 2, 128, False),
    ([200, 0, 150, 90] * 4, [200, 0, 150, 90] * 4, 2, 64, 2, 128, True),  # 114 a prompt
    ([40, 200, 500, 900], [40, 150, 500, 900], 1, 64, 4, 64, True),
    ([64] * 64, [16] * 64, 1, 16, 8, 64, True),
    ([64] * 65, [16] * 65, 1, 16, 8, 64, False),
    ([600, 408], [600, 408], 1, 64, 4, 64, False),                       # 4 x 128 tiles
    ([608, 408], [608, 408], 1, 64, 4, 64, True),                        # 4 x 129
    ([2000, 1500, 900, 900, 700], [2000, 1500, 900, 900, 700], 1, 64, 2, 64, True),  # 1500 slots with rows
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: "T%d_B%d_L%d_hq%d_hkv%d_d%d" % (
    sum(c[0]), len(c[0]), *c[2:6]))
def test_attention_tile_order(c):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    lens, picks, L, hq, hkv, d, ordered = c
    print(f"[attn-order] {sum(lens)} rows, {len(lens)} prompts, {L} layers, {hq}/{hkv} heads, d={d}",
          file=sys.stderr, flush=True)
    rng = np.random.default_rng(sum(lens) + hq)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, B = int(cu[-1]), len(lens)
    rows, cr = np.full((L, T), -1, np.int32), np.zeros((L, B + 1), np.int32)
    for l in range(L):
        n = 0
        for b, pick in enumerate(picks):
            m = max(pick - 37 * l, min(pick, 1))  # later layers hold fewer rows
            r = np.sort(rng.choice(lens[b], m, replace=False)) + cu[b] if m else np.zeros(0, np.int32)
            rows[l, n:n + m] = r
            n += m
            cr[l, b + 1] = n
    n_max = int(cr[:, -1].max())
    bf = lambda *s: numerics.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))  # noqa: E731
    q, kf, vf = bf(L, T, hq, d), bf(L, hkv, T, d), bf(L, hkv, T, d)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()  # noqa: E731
    d_rows, d_cr, d_cu = (torch.from_numpy(a).cuda() for a in (rows, cr, cu))
    q_d, k_d, v_d = dev(q), dev(kf), dev(vf)
    size = (hq, hkv, d, T, B, max(lens), n_max)
    args = (d_cu, B, max(lens), d_rows, d_cr, 1, n_max)
    outs = []
    for layered in (False, True):
        out = torch.full((L, T, hq, d), -1, dtype=torch.int16, device="cuda")
        kc, vc = k_d.clone(), v_d.clone()
        v16 = torch.zeros((L, hkv, T, d), dtype=torch.int16, device="cuda")
        need = kvb.kvb_sparse_attn_workspace_bytes(L, *size, 1)
        ws = torch.full((max(need, 16),), 255, dtype=torch.uint8, device="cuda")
        if layered:
            pb = kvb.kvb_attn_plans_bytes(L, *size)
            plans = torch.full((max(pb, 16),), 255, dtype=torch.uint8, device="cuda")
            kvb.kvb_patch(L, hq, hkv, d, T, *args, k_d, v_d, kc, vc, v16, plans, pb)
            for l in range(L):
                kvb.kvb_sparse_attn_layer(l, L, hq, hkv, d, T, *args, q_d, kc, v16, plans, pb, d ** -0.5,
                                          kvb.KVB_BF16, out, ws, need)
        else:
            kvb.kvb_sparse_attn(L, hq, hkv, d, T, *args, q_d, k_d, v_d, kc, vc, v16, d ** -0.5,
                                kvb.KVB_BF16, out, ws, need)
            # the order of the slots follows the plan's four words
            slots = -(-n_max // (128 * hkv // hq)) + B
            order = ws[16:16 + 4 * slots].cpu().numpy().view(np.int32)
            assert np.array_equal(np.sort(order), np.arange(slots) if ordered else np.full(slots, -1))
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy())
    for l in range(L):
        mine = rows[l, :cr[l, -1]]
        ref = oatt.attend_rows(q[l], kf[l], vf[l], mine, cu)
        for out in outs:
            got = numerics.bf16_bits_to_f32(out.view(np.uint16)[l][mine]).astype(np.float64)
            err = worst_rel(got, ref)
            print(f"[attn-order] layer {l}: worst relative error {err:.2e}", file=sys.stderr, flush=True)
            assert err <= REL["bf16"], (l, err)
            others = np.setdiff1d(np.arange(T), mine)
            assert np.all(out[l][others] == -1), "a row outside the list was written"
