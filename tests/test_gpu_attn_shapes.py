"""GPU attention over the launch shapes that several layers and long prompts take.

Balanced ranges (tiles cut between workgroups, merged by the combine launch) with
head size 64, several prompts (an empty one among them), fp32 output, and a plan
over several layers whose row sets differ.  That a case takes them is read from
the workspace, where only balanced ranges leave partial records.  Against the
float64 oracle within the bound of attn_check.

A layer's call gives what a one-layer combined call over the same rows gives, bit
for bit, however many layers the caches hold; a combined call over all layers may
take another launch shape (decided from all its tiles), and then agrees within the
same bound.

A query with a NaN gives NaN for its own row and head and changes nothing else
(key-split and whole tiles)."""
import sys

import numpy as np
import pytest
import torch

from attn_check import REL, worst_rel
from oracle import attention as oatt
from oracle import numerics

pytestmark = pytest.mark.gpu

LONG = [4200, 0, 3000]


class Case:
    """Standard normal tensors, `picks` random rows of every prompt (the last row
    among them; layer l holds l rows fewer) and the buffers of the calls."""

    def __init__(self, lens, picks, L, hq, hkv, d, f32, seed=0):
        from paper_2608_21362_amd import kvb

        rng = np.random.default_rng(sum(lens) + hq + seed)
        self.kvb, self.L, self.d, self.f32 = kvb, L, d, f32
        self.cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        self.T, B = int(self.cu[-1]), len(lens)
        self.rows, self.cr = np.full((L, self.T), -1, np.int32), np.zeros((L, B + 1), np.int32)
        for l in range(L):
            n = 0
            for b, pick in enumerate(picks):
                m = max(pick - l, 1) if pick else 0
                r = rng.choice(lens[b] - 1, m - 1, replace=False) if m else []
                r = sorted(int(self.cu[b] + i) for i in list(r) + ([lens[b] - 1] if m else []))
                self.rows[l, n:n + m] = r
                n += m
                self.cr[l, b + 1] = n
        n_max = int(self.cr[:, -1].max())
        bf = lambda *s: numerics.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))  # noqa: E731
        self.q, self.k, self.v = bf(L, self.T, hq, d), bf(L, hkv, self.T, d), bf(L, hkv, self.T, d)
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()  # noqa: E731
        self.q_d, self.k_d, self.v_d = dev(self.q), dev(self.k), dev(self.v)
        d_cu, self.d_rows, self.d_cr = (torch.from_numpy(a).cuda() for a in (self.cu, self.rows, self.cr))
        self.shape, self.size = (hq, hkv, d, self.T), (hq, hkv, d, self.T, B, max(lens), n_max)
        self.lists = lambda rows, cr: (d_cu, B, max(lens), rows, cr, 1, n_max)  # noqa: E731
        self.out_code = kvb.KVB_F32 if f32 else kvb.KVB_BF16

    def _buffers(self, L, v16_given):
        """Output of L layers, and a workspace of as many as the call takes."""
        self.out = torch.full((L, self.T, self.size[0], self.d), -1, dtype=torch.float32 if self.f32 else torch.int16,
                              device="cuda")
        n = 1 if v16_given else L
        need = self.kvb.kvb_sparse_attn_workspace_bytes(n, *self.size, int(v16_given))
        return torch.full((need,), 255, dtype=torch.uint8, device="cuda")

    def _recorded(self, ws):
        """Whether the launch left partial records: they are the workspace's last
        part, 2048 x 128 x (d fp16 values and two floats)."""
        return bool((ws[-2048 * 128 * (2 * self.d + 8):] != 255).any())

    def layered(self):
        """kvb_patch of every layer, then a call per layer."""
        L = self.L
        kc, vc = self.k_d.clone(), self.v_d.clone()
        v16 = torch.zeros((L,) + tuple(kc.shape[1:]), dtype=torch.int16, device="cuda")
        pb = self.kvb.kvb_attn_plans_bytes(L, *self.size)
        plans = torch.full((max(pb, 16),), 255, dtype=torch.uint8, device="cuda")
        ws = self._buffers(L, True)
        args = self.lists(self.d_rows, self.d_cr)
        self.kvb.kvb_patch(L, *self.shape, *args, self.k_d, self.v_d, kc, vc, v16, plans, pb)
        for l in range(L):
            self.kvb.kvb_sparse_attn_layer(l, L, *self.shape, *args, self.q_d, kc, v16, plans, pb, self.d ** -0.5,
                                           self.out_code, self.out, ws, ws.numel())
        torch.cuda.synchronize()
        return self.out.cpu().numpy(), self._recorded(ws)

    def combined(self, layer=None):
        """One combined call over all layers, or over one of them alone; with the
        fp16 copy of V in the workspace."""
        at = slice(0, self.L) if layer is None else slice(layer, layer + 1)
        n = at.stop - at.start
        ws = self._buffers(n, False)
        kf, vf, q, rows, cr = (t[at].contiguous() for t in (self.k_d, self.v_d, self.q_d, self.d_rows, self.d_cr))
        kc, vc = kf.clone(), vf.clone()
        self.kvb.kvb_sparse_attn(n, *self.shape, *self.lists(rows, cr), q, kf, vf, kc, vc, None, self.d ** -0.5,
                                 self.out_code, self.out, ws, ws.numel())
        torch.cuda.synchronize()
        return self.out.cpu().numpy(), self._recorded(ws)

    def values(self, out, l, rows):
        return (out[l] if self.f32 else numerics.bf16_bits_to_f32(out.view(np.uint16)[l]))[rows]

    def check(self, out, layers=None):
        kind = "f32" if self.f32 else "bf16"
        for l in range(self.L) if layers is None else layers:
            mine = self.rows[l, :self.cr[l, -1]]
            ref = oatt.attend_rows(self.q[l], self.k[l], self.v[l], mine, self.cu)
            err = worst_rel(self.values(out, l, mine), ref)
            print(f"[attn-shapes] layer {l}: worst relative error {err:.2e}", file=sys.stderr, flush=True)
            assert err <= REL[kind], (l, err)
            others = np.setdiff1d(np.arange(self.T), mine)
            assert np.all(out[l][others] == -1), "a row outside the list was written"


def _same(a, b):
    return np.array_equal(a.view(np.uint8), b.view(np.uint8))


BALANCED = [  # (prompt lengths, rows per prompt, layers, q heads, kv heads, d, f32 out)
    (LONG, [90, 0, 40], 1, 4, 2, 64, False),
    (LONG, [90, 0, 40], 1, 4, 2, 64, True),
    (LONG, [90, 0, 40], 1, 16, 2, 128, True),
    ([4200], [90], 4, 16, 2, 128, False),
    ([4200], [90], 4, 4, 2, 64, True),
]


@pytest.mark.parametrize("c", BALANCED, ids=lambda c: "T%d_B%d_L%d_hq%d_hkv%d_d%d_%s" % (
    sum(c[0]), len(c[0]), *c[2:6], "f32" if c[6] else "bf16"))
def test_balanced_ranges(c):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[attn-shapes] balanced {c}", file=sys.stderr, flush=True)
    s = Case(*c)
    per_layer, recorded = s.layered()
    assert recorded, "the layer calls left no partial records: no tile was cut"
    s.check(per_layer)
    together, recorded = s.combined()
    assert recorded, "the combined call left no partial records: no tile was cut"
    s.check(together)


CONTRACT = [  # (prompt lengths, rows per prompt, layers, q heads, kv heads, d, f32 out)
    ([256], [163], 12, 16, 2, 128, False),        # a layer key-split, all of them whole tiles
    ([300, 300], [300, 300], 8, 32, 8, 128, True),
    ([700, 0, 33], [700, 0, 33], 4, 8, 8, 64, False),
    ([4200], [90], 3, 16, 2, 128, True),          # balanced ranges, other cuts
    ([900, 1100], [900, 1100], 2, 64, 4, 64, True),
]


@pytest.mark.parametrize("c", CONTRACT, ids=lambda c: "T%d_B%d_L%d_hq%d_hkv%d_d%d_%s" % (
    sum(c[0]), len(c[0]), *c[2:6], "f32" if c[6] else "bf16"))
def test_layer_calls_equal_one_layer_combined_calls(c):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[attn-shapes] contract {c}", file=sys.stderr, flush=True)
    s = Case(*c)
    per_layer, _ = s.layered()
    for l in range(s.L):
        assert _same(per_layer[l], s.combined(l)[0][0]), l
    together, _ = s.combined()
    ends = sorted({0, s.L - 1})
    s.check(per_layer, ends)
    s.check(together, ends)


NAN = [  # key-split tiles, whole tiles
    ([500], [200], 1, 16, 2, 128, False),
    ([900, 1100], [900, 1100], 1, 64, 4, 64, False),
]


@pytest.mark.parametrize("c", NAN, ids=lambda c: "T%d_B%d_hq%d_hkv%d_d%d" % (sum(c[0]), len(c[0]), *c[3:6]))
def test_nan_query_stays_alone(c):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[attn-shapes] nan {c}", file=sys.stderr, flush=True)
    s = Case(*c)
    clean, _ = s.layered()
    mine = s.rows[0, :s.cr[0, -1]]
    t, h = int(mine[len(mine) // 2]), s.size[0] - 1
    s.q_d[0, t, h, 3] = 0x7FC0
    got, _ = s.layered()
    a, b = s.values(clean, 0, np.arange(s.T)), s.values(got, 0, np.arange(s.T))
    assert np.all(np.isnan(b[t, h])) and np.all(np.isfinite(a[mine]))
    got[0, t, h] = clean[0, t, h]
    assert _same(got, clean)
