"""GPU patch with the fp16 copy of V, on both sides of the row count up to which
one launch does both: prompts that end inside a workgroup's rows, one row, no
selected row, every row, lists in any order with rows outside the cache among
them (skipped), row sets shared by the layers or their own, kv heads that fill
less and more than one round of a workgroup.  Caches and copy equal numpy's bit
for bit; the status word reports a value fp16 cannot hold."""
import sys

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [  # (rows of the cache, selected, layers, kv heads, d, sets per layer)
    (1, 1, 1, 1, 64, True),
    (33, 0, 1, 2, 128, True),
    (97, 97, 3, 3, 64, False),
    (500, 77, 2, 16, 128, True),
    (9001, 4096, 4, 2, 128, True),
    (9001, 4097, 4, 2, 64, True),
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: "T%d_n%d_L%d_h%d_d%d" % c[:5])
def test_patch_and_fp16_copy(c):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    T, n, L, H, d, own = c
    print(f"[patch-span] {c}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(T + n)
    S = L if own else 1
    bf = lambda: (rng.standard_normal((L, H, T, d)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)  # noqa: E731
    kf, vf, kc, vc = bf(), bf(), bf(), bf()
    rows, cr = np.full((S, T), -1, np.int32), np.zeros((S, 2), np.int32)
    for s in range(S):
        m = max(n - 3 * s, 0)
        rows[s, :m] = rng.permutation(T)[:m]
        if m > 2:
            rows[s, 1], rows[s, m - 1] = -5, T
        cr[s, 1] = m
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()  # noqa: E731
    d_rows, d_cr = torch.from_numpy(rows).cuda(), torch.from_numpy(cr).cuda()
    d_cu = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    d_kf, d_vf = dev(kf), dev(vf)
    for wide in (False, True):
        if wide:
            vc[L - 1, H - 1, T - 1, d - 1] = vf[L - 1, H - 1, T - 1, d - 1] = 0x4780  # 65536
            d_vf = dev(vf)
        d_kc, d_vc = dev(kc), dev(vc)
        v16 = torch.zeros((L, H, T, d), dtype=torch.int16, device="cuda")
        status = torch.zeros(4, dtype=torch.int32, device="cuda")
        kvb.kvb_patch(L, H, H, d, T, d_cu, 1, T, d_rows, d_cr, int(own), n, d_kf, d_vf, d_kc, d_vc, v16,
                      None, 0, v_status=status)
        torch.cuda.synchronize()
        rk, rv = kc.copy(), vc.copy()
        for l in range(L):
            s = l if own else 0
            t = rows[s, :cr[s, 1]]
            t = t[(t >= 0) & (t < T)]
            rk[l][:, t], rv[l][:, t] = kf[l][:, t], vf[l][:, t]
        with np.errstate(over="ignore"):
            r16 = (rv.astype(np.uint32) << 16).view(np.float32).astype(np.float16).view(np.uint16)
        host = lambda x: x.cpu().numpy().view(np.uint16)  # noqa: E731
        assert np.array_equal(host(d_kc), rk) and np.array_equal(host(d_vc), rv)
        assert np.array_equal(host(v16), r16)
        assert status.cpu().numpy()[0] == int(wide)
