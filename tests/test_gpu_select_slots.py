"""GPU selection against the oracle where the register kernel's split changes:
prompt lengths at the edges of a wave's run, of the slot counts (8, 16, 32, 48
and 64 rows per thread) and past them (the streaming kernel), batches with
empty and one-row prompts; k at its edges; deviations that end the digit passes
early (all distinct), late (one value, or values equal in their upper 24 bits)
and with many ties at the cut.  Bit-exact."""
import sys

import numpy as np
import pytest
import torch

from oracle import selection as osel

pytestmark = pytest.mark.gpu

LENS = [[1], [64], [1023], [1024], [1025], [8192], [8193], [16385], [32769], [49153], [65536],
        [65537], [3, 0, 1024, 1, 1025, 0], [66000, 5]]


def _delta(rng, kind, n):
    if kind == "distinct":
        return (rng.permutation(n) / n).astype(np.float32)
    if kind == "one":
        return np.full(n, 0.25, np.float32)
    if kind == "close":  # equal down to the last byte
        return (np.float32(1.0).view(np.uint32) + rng.integers(0, 200, n).astype(np.uint32)).view(np.float32)
    return rng.choice(np.array([-1.0, -0.0, 0.0, 1e-9, 0.5], np.float32), n)


@pytest.mark.parametrize("lens", LENS, ids=lambda x: "_".join(map(str, x)))
def test_select_slots(lens):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    print(f"[select-slots] {lens}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(sum(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, B = int(cu[-1]), len(lens)
    cand = rng.random(T) < 0.9
    forced = (~cand & (rng.random(T) < 0.5)) | (rng.random(T) < 0.02)
    flags = cand.astype(np.uint8) | (forced.astype(np.uint8) << 1)
    n = np.array([int(cand[cu[b]:cu[b + 1]].sum()) for b in range(B)])
    kinds = ["distinct", "one", "close", "ties"]
    ks = [np.maximum(n * 15 // 100, 1), np.maximum(n - 1, 0), n, np.minimum(n, 1), n * 0, n + 3, n // 2]
    sets = [(kind, k) for kind in kinds for k in ks]
    delta = np.stack([_delta(rng, kind, T) for kind, _ in sets])
    k = np.stack([k for _, k in sets]).astype(np.int32)
    S = len(sets)
    need = kvb.kvb_select_workspace_bytes(S, T, B)
    ws = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    rows = torch.full((S, T), -1, dtype=torch.int32, device="cuda")
    cr = torch.full((S, B + 1), -1, dtype=torch.int32, device="cuda")
    kvb.kvb_select(S, T, torch.from_numpy(cu).cuda(), B, torch.from_numpy(delta).cuda(),
                   torch.from_numpy(flags).cuda(), torch.from_numpy(k).cuda(), rows, cr, ws, need)
    torch.cuda.synchronize()
    rows, cr = rows.cpu().numpy(), cr.cpu().numpy()
    for s in range(S):
        r_rows, r_cu = osel.select(delta[s], cand, forced, cu, k[s])
        assert np.array_equal(cr[s], r_cu), sets[s]
        assert np.array_equal(rows[s, :r_cu[-1]], r_rows), sets[s]
        assert np.all(rows[s, r_cu[-1]:] == -1), sets[s]
