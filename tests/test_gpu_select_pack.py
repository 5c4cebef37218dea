"""GPU selection where the packing of a batch's prompts changes its course: 64
prompts and one more (the counts are summed 64 at a time), prompts that keep
no row, exactly 1024 and more than 1024 rows (the first 1024 are read ahead),
empty prompts at both ends.  Rows and offsets equal the oracle's."""
import sys

import numpy as np
import pytest
import torch

import kvb_workload as kw
from oracle import selection as osel

pytestmark = pytest.mark.gpu

BATCHES = [  # (prompt lengths, percent selected)
    ([1500, 1024, 1025, 7], 100),
    ([0, 3000, 0, 40, 0], 50),
    ([17] * 64, 30),
    ([17] * 65, 30),
    ([5, 0] * 70 + [1300], 0),
]


@pytest.mark.parametrize("lens,rho", BATCHES, ids=lambda x: str(len(x)) if isinstance(x, list) else f"rho{x}")
def test_select_packs_prompts(lens, rho):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    n_sets = 2
    rng = np.random.default_rng(len(lens) + rho)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, B = int(cu[-1]), len(lens)
    print(f"[select-pack] T={T} prompts={B}", file=sys.stderr, flush=True)
    cand = rng.random(T) < 0.9 if rho < 100 else np.ones(T, bool)
    forced = (~cand & (rng.random(T) < 0.5)) | (cand & (rng.random(T) < 0.05 * (rho > 0)))
    flags = (cand.astype(np.uint8) | (forced.astype(np.uint8) << 1)).astype(np.uint8)
    delta = kw.deviation_draw(n_sets, T, seed=B, n_levels=7)
    ks = np.array([osel.k_per_prompt(cu, cand, rho, 100)] * n_sets, np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    rows = torch.full((n_sets, T), -1, dtype=torch.int32, device="cuda")
    cur = torch.full((n_sets, B + 1), -1, dtype=torch.int32, device="cuda")
    wsb = kvb.kvb_select_workspace_bytes(n_sets, T, B)
    ws = torch.full((max(wsb, 16),), 255, dtype=torch.uint8, device="cuda")
    kvb.kvb_select(n_sets, T, dev(cu), B, dev(delta), dev(flags), dev(ks), rows, cur, ws, wsb)
    torch.cuda.synchronize()
    r, c = rows.cpu().numpy(), cur.cpu().numpy()
    for s in range(n_sets):
        rr, rc = osel.select(delta[s], cand, forced, cu, ks[s])
        assert np.array_equal(c[s], rc) and np.array_equal(r[s, :rc[-1]], rr), s
        assert np.all(r[s, rc[-1]:] == -1), "an entry past the list was written"
