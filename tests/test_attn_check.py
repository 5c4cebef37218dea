"""The attention tests' bound sees what it is there for: the oracle with keys left
out of long prompts fails it, the oracle rounded as an output is passes it."""
import numpy as np
import pytest

from attn_check import REL, worst_rel
from oracle import attention as oatt
from oracle import numerics


@pytest.mark.parametrize("T", [300, 2100, 4200])
def test_bound_sees_missing_keys(T):
    rng = np.random.default_rng(T)
    bf = lambda *s: numerics.bf16_bits_to_f32(numerics.f32_to_bf16_bits(  # noqa: E731
        rng.standard_normal(s).astype(np.float32))).astype(np.float64)
    q, k, v = bf(T, 2, 64), bf(1, T, 64), bf(1, T, 64)
    rows, cu = [T - 1], [0, T]
    ref = oatt.attend_rows(q, k, v, rows, cu)
    as_bf16 = numerics.bf16_bits_to_f32(numerics.f32_to_bf16_bits(ref.astype(np.float32)))
    assert worst_rel(as_bf16, ref) <= REL["bf16"] / 2
    # one key, a block of 32, and every fourth block
    lost = [np.array([T // 2]), np.arange(64, 96), np.arange(T).reshape(-1)[(np.arange(T) // 32) % 4 == 1]]
    for at in lost:
        kept = np.setdiff1d(np.arange(T), at)
        n = len(kept)
        got = oatt.attend_rows(q[T - n:], k[:, kept], v[:, kept], [n - 1], [0, n])
        assert worst_rel(got, ref) > REL["bf16"], len(at)
