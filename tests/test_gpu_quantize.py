"""GPU quantisation against the oracle, bit-exact, where the kernels split the
work differently: every key group size (inside a thread's quads, one thread,
two and four threads through LDS), every value group size (2 to 16 lanes), both
head sizes and widths, fp32 and fp64 input, several input layers written at an
offset; and values that decide the rounding: exact halves (integers over a
range of 2 (2^b - 1)), constant groups, zeros of both signs, and ranges whose
reciprocal is subnormal or infinite."""
import sys

import numpy as np
import pytest
import torch

from oracle import kivi

pytestmark = pytest.mark.gpu

SHAPES = [  # (chunks, pool layers, first layer, input layers, kv heads, d, bits, Gk, Gv, dtype)
    (3, 3, 1, 2, 2, 128, 4, 32, 32, np.float64),
    (2, 1, 0, 1, 2, 128, 8, 128, 128, np.float64),
    (2, 2, 0, 2, 1, 128, 8, 64, 64, np.float32),
    (1, 1, 0, 1, 3, 128, 4, 4, 16, np.float32),
    (2, 1, 0, 1, 2, 64, 4, 16, 16, np.float64),
    (1, 2, 1, 1, 2, 64, 8, 8, 64, np.float64),
    (5, 1, 0, 1, 1, 64, 8, 128, 32, np.float32),
    (3, 1, 0, 1, 4, 64, 4, 64, 32, np.float64),
]


def _values(rng, shape, bits, dt):
    """One kind of values per chunk token group of 4, cycling along the tokens."""
    levels = (1 << bits) - 1
    x = rng.standard_normal(shape) * np.exp(rng.uniform(-3, 3, shape[:-2] + (1, shape[-1])))
    half = rng.integers(0, 2 * levels + 1, shape).astype(np.float64)  # odd ones are exact halves
    half[..., 0, :], half[..., -1, :] = 0, 2 * levels
    half[..., :, 0], half[..., :, -1] = 0, 2 * levels
    h = shape[1] % 3
    for p in range(shape[0]):
        for l in range(shape[1]):
            kind = (p + l + h) % 4
            if kind == 1:
                x[p, l] = half[p, l]
            elif kind == 2:
                x[p, l] = np.where(rng.random(x[p, l].shape) < 0.5, 0.0, -0.0) + 3.0 * (l % 2)
            elif kind == 3:
                x[p, l] *= 1e-38 if dt == np.float32 else 1e-307
    if dt == np.float64:
        x[0, 0, 0, :4] *= 1e305  # ranges past the fast path's limits, still finite
    return x.astype(dt)


@pytest.mark.parametrize("s", SHAPES, ids=lambda s: "P%d_L%d_%d_%d_H%d_d%d_b%d_k%d_v%d_%s" % (
    *s[:9], np.dtype(s[9]).name))
def test_quantise_bit_exact(s):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    P, L, first, n_in, H, d, bits, gk, gv, dt = s
    print(f"[quantise] {s}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(P * 100 + gk + gv)
    k = _values(rng, (P, n_in, H, 128, d), bits, dt)
    v = _values(rng, (P, n_in, H, 128, d), bits, dt)
    pool = kvb.pool_layout(L, H, d, bits, gk, gv)
    new = lambda *shape, dtype: torch.full(shape, 77, dtype=dtype, device="cuda")  # noqa: E731
    kc, vc = (new(P, L, H, 128, d * bits // 8, dtype=torch.uint8) for _ in range(2))
    ks, kz = (new(P, L, H, 128 // gk, d, dtype=torch.float32) for _ in range(2))
    vs, vz = (new(P, L, H, 128, d // gv, dtype=torch.float32) for _ in range(2))
    kvb.kvb_kivi_quantize(pool, P, first, n_in, kvb.KVB_F64 if dt == np.float64 else kvb.KVB_F32,
                          torch.from_numpy(k).cuda(), torch.from_numpy(v).cuda(), kc, ks, kz, vc, vs, vz)
    torch.cuda.synchronize()
    for (codes, scale, zero), got in ((kivi.quantise_keys(k, bits, gk), (kc, ks, kz)),
                                      (kivi.quantise_values(v, bits, gv), (vc, vs, vz))):
        for ref, t in zip((kivi.pack(codes, bits), scale, zero), got):
            t = t.cpu().numpy()
            assert np.array_equal(t[:, first:first + n_in], ref)
            rest = np.delete(t, np.s_[first:first + n_in], axis=1)
            assert np.all(rest == 77), "a layer outside the call was written"


def _groups_ref(x, axis, bits):
    """Codes, scale and zero of x f64 in groups along `axis`, for any values: a
    minimum and maximum pass over NaN, and a quotient that is NaN gives code 0."""
    levels = float((1 << bits) - 1)
    mn = np.fmin.reduce(x, axis=axis, initial=np.inf, keepdims=True)
    mx = np.fmax.reduce(x, axis=axis, initial=-np.inf, keepdims=True)
    r = mx - mn
    t = np.where(r != 0, (x - mn) / np.where(r != 0, r, 1) * levels, 0.0)
    code = np.fmin(np.fmax(np.rint(t), 0.0), levels).astype(np.uint8)
    return code, np.where(r == 0, 0, r / levels).astype(np.float32), mn.astype(np.float32)


@pytest.mark.parametrize("bits,gk,gv,dt", [(4, 32, 16, np.float64), (8, 128, 64, np.float32), (8, 4, 32, np.float64)])
@pytest.mark.filterwarnings("ignore::RuntimeWarning")
def test_quantise_nan_and_infinities(bits, gk, gv, dt):
    """Infinities and NaN, alone in a group, beside finite values and filling one."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_21362_amd import kvb

    print(f"[quantise] special values b{bits} k{gk} v{gv} {np.dtype(dt).name}", file=sys.stderr, flush=True)
    P, d = 3, 64
    rng = np.random.default_rng(bits + gk)
    x = rng.standard_normal((2, P, 1, 1, 128, d)).astype(dt)
    for p, special in enumerate((np.nan, np.inf, -np.inf)):
        x[:, p][rng.random(x[:, p].shape) < 0.02] = special
        x[:, p, 0, 0, :, 5] = x[:, p, 0, 0, 7, :] = special      # a whole channel, a whole token
    k, v = x
    pool = kvb.pool_layout(1, 1, d, bits, gk, gv)
    new = lambda *shape, dtype: torch.zeros(shape, dtype=dtype, device="cuda")  # noqa: E731
    kc, vc = (new(P, 1, 1, 128, d * bits // 8, dtype=torch.uint8) for _ in range(2))
    ks, kz = (new(P, 1, 1, 128 // gk, d, dtype=torch.float32) for _ in range(2))
    vs, vz = (new(P, 1, 1, 128, d // gv, dtype=torch.float32) for _ in range(2))
    kvb.kvb_kivi_quantize(pool, P, 0, 1, kvb.KVB_F64 if dt == np.float64 else kvb.KVB_F32,
                          torch.from_numpy(k).cuda(), torch.from_numpy(v).cuda(), kc, ks, kz, vc, vs, vz)
    torch.cuda.synchronize()
    kg = _groups_ref(k.astype(np.float64).reshape(P, 1, 1, 128 // gk, gk, d), -2, bits)
    vg = _groups_ref(v.astype(np.float64).reshape(P, 1, 1, 128, d // gv, gv), -1, bits)
    for (code, scale, zero), (c, s, z) in ((kg, (kc, ks, kz)), (vg, (vc, vs, vz))):
        assert np.array_equal(c.cpu().numpy(), kivi.pack(code.reshape(P, 1, 1, 128, d), bits))
        for ref, t in ((scale, s), (zero, z)):
            assert np.array_equal(t.cpu().numpy(), ref.reshape(t.shape), equal_nan=True)
