"""Packing at any alignment and over the whole fp16 range, byte for byte."""
import numpy as np
import pytest

from oracle import grinqh_oracle as orc
from synth import inputs
from test_gpu_parity import _dev, _host, g, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _at(torch, a, dtype, offset):  # noqa: F811
    """A contiguous device copy of `a` that starts `offset` elements into its buffer."""
    flat = torch.empty(a.size + offset, dtype=dtype, device="cuda")
    flat[offset:] = _dev(torch, a.reshape(-1))
    return flat[offset:].view(a.shape)


@pytest.mark.parametrize("offset", [0, 1, 4])
@pytest.mark.parametrize("K,N,levels,tile_n", [
    (128, 256, (0, 2, 4, 8), 256), (384, 1536, (0, 2, 4, 6), 512), (256, 2048, (0, 2, 4), 2048),
    (256, 1024, (0, 2, 3, 4, 8), 512), (128, 1024, (0, 1, 4), 1024)])
def test_pack_any_alignment(g, torch, offset, K, N, levels, tile_n):  # noqa: F811
    desc = g.grinqh_resolve_desc(g.make_desc(K, N, levels, tile_n=tile_n))
    b_max, (nc, _) = levels[-1], g.grinqh_packed_bytes(desc)
    out = torch.empty(nc + 4 * offset, dtype=torch.uint8, device="cuda")[4 * offset:]
    W = inputs.weights(N, K, 93)
    q, s = orc.rtn_quantize(W, b_max=b_max)
    pc, ps = g.grinqh_pack(desc, W=_at(torch, W, torch.float16, offset), out_codes=out)
    want = orc.pack_codes_fast(q, desc.plane_bits, tile_n, b_max)
    assert np.array_equal(_host(pc), want)
    assert np.array_equal(_host(ps).view(np.uint16), s.view(np.uint16))
    # given codes: bits above b_max drop out
    codes = inputs.random_codes(N, K, 93)
    pc, _ = g.grinqh_pack(desc, codes=_at(torch, codes, torch.uint8, offset),
                          scales=_dev(torch, np.ascontiguousarray(s.T)), out_codes=out)
    want = orc.pack_codes_fast(codes & ((1 << b_max) - 1), desc.plane_bits, tile_n, b_max)
    assert np.array_equal(_host(pc), want)


@pytest.mark.parametrize("levels", [(0, 2, 4, 8), (0, 2, 4, 6), (0, 2, 4)])
def test_pack_rounds_as_the_quotient(g, torch, levels):  # noqa: F811
    # groups at every scale down to subnormals, with exact halves of the scale
    # (ties to even) and their neighbours: rne(w / s) by one reciprocal and a
    # residual step has to give the rounded quotient's codes
    N, K, b_max = 512, 1024, levels[-1]
    r = np.random.default_rng(94)
    W = (r.standard_normal((N, K)) * np.exp2(r.uniform(-22, 12, size=(N, K // 128)).repeat(128, 1)))
    W = np.clip(W, -60000, 60000).astype(np.float16)
    amax = np.abs(W.reshape(N, -1, 128).astype(np.float32)).max(2)
    s = (amax / np.float32(2 ** (b_max - 1) - 1)).astype(np.float16).astype(np.float32)
    ties = (r.integers(-2 ** (b_max - 1), 2 ** (b_max - 1) - 1, size=(N, K // 128, 32)) + 0.5) * s[:, :, None]
    ties = np.clip(ties, -amax[:, :, None], amax[:, :, None]).astype(np.float16)
    near = ties.view(np.uint16).copy()
    near[:, :, ::2] ^= 1
    Wg = W.reshape(N, K // 128, 128)
    keep = np.abs(Wg.astype(np.float32)) == amax[:, :, None]          # the scale's own weight stays
    Wg[:, :, :32] = np.where(keep[:, :, :32], Wg[:, :, :32], ties)
    Wg[:, :, 32:64] = np.where(keep[:, :, 32:64], Wg[:, :, 32:64], near.view(np.float16))
    desc = g.grinqh_resolve_desc(g.make_desc(K, N, levels))
    q, sc = orc.rtn_quantize(W, b_max=b_max)
    pc, ps = g.grinqh_pack(desc, W=_dev(torch, W))
    assert np.array_equal(_host(ps).view(np.uint16), sc.view(np.uint16))
    assert np.array_equal(_host(pc), orc.pack_codes_fast(q, desc.plane_bits, desc.tile_n, b_max))


@pytest.mark.parametrize("levels", [(0, 2, 4, 8), (0, 2, 4, 6), (0, 2, 3, 4, 8), (0, 2, 4)])
def test_pack_non_finite_weights(g, torch, levels):  # noqa: F811
    # a NaN takes no part in its group's scale and gets code 0, as does an
    # infinity; the finite weights beside an infinity get the code of zero
    N, K, b_max = 512, 256, levels[-1]
    half = 1 << (b_max - 1)
    W = inputs.weights(N, K, 95).copy()
    W[0, 3], W[1, 127], W[2, 5], W[3, 9:20] = np.nan, -np.nan, np.inf, -np.inf
    W[4, 7], W[4, 8], W[5, 0:128], W[6, 1:128] = np.inf, np.nan, np.nan, np.nan
    W[7, :128], W[7, 50], W[8, :128] = 0, np.nan, 65504.0
    Wg = W.reshape(N, K // 128, 128).astype(np.float32)
    amax = np.fmax.reduce(np.abs(Wg), axis=2)                # ignores NaN
    with np.errstate(invalid="ignore", divide="ignore", over="ignore"):
        s = (amax / np.float32(half - 1)).astype(np.float16)
        r = np.rint(Wg / s.astype(np.float32)[:, :, None])
        r = np.fmin(np.fmax(r, -half), half - 1)             # a NaN becomes -half
        q = np.where(s[:, :, None] == 0, half, r + half).astype(np.uint8).reshape(N, K)
    desc = g.grinqh_resolve_desc(g.make_desc(K, N, levels))
    pc, ps = g.grinqh_pack(desc, W=_dev(torch, W))
    assert np.array_equal(_host(ps), np.ascontiguousarray(s.T), equal_nan=True)
    assert np.array_equal(_host(pc), orc.pack_codes_fast(q, desc.plane_bits, desc.tile_n, b_max))


@pytest.mark.parametrize("S", [1, 7, 585, 1025])
@pytest.mark.parametrize("levels", [(0, 8), (0, 2, 4, 6, 8), (0, 1, 2, 3, 4, 5, 6, 7, 8)])
def test_calibrate_mean_stages(g, torch, S, levels):  # noqa: F811
    # up to and past one stage of staged values (4096 / thresholds samples)
    K, n = 128, len(levels)
    p = [10000 // n] * (n - 1)
    p.append(10000 - sum(p))
    x = inputs.activations_t3(K, S, 95)
    desc = g.make_desc(K, 1024, levels)
    got = _host(g.grinqh_calibrate(desc, _dev(torch, x), p))
    want = orc.calibrate_thresholds([np.abs(row.astype(np.float64)) for row in x], p)
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
