"""Prefill of short prompts: blocks of tokens, turns, columns and K splits."""
import numpy as np
import pytest

from oracle import grinqh_oracle as orc
from synth import inputs
from test_gpu_parity import Layer, _dev, _host, g, opts, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _bound(L, x, sums):
    """(2^-11 + K 2^-24) sum |x| |w_hat| per element, the stated contract."""
    return (2.0 ** -11 + L.K * 2.0 ** -24) * sums


def _sums(L, x):
    half = 1 << (L.b_max - 1)
    w = np.abs(L.codes.astype(np.float64) - half) * np.repeat(L.scales.astype(np.float64).T, 128, axis=1)
    return np.abs(x.astype(np.float64)) @ w.T


# K = 128: two turns for eight waves; N = 256 .. 8448: K split in two (up to 128
# workgroups), one workgroup per 64 outputs, two columns per workgroup (over 256,
# 16640 outputs); M around the 16-token tiles and the 80-token blocks
@pytest.mark.parametrize("K,N,levels,tile_n,Ms", [
    (128, 256, (0, 2, 4, 8), 256, (1, 16, 17, 80, 81)),
    (1152, 1024, (0, 2, 4, 6, 8), 1024, (5, 33, 48, 161)),
    (640, 512, (0, 2, 4, 6), 512, (2, 64, 77)),
    (256, 2048, (0, 2, 4), 2048, (15, 96)),
    (384, 1024, (0, 2, 3, 4, 8), 512, (1, 31, 80, 130)),
    (256, 1024, (0, 1, 4), 1024, (49,)),
    (256, 8448, (0, 2, 4, 8), 256, (3, 78)),
    (256, 16640, (0, 2, 4, 8), 256, (18, 79)),
    (256, 16896, (0, 2, 3, 4, 8), 512, (40,))])
def test_prefill_small(g, torch, K, N, levels, tile_n, Ms):  # noqa: F811
    L = Layer(g, torch, K, N, levels, cfg=96, tile_n=tile_n, codes_src=True)
    for M in Ms:
        x = inputs.activations_t3(K, M, 96)
        xd = _dev(torch, x)
        y = g.grinqh_prefill(L.desc, L.pc, L.ps, xd)
        ref = orc.prefill(L.codes, L.scales, x, b_max=L.b_max)
        bound = _bound(L, x, _sums(L, x))
        assert np.all(np.abs(_host(y) - ref) <= bound), M
        # bit for bit again, over whatever y held; added to y on request
        y2 = torch.full_like(y, 3.5)
        for _ in range(3):
            g.grinqh_prefill(L.desc, L.pc, L.ps, xd, y=y2)
            assert torch.equal(y, y2), M
        g.grinqh_prefill(L.desc, L.pc, L.ps, xd, y=y2, accumulate=True)
        assert np.all(np.abs(_host(y2) - 2 * ref) <= 2.1 * bound), M


def test_prefill_small_rows_past_m_are_not_written(g, torch):  # noqa: F811
    L = Layer(g, torch, 256, 512, (0, 2, 4, 8), cfg=97, codes_src=True)
    M = 19
    buf = torch.full((M + 13, 512), 7.0, device="cuda")
    g.grinqh_prefill(L.desc, L.pc, L.ps, _dev(torch, inputs.activations_t3(256, M, 97)), y=buf[:M])
    assert bool((buf[M:] == 7.0).all())


@pytest.mark.parametrize("K,N,levels,M", [
    (1024, 512, (0, 2, 4, 8), 150), (1152, 1024, (0, 2, 4, 6, 8), 1), (14336, 512, (0, 2, 4, 6, 8), 77),
    (1024, 1024, (0, 2, 3, 4, 8), 20), (640, 512, (0, 2, 4), 47), (896, 2048, (0, 2, 4, 8), 64),
    (2048, 8192, (0, 2, 4, 8), 100), (256, 16640, (0, 2, 4, 8), 18)])
def test_prefill_small_adds_what_it_would_store(g, torch, K, N, levels, M):  # noqa: F811
    # accumulating grows y by the overwriting result, bit for bit, whether the
    # halves of K go to two workgroups, to one in turn, or K is not halved
    L = Layer(g, torch, K, N, levels, cfg=98, codes_src=True)
    xd = _dev(torch, inputs.activations_t3(K, M, 98))
    y1 = g.grinqh_prefill(L.desc, L.pc, L.ps, xd)
    base = torch.randn((M, N), generator=torch.Generator("cuda").manual_seed(98), device="cuda")
    y2 = base.clone()
    g.grinqh_prefill(L.desc, L.pc, L.ps, xd, y=y2, accumulate=True)
    assert torch.equal(y2, base + y1)


@pytest.mark.parametrize("levels,K,M,small", [
    ((0, 2, 4, 8), 256, 65, False), ((0, 2, 4, 8), 256, 49, False), ((0, 2, 3, 4, 8), 256, 80, False),
    ((0, 2, 4, 8), 256, 48, True), ((0, 2, 4, 8), 512, 33, False), ((0, 2, 3, 4, 8), 384, 48, False),
    ((0, 2, 4, 8), 512, 32, True)])
def test_prefill_small_leaves_a_second_round_to_the_wide_tiles(g, torch, opts, levels, K, M, small):  # noqa: F811
    # 256 outputs per CU: two rounds of 128-output workgroups, one of 256 x 256
    # tiles, whose sums come in another order
    N = 256 * torch.cuda.get_device_properties(0).multi_processor_count
    L = Layer(g, torch, K, N, levels, cfg=99, codes_src=True)
    xd = _dev(torch, inputs.activations_t3(K, M, 99))
    y = g.grinqh_prefill(L.desc, L.pc, L.ps, xd)
    opts(g.GRINQH_OPT_PREFILL_TILE, 1)
    wide = g.grinqh_prefill(L.desc, L.pc, L.ps, xd)
    assert torch.equal(y, wide) == (not small)
    ref = orc.prefill(L.codes[:512], L.scales[:, :512], inputs.activations_t3(K, M, 99))
    assert np.abs(_host(y)[:, :512] - ref).max() <= 1e-3 * np.abs(ref).max()
