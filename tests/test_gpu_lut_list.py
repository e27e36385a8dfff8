"""LUT VMM: the sorted channel list at its edges (empty, full, level borders)."""
import numpy as np
import pytest

from synth import inputs
from test_gpu_parity import LutLayer, _dev, _host, g, opts, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# channels of each level, in runs of the given lengths (the rest at level 0):
# one entry, a wave's 16 rows, the workgroup's 64, one more and one fewer, a
# border inside a wave, the last round of the ring of four
RUNS = [(1,), (0, 1), (16, 16), (15, 17), (64,), (63, 2), (65, 64, 63), (128, 100, 28), (0, 0, 256),
        (257, 1, 1)]


@pytest.mark.parametrize("K,levels,tile_n", [
    (128, (0, 2, 4, 8), 256), (640, (0, 2, 4, 6, 8), 512), (2176, (0, 2, 4, 6), 256),
    (640, (0, 1, 2, 3, 4, 5, 6, 7, 8), 512), (384, (0, 1, 3, 6), 512), (640, (0, 2, 3, 4, 8), 512)])
@pytest.mark.parametrize("gps", [1, 4, 16])
def test_lut_list_edges(g, torch, opts, K, levels, tile_n, gps):  # noqa: F811
    opts(g.GRINQH_OPT_LUT_GROUPS, str(gps))
    N = 512
    L = LutLayer(g, torch, K, N, levels, layer=K + gps, tile_n=tile_n)
    rng = np.random.default_rng(K + gps)
    for runs in RUNS:
        x = inputs.activations_t3(K, 2, 97, len(runs))
        lm = np.zeros((2, K), dtype=np.uint8)
        for t in range(2):
            order, at = rng.permutation(K), 0
            for j, n in enumerate(runs):
                lm[t, order[at:at + n]] = min(j + 1 + t, len(levels) - 1)
                at += n
        # level-0 channels take no part, whatever they hold
        x[lm == 0] = np.inf
        y = L.run(g, torch, x, lm)
        x[lm == 0] = 0
        ref = L.ref(x, lm)
        # fp32 sums of exact products: (K + 8) 2^-24 sum |x| |table value|
        top = max(np.abs(t.astype(np.float64)).max() for t in L.tables.values())
        bound = (K + 8) * 2.0 ** -24 * top * np.abs(x.astype(np.float64)).sum(axis=1, keepdims=True)
        assert np.all(np.abs(y - ref) <= bound), (runs, np.max(np.abs(y - ref) / np.maximum(bound, 1e-30)))


@pytest.mark.parametrize("B", [2, 3, 7, 8, 9, 11, 16, 17, 33])
@pytest.mark.parametrize("K,N,levels,tile_n,gps", [
    (640, 1536, (0, 2, 4, 8), 512, 2), (384, 1024, (0, 2, 4, 6, 8), 1024, 1), (256, 768, (0, 2, 4), 256, 16),
    (384, 1536, (0, 2, 3, 4, 8), 512, 2), (512, 2048, (0, 2, 4), 2048, 3)])
def test_lut_tokens_side_by_side(g, torch, opts, K, N, levels, tile_n, gps, B):  # noqa: F811
    # up to eight tokens share a row of workgroups; where the tokens don't fill the
    # last row its spare workgroups leave.  Every token, tile, sub-tile and split, and the
    # level map that the first sub-tile's workgroups write
    opts(g.GRINQH_OPT_LUT_GROUPS, str(gps))
    L = LutLayer(g, torch, K, N, levels, layer=K + N, tile_n=tile_n)
    x = inputs.activations_t3(K, B, 98)
    th = np.quantile(np.abs(x.astype(np.float64)), np.linspace(0.2, 0.8, len(levels) - 1)).astype(np.float32)
    lm = (np.abs(x.astype(np.float32))[:, :, None] >= th).sum(axis=2).astype(np.uint8)
    ref = L.ref(x, lm)
    top = max(np.abs(t.astype(np.float64)).max() for t in L.tables.values())
    bound = (K + 8) * 2.0 ** -24 * top * np.abs(x.astype(np.float64)).sum(axis=1, keepdims=True)
    y = L.run(g, torch, x, lm)
    assert np.all(np.abs(y - ref) <= bound)
    lo = torch.full((B, K), 255, dtype=torch.uint8, device="cuda")
    buf = torch.full((B + 1, N), 7.0, device="cuda")
    g.grinqh_vmm_lut_threshold(L.desc, L.pc, L.luts, _dev(torch, x), th, y=buf[:B], level_map_out=lo)
    assert np.all(np.abs(_host(buf)[:B] - ref) <= bound) and bool((buf[B:] == 7.0).all())
    assert np.array_equal(_host(lo), lm)
