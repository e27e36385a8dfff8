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
