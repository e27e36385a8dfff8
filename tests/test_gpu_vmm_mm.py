"""The matrix-core decode VMM at the edges of its lists, passes and columns."""
import types

import numpy as np
import pytest

from oracle import grinqh_oracle as orc
from synth import inputs
from test_gpu_parity import Layer, _dev, _host, g, opts, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _maps(kind, B, K, top, seed):
    r = np.random.default_rng(seed)
    lm = np.zeros((B, K), np.uint8)
    if kind == "full":                        # every row to full depth: a second pass
        lm[:] = top
    elif kind == "uneven":                    # one list of 32 channels full, its neighbours empty
        lm[:, 32:64] = top
        lm[:, 128 + 96:128 + 128] = top
    elif kind == "one":                       # a single row
        lm[:, K - 1] = 1
    elif kind == "random":                    # every depth, tokens of their own
        lm[:] = r.integers(0, top + 1, size=(B, K))
    return lm


def _bound(L, x, lm, u):
    """Per output: a unit of X is 2^-24 of a power of two at most twice the
    group's largest active |x| (2^-23 for 1-bit planes); what a group's X leave
    of x is at most half a unit per channel and two in all, times a weight of
    at most 128 (8-bit units); and a group's sum takes fewer than 16 float32
    roundings of sums of x times codes of at most 255, plus one per group in
    the adds."""
    G = L.K // 128
    xa = np.abs(x.astype(np.float64)) * (lm > 0)
    xa = xa.reshape(-1, G, 128)
    left = np.minimum((lm.reshape(-1, G, 128) > 0).sum(2), 4) / 2
    per = left * xa.max(2) * (2 if u == 1 else 1) + (16 + G) * xa.sum(2)
    s = L.scales.astype(np.float64) * 2.0 ** (L.b_max - 8)
    return 2.0 ** -24 * 255 * per @ s


@pytest.mark.parametrize("kind", ["full", "uneven", "one", "empty", "random"])
@pytest.mark.parametrize("K,N,levels,tile_n,B", [
    (256, 256, (0, 2, 4, 8), 256, 1), (256, 1024, (0, 2, 4, 6, 8), 512, 4),
    (384, 1024, (0, 2, 4, 6, 8), 1024, 2), (256, 2048, (0, 2, 4, 6), 2048, 3),
    (256, 512, (0, 2, 4), 256, 4), (256, 1536, (0, 2, 4), 512, 1),
    (256, 1024, (0, 2, 3, 4, 8), 512, 1), (256, 1024, (0, 2, 3, 4, 8), 1024, 4),
    (256, 1024, (0, 1, 2, 3, 4), 512, 3), (256, 2048, (0, 1, 3, 6), 2048, 2)])
def test_vmm_mm_lists(g, torch, kind, K, N, levels, tile_n, B):  # noqa: F811
    L = Layer(g, torch, K, N, levels, cfg=90, tile_n=tile_n, codes_src=True)
    x = inputs.activations_t3(K, B, 90)
    lm = _maps(kind, B, K, len(levels) - 1, 90)
    y = g.grinqh_vmm(L.desc, L.pc, L.ps, _dev(torch, x), _dev(torch, lm))
    ref = orc.vmm_batch(L.codes, L.scales, x, lm, levels)
    err = np.abs(_host(y) - ref)
    assert np.all(err <= _bound(L, x, lm, L.desc.plane_bits)), (err.max(), np.abs(ref).max())


@pytest.mark.parametrize("K,N,levels,tile_n,run,full", [
    (128, 1536 * 256, (0, 2, 4, 8), 256, 2, False), (128, 1537 * 256, (0, 2, 4, 8), 256, 3, False),
    (1024, 97 * 512, (0, 2, 4, 6, 8), 512, 2, True), (1024, 98 * 512, (0, 2, 4, 6), 1024, 2, True),
    (512, 259 * 512, (0, 2, 4, 6, 8), 512, 2, False), (1024, 97 * 512, (0, 2, 4), 512, 2, True),
    (1024, 97 * 512, (0, 2, 3, 4, 8), 512, 2, True), (512, 259 * 512, (0, 2, 3, 4, 8), 512, 2, False),
    (1152, 88 * 512, (0, 2, 3, 4, 8), 1024, 2, True)])
def test_vmm_mm_columns_per_workgroup(g, torch, opts, K, N, levels, tile_n, run, full):  # noqa: F811
    # several columns per workgroup, the last workgroup with fewer where their
    # number leaves a remainder; a second pass over a column (512 outputs, full
    # depth) or LDS for all of it (at most two workgroups per CU).  `run` and
    # `full` are the launcher's rule for 256 CUs, stated here again.
    width, groups = min(tile_n, 512), K // 128
    cols, r = N // width, 1
    while -(-cols // r) * groups > 3 * 256:
        r += 1
    assert r == run and (-(-cols // r) * groups <= 2 * 256) == full
    L = Layer(g, torch, K, N, levels, cfg=91, tile_n=tile_n, codes_src=True)
    opts(g.GRINQH_OPT_GROUPS_PER_WG, 1)       # this kernel, whatever the layer's size
    x = inputs.activations_t3(K, 1, 91)
    idx = np.unique(np.concatenate([np.arange(0, N, 37), np.arange(N - width, N)]))   # some of every column
    part = types.SimpleNamespace(K=K, b_max=L.b_max, scales=np.ascontiguousarray(L.scales[:, idx]))
    codes = np.ascontiguousarray(L.codes[idx])
    for kind in ("full", "uneven", "random", "empty"):
        lm = _maps(kind, 1, K, len(levels) - 1, 91)
        y = _host(g.grinqh_vmm(L.desc, L.pc, L.ps, _dev(torch, x), _dev(torch, lm)))[:, idx]
        ref = orc.vmm_batch(codes, part.scales, x, lm, levels)
        err, bound = np.abs(y - ref), _bound(part, x, lm, L.desc.plane_bits)
        assert np.all(err <= bound), (kind, np.max(err / np.maximum(bound, 1e-300)))


@pytest.mark.parametrize("levels,B", [((0, 2, 4, 6, 8), 1), ((0, 2, 4, 6, 8), 3), ((0, 2, 3, 4, 8), 2)])
def test_vmm_mm_skipped_and_non_finite(g, torch, levels, B):  # noqa: F811
    # a skipped channel leaves no trace, however large or non-finite its x; an
    # active infinity or NaN reaches every output of its token and no other
    K, N = 256, 1024
    L = Layer(g, torch, K, N, levels, cfg=92, codes_src=True)
    x = (inputs.activations_t3(K, B, 92) * np.float16(1e-3)).astype(np.float16)
    lm = _maps("random", B, K, len(levels) - 1, 92)
    lm[:, [5, 70, 200]] = 0
    lm[:, 9] = 2
    ref = orc.vmm_batch(L.codes, L.scales, np.where(lm > 0, x, 0).astype(np.float16), lm, levels)
    bound = _bound(L, x, lm, L.desc.plane_bits)
    big = x.copy()
    big[:, 5], big[:, 70], big[:, 200] = 60000.0, np.inf, np.nan
    y = _host(g.grinqh_vmm(L.desc, L.pc, L.ps, _dev(torch, big), _dev(torch, lm)))
    assert np.all(np.abs(y - ref) <= bound)
    for v in (np.inf, -np.inf, np.nan):
        bad = big.copy()
        bad[0, 9] = v
        y = _host(g.grinqh_vmm(L.desc, L.pc, L.ps, _dev(torch, bad), _dev(torch, lm)))
        assert not np.isfinite(y[0]).any()
        assert np.all(np.abs(y[1:] - ref[1:]) <= bound[1:])


WIDE = [(256, 256, (0, 2, 4, 8), 256, 1), (256, 1024, (0, 2, 4, 6, 8), 1024, 1), (256, 512, (0, 2, 4, 6, 8), 512, 4),
        (384, 512, (0, 2, 4), 512, 2), (256, 2048, (0, 2, 4, 6), 2048, 3),
        (256, 1024, (0, 2, 3, 4, 8), 512, 1), (256, 1024, (0, 2, 3, 4, 8), 1024, 4), (256, 512, (0, 1, 2, 3, 4), 512, 2)]


@pytest.mark.parametrize("small", ["half", "ramp", "wide"])
@pytest.mark.parametrize("K,N,levels,tile_n,B,mode", [w + (m,) for w in WIDE for m in ("map", "threshold")] +
                         [w + ("topk",) for w in WIDE[:2]])
def test_vmm_mm_wide_range_in_a_group(g, torch, K, N, levels, tile_n, B, small, mode):  # noqa: F811
    # one channel of a group far above the others, its weight near zero: the
    # others' x has to reach the sums although it is below the units of the
    # largest one's 24 bits (all of one sign and to one side, so that losses add up)
    L = Layer(g, torch, K, N, levels, cfg=100, tile_n=tile_n, codes_src=True)
    top, half = len(levels) - 1, 1 << (L.b_max - 1)
    L.codes[:, 5] = half
    L.pc, L.ps = g.grinqh_pack(L.desc, codes=_dev(torch, L.codes),
                               scales=_dev(torch, np.ascontiguousarray(L.scales.T)))
    r = np.random.default_rng(100)
    x = np.zeros((B, K), np.float16)
    unit = 2.0 ** (-8 if L.desc.plane_bits == 2 else -7)      # of X beside 32768
    for t in range(B):
        x[t] = {"half": np.full(K, unit / 2), "ramp": unit * np.linspace(0.1, 9.6, K),
                "wide": unit * np.exp2(r.uniform(-14, 8, K))}[small].astype(np.float16)
        x[t, 5] = 32768.0 if t < 3 else 2.0 ** -3             # (the last token: an ordinary range)
    xd = _dev(torch, x)
    if mode == "map":
        lm = np.full((B, K), top, np.uint8)
        lm[:, K - 1] = 0
        lm[:, 40:60] = r.integers(0, top + 1, size=(B, 20))
        y = g.grinqh_vmm(L.desc, L.pc, L.ps, xd, _dev(torch, lm))
    elif mode == "threshold":
        th = np.quantile(np.abs(x[0].astype(np.float64)), np.linspace(0.05, 0.4, top)).astype(np.float32)
        lm = orc.assign_threshold(x, th)
        y = g.grinqh_vmm_threshold(L.desc, L.pc, L.ps, xd, th)
    else:
        counts = g.grinqh_topk_counts(K, [500] + [9500 // top] * (top - 1) + [9500 - 9500 // top * (top - 1)])
        lm = orc.assign_topk(x, counts)
        y = g.grinqh_vmm_topk(L.desc, L.pc, L.ps, xd, counts)
    ref = orc.vmm_batch(L.codes, L.scales, x, lm, levels)
    err = np.abs(_host(y) - ref)
    bound = _bound(L, x, lm, L.desc.plane_bits)
    assert np.all(err <= bound), (np.max(err / bound), np.abs(ref).max())


@pytest.mark.parametrize("tile_n,levels,units,mm", [
    (256, (0, 2, 4, 8), 768, True), (512, (0, 2, 4, 6), 768, True), (512, (0, 2, 4), 768, True),
    (512, (0, 2, 4, 8), 768, False), (1024, (0, 2, 4, 6), 768, False), (1024, (0, 2, 4, 8), 767, True)])
def test_batch1_kernel_by_size(g, torch, opts, tile_n, levels, units, mm):  # noqa: F811
    # one group, so one add per output: the two kernels' sums are told apart by
    # their bits (`units` for 256 CUs)
    K, N = 128, units * tile_n
    L = Layer(g, torch, K, N, levels, cfg=101, tile_n=tile_n, codes_src=True)
    x, lm = inputs.activations_t3(K, 1, 101), _maps("random", 1, K, len(levels) - 1, 101)

    def call(force):
        opts(g.GRINQH_OPT_GROUPS_PER_WG, force)
        return g.grinqh_vmm(L.desc, L.pc, L.ps, _dev(torch, x), _dev(torch, lm))

    y = call(0)
    assert torch.equal(y, call(1)) == mm and torch.equal(y, call(2)) == (not mm)
    idx = np.unique(np.concatenate([np.arange(0, N, 97), np.arange(N - tile_n, N)]))
    ref = orc.vmm_batch(np.ascontiguousarray(L.codes[idx]), np.ascontiguousarray(L.scales[:, idx]), x, lm, levels)
    assert np.abs(_host(y)[:, idx] - ref).max() <= 1e-4 * np.abs(ref).max()
