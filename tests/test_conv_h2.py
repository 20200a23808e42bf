"""The two-term fp16 convolution kernel (a launch configuration with waves = 0),
forced where it can go wrong -- remainders of its tiles, patches over several
images and over blocks of one, partial chunks, splits, every window kind --
standalone (a float32 filter) and in plans (converted filters), against the
oracle; and values outside the range its terms hold."""
import numpy as np
import pytest

import oracle as orc
from paper_1809_02697_amd import workloads as wl

from gpu_util import assert_close, dev, gamma, host, rel_l2, torch_cuda

pytestmark = pytest.mark.gpu

TILES = ["4,4", "4,2", "2,4", "2,2"]


@pytest.fixture(scope="module")
def neo():
    torch_cuda()
    from paper_1809_02697_amd import neo as n
    n.lib()
    return n


def run(neo, c, xb=16, yb=16, x=None, w=None):
    """The case through neo_conv2d_nchwxc, the output in NCHW."""
    w = c.w if w is None else w
    bias = c.bias
    if c.bn is not None:
        w, bias = neo.fold_bn(w, bias, c.bn["gamma"], c.bn["beta"], c.bn["mean"], c.bn["var"], c.bn["eps"])
    bp = np.zeros(-(-c.K // 16) * 16, np.float32)
    bp[:c.K] = bias
    x = c.x if x is None else x
    res = None
    if c.epilogue == "res":
        res = neo.layout_transform(dev(c.residual), 0, yb, *c.residual.shape)
    act = "relu" if c.epilogue in ("relu", "res") else "none"
    y = neo.conv2d_nchwxc(neo.layout_transform(dev(x), 0, xb, *x.shape), c.C, neo.pack_filter(dev(w)), c.K, c.R, c.S,
                          bias=dev(bp), stride=c.stride, pad=c.pad, act=act, residual=res, y_block=yb)
    return orc.from_blocked(host(y), c.K)


CASES = [
    # C, K, R, S, stride, pad, H, W, N, epilogue
    (64, 64, 3, 3, 1, 1, 14, 13, 3, "relu"),        # rows of several images per tile
    (17, 40, 3, 3, 2, 1, 13, 11, 2, "res"),         # ragged channels, stride 2
    (80, 96, 1, 1, 1, 0, 9, 7, 3, "res"),           # pointwise, a partial chunk of blocks
    (48, 33, 1, 1, 2, 0, 11, 9, 2, "none"),         # pointwise, stride 2
    (32, 150, 1, 7, 1, (0, 3), 35, 33, 1, "relu"),
    (33, 64, 7, 1, 1, (3, 0), 17, 5, 2, "relu"),
    (16, 16, 5, 5, 1, 2, 7, 7, 5, "res"),           # one block each way, images smaller than a tile
    (96, 200, 3, 3, 1, 1, 40, 40, 1, "relu"),       # blocks of one image
    (5, 20, 3, 3, 1, 0, 5, 5, 1, "none"),           # fewer pixels than one instruction's
    (32, 48, 1, 2, 2, 0, 20, 24, 2, "relu"),        # stride above the window
    (3, 64, 7, 7, 2, 3, 45, 50, 2, "relu"),         # stems: a window of whole column groups and a part of one,
    (1, 20, 3, 3, 1, 1, 12, 9, 3, "res"),           # one channel, rows of several images,
    (4, 40, 5, 5, 2, 2, 21, 11, 2, "relu"),         # four,
    (3, 33, 1, 1, 1, 0, 30, 31, 1, "none"),         # pointwise,
    (2, 16, 5, 1, 2, 1, 70, 33, 1, "relu"),         # stride above the window's width
]


def _case(e, seed=0):
    C, K, R, S, st, pd, H, W, N, epi = e
    ph, pw = pd if isinstance(pd, tuple) else (pd, pd)
    OH, OW = orc.out_size(H, R, st, ph), orc.out_size(W, S, st, pw)
    return wl.conv_case(C, K, R, S, st, pd, H, W, N=N, epilogue=epi, out_hw=(OH, OW), seed=seed)


@pytest.mark.parametrize("e", CASES, ids=[f"C{e[0]}K{e[1]}_{e[2]}x{e[3]}" for e in CASES])
def test_every_tile_and_split(neo, e, monkeypatch):
    """Within the float32 tolerance of the oracle, closer to it than the tile
    kernel's one-chain sum (with 1.5 for the spread of small layers), the
    same bits twice and for other blocks."""
    c = _case(e)
    ref = orc.layer_forward(c)
    monkeypatch.setenv("NEO_CONV_CONFIG", "1,1,1,1")
    tile = rel_l2(run(neo, c), ref)
    for cfg in [f"{t},{sp},0" for t in TILES for sp in (1, 2)]:
        monkeypatch.setenv("NEO_CONV_CONFIG", cfg)
        print(f"\n[h2] {e} {cfg}", flush=True)
        y = run(neo, c)
        err = assert_close(y, ref, cfg)
        assert err <= 1.5 * max(tile, 2e-8), (err, tile)
        np.testing.assert_array_equal(run(neo, c), y)
        for xb, yb in [(32, 16), (16, 64)] + ([(1, 16), (4, 32)] if c.C <= 4 else []):
            np.testing.assert_array_equal(run(neo, c, xb, yb), y, err_msg=f"{cfg} {xb}/{yb}")


@pytest.mark.parametrize("e", CASES, ids=[f"C{e[0]}K{e[1]}_{e[2]}x{e[3]}" for e in CASES])
def test_plan_with_converted_filters(neo, e, tmp_path):
    """Plans whose results file names the kernel: every tile and a split,
    against the oracle; a second run and a replayed graph give the same bits."""
    C, K, R, S, st, pd, H, W, N, epi = e
    ph, pw = pd if isinstance(pd, tuple) else (pd, pd)
    g = wl.Graph(name="one", input_shape=(N, C, H, W))
    c = _case(e, 3)
    g.nodes = [wl.Node(op="input"),
               wl.Node(op="conv", inputs=(0,), K=K, R=R, S=S, stride=(st, st), pad=(ph, pw), act="relu", w=c.w,
                       bias=c.bias, bn=c.bn),
               wl.Node(op="output", inputs=(1,))]
    g.x = c.x
    ref = orc.run_graph(g)
    for cfg in [f"{t} 1 0" for t in TILES] + ["4 2 2 0"]:
        neo.tune_db_clear()
        path = tmp_path / "db.txt"
        path.write_text(f"gfx950 {N} {C} {H} {W} {K} {R} {S} {st} {st} {ph} {pw} 1 16 16 {cfg.replace(',', ' ')} 1.0\n")
        assert neo.tune_db_load(path) == 1
        print(f"\n[h2 plan] {e} {cfg}", flush=True)
        p = neo.Plan(g, flags=neo.PLAN_HIPGRAPH)
        conv = [s for s in p.describe()["steps"] if s["kind"] == "conv"][0]["conv"]
        if C > 4 or not cfg.endswith(" 2 0"):
            assert conv["waves"] == 0 and conv["tuned"]
        x = dev(g.x)
        y = host(p.run(x))
        assert_close(y, ref.reshape(y.shape), cfg)
        for _ in range(2):
            np.testing.assert_array_equal(host(p.run(x)), y)
        p.destroy()
    neo.tune_db_clear()


def _both(neo, c, monkeypatch, cfg, **kw):
    monkeypatch.setenv("NEO_CONV_CONFIG", "1,1,1,1")
    t = run(neo, c, **kw)
    monkeypatch.setenv("NEO_CONV_CONFIG", cfg)
    return t, run(neo, c, **kw)


@pytest.mark.parametrize("cfg", ["4,4,1,0", "2,2,2,0"])
def test_infinities_and_nans(neo, cfg, monkeypatch):
    """Infinite and NaN inputs and weights, and the largest float: the same
    non-finite outputs as the tile kernel, the finite ones within tolerance."""
    for kind in range(6):
        C = 3 if kind > 2 else 40
        if C == 3 and "2,0" in cfg:
            break
        c = wl.conv_case(C, 48, 3, 3, 1, 1, 12, 12, N=2, epilogue="none", with_bn=False)
        x, w = c.x.copy(), c.w.copy()
        if kind % 3 == 0:
            x[0, 2, 4, 5], x[1, C - 1, 0, 0], x[1, 1, 11, 11] = np.inf, np.nan, -np.inf
        elif kind % 3 == 1:
            w[7, 2, 1, 1], w[40, 1, 0, 2] = np.inf, np.nan
        else:
            x[0, 1, 6, 6] = np.finfo(np.float32).max
        print(f"\n[h2 non-finite] {cfg} {kind}", flush=True)
        t, y = _both(neo, c, monkeypatch, cfg, x=x, w=w)
        np.testing.assert_array_equal(np.isnan(y), np.isnan(t))
        np.testing.assert_array_equal(np.isinf(y), np.isinf(t))
        np.testing.assert_array_equal(y[np.isinf(y)], t[np.isinf(y)])
        ok = np.isfinite(y)
        assert ok.sum() > y.size // 2
        # (two orders of a 360-term float32 sum)
        assert (np.abs(y[ok] - t[ok]) <= 2 * gamma(364) * 40 * np.maximum(1, np.abs(x[np.isfinite(x)]).max())).all()


@pytest.mark.parametrize("cfg", ["4,4,1,0", "2,4,1,0"])
def test_range_of_values(neo, cfg, monkeypatch):
    """Inputs far from unit scale: all tiny, all huge, one pixel 10^9 times the
    rest (beyond the range of the sampled scale), magnitudes over six decades
    with weights that undo them, and zeros.  Element-wise within the a-priori
    bound of a float32 sum."""
    c = wl.conv_case(64, 48, 3, 3, 1, 1, 16, 16, N=2, epilogue="none", with_bn=False)
    c.bias = np.zeros_like(c.bias)
    decades = np.float32(10.0) ** np.linspace(-6, 0, 64).astype(np.float32)
    spike = c.x.copy()
    spike[1, 33, 9, 9] *= np.float32(1e9)
    cases = [("tiny", c.x * np.float32(1e-20), c.w), ("huge", c.x * np.float32(1e20), c.w), ("spike", spike, c.w),
             ("decades", c.x * decades[None, :, None, None], c.w / decades[None, :, None, None]),
             ("small weights", c.x, c.w * np.float32(1e-25)), ("zeros", np.zeros_like(c.x), c.w),
             ("late", c.x * (np.arange(64) >= 40).astype(np.float32)[None, :, None, None], c.w)]
    for name, x, w in cases:
        x, w = x.astype(np.float32), w.astype(np.float32)
        monkeypatch.setenv("NEO_CONV_CONFIG", cfg)
        print(f"\n[h2 range] {cfg} {name}", flush=True)
        y = run(neo, c, x=x, w=w).astype(np.float64)
        xp = np.pad(x.astype(np.float64), ((0, 0), (0, 0), (1, 1), (1, 1)))
        win = np.lib.stride_tricks.sliding_window_view(xp, (3, 3), axis=(2, 3))
        w64 = w.astype(np.float64)
        ref = np.einsum("nchwrs,kcrs->nkhw", win, w64)
        cond = np.einsum("nchwrs,kcrs->nkhw", np.abs(win), np.abs(w64))
        bound = gamma(580) * cond
        bad = np.abs(y - ref) > bound + np.finfo(np.float32).tiny
        assert not bad.any(), (name, int(bad.sum()), float((np.abs(y - ref) / np.maximum(bound, 1e-300)).max()))


def test_refused_where_it_does_not_apply(neo, tmp_path):
    """A window whose patch exceeds the workgroup's keeps the tile kernel
    whatever the results file says."""
    for C, R, H in ((8, 25, 64),):
        neo.tune_db_clear()
        g = wl.Graph(name="one", input_shape=(1, C, H, H))
        c = wl.conv_case(C, 16, R, R, 1, 0, H, H)
        g.nodes = [wl.Node(op="input"), wl.Node(op="conv", inputs=(0,), K=16, R=R, S=R, w=c.w, bias=c.bias),
                   wl.Node(op="output", inputs=(1,))]
        path = tmp_path / "db.txt"
        path.write_text(f"gfx950 1 {C} {H} {H} 16 {R} {R} 1 1 0 0 1 16 16 4 4 1 0 1.0\n")
        assert neo.tune_db_load(path) == 1
        p = neo.Plan(g)
        conv = [s for s in p.describe()["steps"] if s["kind"] == "conv"][0]["conv"]
        assert conv["waves"] > 0 and not conv["tuned"]
        y = host(p.run(dev(c.x)))
        g.x = c.x
        assert_close(y, orc.run_graph(g).reshape(y.shape), f"C{C} R{R}")
        p.destroy()
    neo.tune_db_clear()
