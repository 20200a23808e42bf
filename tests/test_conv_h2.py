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
    (1, 20, 7, 7, 1, 3, 12, 9, 3, "res"),           # one channel, rows of several images,
    (4, 40, 5, 5, 2, 2, 21, 11, 2, "relu"),         # four,
    (4, 33, 2, 3, 1, 0, 30, 31, 1, "none"),         # the shortest reduction,
    (3, 16, 9, 1, 2, 1, 70, 33, 1, "relu"),         # stride above the window's width
]


def assert_two_term(neo, c, xb=16, yb=16):
    """The configuration that is set runs the two-term kernel for this case:
    one product per output of a = 1 + r with itself, whose r^2 (two units of the
    last place) only a float32 product holds."""
    r = np.float32(2.0 ** -11 - 2.0 ** -18)
    a = np.float32(1) + r
    one = wl.conv_case(c.C, c.K, c.R, c.S, c.stride, c.pad, c.H, c.W, N=c.N, epilogue="none", with_bn=False)
    one.bias = np.zeros_like(one.bias)
    w = np.zeros_like(one.w)
    w[:, 0, c.R // 2, c.S // 2] = a
    y = run(neo, one, xb, yb, x=np.full_like(one.x, a), w=w)
    y = y[y != 0]
    assert y.size and (y == np.float32(1) + 2 * r).all()


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
    for cfg in [f"{t},{sp},0" for t in TILES for sp in ((1, 2) if c.C > 4 else (1,))]:
        monkeypatch.setenv("NEO_CONV_CONFIG", cfg)
        print(f"\n[h2] {e} {cfg}", flush=True)
        assert_two_term(neo, c)
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
    for cfg in [f"{t} 1 0" for t in TILES] + (["4 2 2 0"] if C > 4 else []):
        neo.tune_db_clear()
        path = tmp_path / "db.txt"
        path.write_text(f"gfx950 {N} {C} {H} {W} {K} {R} {S} {st} {st} {ph} {pw} 1 16 16 {cfg.replace(',', ' ')} 1.0\n")
        assert neo.tune_db_load(path) == 1
        print(f"\n[h2 plan] {e} {cfg}", flush=True)
        p = neo.Plan(g, flags=neo.PLAN_HIPGRAPH)
        conv = [s for s in p.describe()["steps"] if s["kind"] == "conv"][0]["conv"]
        assert conv["waves"] == 0 and conv["tuned"]
        x = dev(g.x)
        y = host(p.run(x))
        assert_close(y, ref.reshape(y.shape), cfg)
        for _ in range(2):
            np.testing.assert_array_equal(host(p.run(x)), y)
        p.destroy()
    neo.tune_db_clear()


def reference(x, w, stride, pad):
    """The convolution in float64, and every output's sum of its terms'
    magnitudes.  Infinities and NaN count as zeros in the latter."""
    ph, pw = pad if isinstance(pad, tuple) else (pad, pad)
    sh, sw = stride if isinstance(stride, tuple) else (stride, stride)
    xp = np.pad(x.astype(np.float64), ((0, 0), (0, 0), (ph, ph), (pw, pw)))
    win = np.lib.stride_tricks.sliding_window_view(xp, w.shape[2:], axis=(2, 3))[:, :, ::sh, ::sw]
    N, C, OH, OW, R, S = win.shape
    win = win.transpose(0, 2, 3, 1, 4, 5).reshape(N * OH * OW, C * R * S)
    w64 = w.astype(np.float64).reshape(len(w), -1).T
    def layer(a, b):
        return (a @ b).reshape(N, OH, OW, -1).transpose(0, 3, 1, 2)
    def finite(a):
        return np.where(np.isfinite(a), np.abs(a), 0.0)
    with np.errstate(invalid="ignore", over="ignore"):
        return layer(win, w64), layer(finite(win), finite(w64))


def spread(y, ref, cond, n, what):
    """Every finite output lies within the a-priori bound of a float32 sum of
    its own n terms (12 units for the operands' two terms and the dropped
    product, 16 for small operands, 4 for the scales and the epilogue), however
    large the values outside its window; the error's rms in units of the terms'
    magnitude."""
    ok = np.isfinite(ref) & np.isfinite(y) & (cond < 2.0 ** 127)
    assert ok.sum() > y.size // 4, what
    assert np.isfinite(y[np.isfinite(ref) & (cond < 2.0 ** 127)]).all(), what
    err = np.abs(y[ok].astype(np.float64) - ref[ok])
    bound = gamma(n + 32) * cond[ok] + n * 2.0 ** -149
    bad = err > bound
    assert not bad.any(), (what, int(bad.sum()), float((err / np.maximum(bound, 1e-300)).max()))
    normal = cond[ok] > 2.0 ** -100
    rel = err[normal] / cond[ok][normal]
    return float(np.sqrt(np.mean(rel ** 2))) if rel.size else 0.0


def wide_cases(c, seed=0):
    """(name, x, w) whose magnitudes differ across pixels, images, channels,
    filters and single values by more than the two terms hold."""
    rng = np.random.default_rng([seed, c.C, c.K])
    f32 = np.float32
    x, w, C, K = c.x, c.w, c.C, c.K
    last = C - max(C // 4, 1)  # channels that the sampled scale does not see where there are several blocks
    chan = (np.arange(C) >= last).astype(f32)[None, :, None, None]
    def decades(lo, hi, shape):
        return (f32(10.0) ** rng.uniform(lo, hi, shape)).astype(f32)
    def at(v, ch):
        z = x.copy()
        z[0, ch, x.shape[2] // 2, x.shape[3] // 2] = v
        return z
    def entry(v, ch):
        z = w.copy()
        z[5, ch, 0, 0] = v
        return z
    yield "as drawn", x, w
    yield "zeros", x * f32(0), w
    yield "zero weights", x, w * f32(0)
    yield "tiny", x * f32(1e-20), w
    yield "huge", x * f32(1e20), w
    yield "small weights", x, w * f32(1e-25)
    for v in (1e9, -1e15, np.finfo(f32).max, np.finfo(f32).min):
        yield f"pixel {v:.0e}, first channel", at(v, 0), w
        yield f"pixel {v:.0e}, last channel", at(v, C - 1), w
    yield "infinity beside small values", at(np.inf, 0) * f32(1e-8), w
    yield "NaN beside small values", at(np.nan, 0) * f32(1e-8), w
    for s in (1e-5, 1e-10, 1e-25, 1e15):
        yield f"images by {s:.0e}", x * np.array([1.0] + [s] * (len(x) - 1), f32)[:, None, None, None], w
    for s in (1e-12, 1e-8, 1.0, 1e8):
        yield f"last channels only, {s:.0e}", x * chan * f32(s), w
    for s in (40.0, 1e6, 1e20):
        yield f"last channels {s:.0e} times the rest", x * (1 + chan * f32(s)), w
    for d in (3, 6, 15):
        k = decades(-d, d, (1, C, 1, 1))
        yield f"channels over {2 * d} decades, weights that undo them", x * k, w / k
        yield f"pixels over {2 * d} decades", x * decades(-d, d, (x.shape[0], 1) + x.shape[2:]), w
        yield f"filters over {2 * d} decades", x, w * decades(-d, d, (K, 1, 1, 1))
        yield f"inputs over {2 * d} decades", x * decades(-d, d, x.shape), w
        yield f"weights over {2 * d} decades", x, w * decades(-d, d, w.shape)
    yield "last weights only", x, w * chan * f32(1e-12)
    yield "last weights 1e9 times the rest", x, w * (1 + chan * f32(1e9))
    yield "one weight 1e12", x, entry(1e12, C - 1)
    yield "one weight 1e-12", x, entry(1e-12, 0)
    few = x.copy()
    few[rng.random(x.shape) < 0.6] = 0
    few[rng.random(x.shape) < 2e-3] *= f32(1e-9)
    yield "half zeros and a few small values", few, w


WIDE = [
    # C, K, R, S, stride, pad, H, W, N
    (64, 40, 3, 3, 1, 1, 12, 13, 2),
    (200, 40, 1, 1, 1, 0, 9, 11, 3),     # pointwise, a partial chunk of blocks
    (33, 64, 1, 7, 1, (0, 3), 11, 24, 2),
    (3, 40, 7, 7, 2, 3, 33, 30, 2),      # stems
    (4, 24, 3, 3, 1, 1, 17, 12, 3),
]


def _wide(e):
    C, K, R, S, st, pd, H, W, N = e
    c = wl.conv_case(C, K, R, S, st, pd, H, W, N=N, epilogue="none", with_bn=False)
    c.bias = np.zeros_like(c.bias)
    return c


def _tuned_plan(neo, c, w, cfg, tmp_path):
    """A plan of the one layer whose results file names configuration cfg."""
    g = wl.Graph(name="one", input_shape=c.x.shape)
    g.nodes = [wl.Node(op="input"),
               wl.Node(op="conv", inputs=(0,), K=c.K, R=c.R, S=c.S, stride=c.stride, pad=c.pad, w=w, bias=c.bias),
               wl.Node(op="output", inputs=(1,))]
    neo.tune_db_clear()
    path = tmp_path / "db.txt"
    N, C, H, W = c.x.shape
    path.write_text(f"gfx950 {N} {C} {H} {W} {c.K} {c.R} {c.S} {c.stride[0]} {c.stride[1]} {c.pad[0]} {c.pad[1]} "
                    f"1 16 16 {cfg.replace(',', ' ')} 1.0\n")
    assert neo.tune_db_load(path) == 1
    p = neo.Plan(g)
    conv = [s for s in p.describe()["steps"] if s["kind"] == "conv"][0]["conv"]
    neo.tune_db_clear()
    assert conv["tuned"]
    return p, conv


@pytest.mark.parametrize("e", WIDE, ids=[f"C{e[0]}K{e[1]}_{e[2]}x{e[3]}" for e in WIDE])
def test_range_of_values(neo, e, monkeypatch, tmp_path):
    """Operands of any range, from a float32 filter and from converted terms:
    every output within the bound of a float32 sum of its own terms, and as
    close to 64 bits as the float32 kernel's (1.5 for the spread)."""
    c = _wide(e)
    n = c.C * c.R * c.S
    for name, x, w in wide_cases(c):
        x, w = x.astype(np.float32), w.astype(np.float32)
        ref, cond = reference(x, w, c.stride, c.pad)
        monkeypatch.setenv("NEO_CONV_CONFIG", "1,1,1,1")
        t = run(neo, c, x=x, w=w)
        tile = spread(t, ref, cond, n, ("tile", name))
        for cfg in ["4,4,1,0", "2,2,1,0"] + (["2,4,2,0", "4,2,2,0"] if c.C > 4 else []):
            monkeypatch.setenv("NEO_CONV_CONFIG", cfg)
            print(f"\n[h2 range] {e} {cfg} {name}", flush=True)
            y = run(neo, c, x=x, w=w)
            p, conv = _tuned_plan(neo, c, w, cfg, tmp_path)
            assert conv["waves"] == 0
            z = host(p.run(dev(x))).reshape(y.shape)
            p.destroy()
            if cfg.endswith(",1,0"):  # the same tiles again in float32, whatever the blocks
                for xb, yb in [(32, 16), (16, 64)] if c.C > 4 else [(1, 16), (4, 32)]:
                    np.testing.assert_array_equal(run(neo, c, xb, yb, x=x, w=w), y, err_msg=f"{name} {cfg} {xb}/{yb}")
            for how, v in (("float32 filter", y), ("converted filter", z)):
                what = (name, cfg, how)
                np.testing.assert_array_equal(np.isnan(v), np.isnan(t), err_msg=str(what))
                if cfg.split(",")[2] == "1":  # (partial sums overflow elsewhere)
                    np.testing.assert_array_equal(v[np.isinf(t)], t[np.isinf(t)], err_msg=str(what))
                rms = spread(v, ref, cond, n, what)
                assert rms <= 1.5 * max(tile, 2.0 ** -24), (what, rms, tile)


@pytest.mark.parametrize("cfg", ["4,4,1,0", "2,2,2,0"])
def test_infinities_and_nans(neo, cfg, monkeypatch, tmp_path):
    """Infinite and NaN inputs and weights: the same non-finite outputs as the
    tile kernel, the finite ones within the bound of their own terms; from
    both forms of the filter, for blocks of channels and stems."""
    for kind in range(4):
        C = 3 if kind > 1 else 40
        if C == 3 and "2,0" in cfg:
            break
        c = wl.conv_case(C, 40, 5, 5, 1, 2, 12, 12, N=2, epilogue="none", with_bn=False)
        c.bias = np.zeros_like(c.bias)
        x, w = c.x.copy(), c.w.copy()
        if kind % 2 == 0:
            x[0, 2, 4, 5], x[1, C - 1, 0, 0], x[1, 1, 11, 11] = np.inf, np.nan, -np.inf
        else:
            w[7, 2, 1, 1], w[30, 1, 0, 2] = np.inf, np.nan
        print(f"\n[h2 non-finite] {cfg} {kind}", flush=True)
        monkeypatch.setenv("NEO_CONV_CONFIG", "1,1,1,1")
        t = run(neo, c, x=x, w=w)
        monkeypatch.setenv("NEO_CONV_CONFIG", cfg)
        y = run(neo, c, x=x, w=w)
        p, conv = _tuned_plan(neo, c, w, cfg, tmp_path)
        assert conv["waves"] == 0
        z = host(p.run(dev(x))).reshape(y.shape)
        p.destroy()
        ref, cond = reference(x, w, 1, 2)
        for v in (y, z):
            np.testing.assert_array_equal(np.isnan(v), np.isnan(t))
            np.testing.assert_array_equal(np.isinf(v), np.isinf(t))
            np.testing.assert_array_equal(v[np.isinf(v)], t[np.isinf(t)])
            assert spread(v, np.where(np.isfinite(v), ref, np.nan), cond, C * 25, (cfg, kind)) < 2.0 ** -21


def test_search_times_ordinary_values(neo):
    """The local search times its launches over activations of ordinary values
    (a two-term launch's time depends on them), not over what the allocation
    held or the launches before it left: a later conv alone, after it, sums
    inputs of [-1, 1) with weights that keep their scale."""
    neo.tune_db_clear()
    rng = np.random.default_rng(5)
    w = [rng.normal(0, np.sqrt(3.0 / (c * 9)), (64, c, 3, 3)).astype(np.float32) for c in (32, 64)]
    g = wl.Graph(name="two", input_shape=(2, 32, 24, 24))
    zero = np.zeros(64, np.float32)
    g.nodes = [wl.Node(op="input")] + [wl.Node(op="conv", inputs=(i,), K=64, R=3, S=3, pad=(1, 1), w=w[i], bias=zero)
                                       for i in (0, 1)] + [wl.Node(op="output", inputs=(2,))]
    p = neo.Plan(g, flags=neo.PLAN_TUNE)
    steps = p.describe()["steps"]
    last = max(i for i, s in enumerate(steps) if s["kind"] == "conv")
    x, out = dev(np.zeros(g.input_shape, np.float32)), dev(np.zeros((2, 64, 24, 24), np.float32))
    p.run_step(last, x, out)
    for i in range(last + 1, len(steps)):
        p.run_step(i, x, out)
    y = host(out)
    p.destroy()
    neo.tune_db_clear()
    assert 0.3 < y.std() < 3 and np.abs(y).max() < 10


def test_refused_where_it_does_not_apply(neo, tmp_path):
    """A window whose patch exceeds the workgroup's, and a reduction of few
    products (whose error would be larger than the float32 kernel's), keep the
    tile kernel whatever the results file says."""
    for C, R, H in ((8, 25, 64), (1, 3, 64), (2, 4, 64), (3, 1, 64), (16, 1, 64), (23, 1, 64)):
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
