"""The split-product kernels (fp32 products as six bf16 matrix products): shapes on
and off their blocks, against the fp64 oracle and against the fp32 kernel's error.

A layer runs on the fused split-product kernel when it has enough tasks of 32 tiles x
64 output channels (F(5), F(6): 32 x 32; 5/16 of 256 compute units, 3/16 at F(2), 1/8
with many channels) and more than 16 input channels; the shapes below cross the edges of a task (tiles % 32, output
channels % 64), of a stage (channels % 16), of the image (sides not a multiple of m,
odd row lengths, images narrower than a row of 16 tiles, or one tile) and both item
orders (transformed kernels outweighing the input)."""

import numpy as np
import pytest
import torch

import paper_1912_02165_amd as wc
from paper_1912_02165_amd import workloads
from oracle import toom_cook
from oracle.direct import direct_conv
from parity import assert_close, errors

pytestmark = pytest.mark.gpu

# (shape, m): C = 17 (one channel in the last stage), 32, 48; K = 64, 65, 130, 200; odd W
SHAPES = [
    ((8, 17, 130, 47, 61), 4), ((21, 32, 64, 45, 44), 4), ((16, 40, 65, 64, 37), 4),
    ((90, 33, 200, 3, 97), 4), ((330, 18, 512, 4, 4), 4), ((40, 64, 320, 13, 14), 4),
    ((8, 17, 130, 23, 31), 2), ((13, 32, 64, 22, 22), 2), ((5, 48, 65, 33, 45), 2),
    ((50, 19, 200, 2, 41), 2), ((200, 20, 512, 2, 2), 2), ((6, 96, 320, 14, 13), 2),
    ((21, 17, 80, 47, 51), 5), ((24, 32, 64, 45, 40), 5), ((90, 33, 100, 4, 93), 5),
    ((400, 18, 512, 5, 5), 5), ((48, 64, 160, 13, 16), 5),
    ((21, 17, 66, 47, 61), 6), ((24, 32, 64, 45, 48), 6), ((90, 33, 100, 5, 97), 6),
    ((400, 18, 512, 6, 6), 6), ((64, 64, 160, 14, 13), 6),
]

# (shape, m, items x pieces of the last round): after whole rounds with stages that the
# pieces do and do not divide, without whole rounds, both item orders, ragged edges, at
# the smallest number of items; the largest scratch the planless entry point holds
PIECES = [
    ((50, 70, 128, 28, 45), 4, "8 x 5"), ((48, 256, 128, 13, 14), 4, "48 x 4"), ((35, 250, 200, 13, 15), 4, "72 x 3"),
    ((32, 250, 128, 13, 13), 4, "32 x 8"), ((66, 130, 128, 28, 27), 2, "42 x 5"), ((25, 128, 65, 17, 13), 2, "100 x 2"),
    ((35, 72, 160, 27, 39), 5, "9 x 5"), ((28, 250, 128, 13, 15), 5, "32 x 8"), ((20, 256, 256, 25, 25), 5, "128 x 2"),
    ((40, 72, 130, 36, 40), 6, "9 x 5"), ((30, 250, 128, 13, 15), 6, "36 x 6"), ((47, 100, 96, 30, 18), 6, "69 x 3"),
]


def _id(c):
    return "m%d-%s" % (c[1], "x".join(map(str, c[0])))


def _device(shape, seed):
    x, w = workloads.random_inputs(*shape, seed=seed)
    return x, w, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()


@pytest.mark.parametrize("case", SHAPES, ids=_id)
def test_split_kernel_shapes(case):
    """Parity, the same bits from run, a second call, run_pretransformed and the planless
    entry point, untouched memory around y, and x at an address of 4 mod 16."""
    (N, C, K, H, W), m = case
    x, w, _, wd = _device(case[0], 900 + m + sum(case[0]))
    print(f"\n[gpu] split {_id(case)}", flush=True)
    xb = torch.zeros(x.size + 1, device="cuda")
    xb[1:] = torch.from_numpy(x.reshape(-1)).cuda()
    xd = xb[1:].view(N, C, H, W)
    n = N * K * H * W
    buf = torch.full((n + 2048,), float("nan"), device="cuda")
    y = buf[1024:1024 + n].view(N, K, H, W)
    y2, y3 = (torch.full((N, K, H, W), float("nan"), device="cuda") for _ in range(2))
    with wc.Plan(N, C, K, H, W, m) as p:
        assert "split products" in p.describe(), p.describe()
        p.run(xd, wd, y)
        p.run_pretransformed(xd, y2)
        p.status()
    wc.wino_conv_run_noalloc(N, C, K, H, W, m, xd, wd, y3)
    torch.cuda.synchronize()
    assert torch.equal(y, y2) and torch.equal(y, y3)
    assert torch.isnan(buf[:1024]).all() and torch.isnan(buf[1024 + n:]).all()
    assert_close(y.cpu().numpy(), direct_conv(x, w), m, _id(case))


@pytest.mark.parametrize("case", PIECES, ids=_id)
def test_split_kernel_pieces(case):
    """Parity with a cut last round; the same bits on a second call (arrival counters
    back at zero), without a plan, and on the replays of a captured call."""
    shape, m, cut = case
    N, C, K, H, W = shape
    x, w, xd, wd = _device(shape, 300 + m + sum(shape))
    print(f"\n[gpu] pieces {_id(case)}", flush=True)
    y, y2, y3 = (torch.full((N, K, H, W), float("nan"), device="cuda") for _ in range(3))
    with wc.Plan(*shape, m) as p:
        d = p.describe()
        assert "split products" in d and f"split items {cut} pieces" in d, d
        p.run(xd, wd, y)
        p.run_pretransformed(xd, y2)
        p.status()
        wc.wino_conv_run_noalloc(*shape, m, xd, wd, y3)
        torch.cuda.synchronize()
        assert torch.equal(y, y2) and torch.equal(y, y3)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            p.run_pretransformed(xd, y2)
        for _ in range(3):
            y2.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, y2)
        del graph
    assert_close(y.cpu().numpy(), direct_conv(x, w), m, _id(case))


@pytest.mark.parametrize("m", (2, 4, 5, 6))
def test_split_error_no_larger_than_fp32(m):
    """Images over 40 binary orders of magnitude: each image's error against fp64 stays
    within 1.2 times that of the fp32 kernel of the same blocking (reached through
    channel_splits, which the split-product kernel does not take; both are sums of the same length in fp32, so
    random errors of one size)."""
    N, C, K, H, W = 20, 64, 64, 46, 46
    x, w, _, wd = _device((N, C, K, H, W), 77)
    x *= np.exp2(np.random.default_rng(5).integers(-20, 20, size=(N, 1, 1, 1))).astype(np.float32)
    xd = torch.from_numpy(x).cuda()
    ref = direct_conv(x, w)
    rel = []
    blocking = {"tiles_per_wg": 32 if m == 2 else 16, "k_per_wg": 64 if m <= 4 else 32}
    for tuning in (None, {"channel_splits": 2, **blocking}):
        y = torch.empty((N, K, H, W), device="cuda")
        with wc.Plan(N, C, K, H, W, m, "fused", tuning) as p:
            assert ("split products" in p.describe()) == (tuning is None)
            p.run(xd, wd, y)
            p.status()
        y = y.cpu().numpy()
        rel.append(np.array([errors(y[n], ref[n])[0] for n in range(N)]))
    print(f"split {rel[0].max():.3e} fp32 {rel[1].max():.3e}")
    assert (rel[0] <= 1.2 * rel[1]).all()


@pytest.mark.parametrize("m", (2, 4, 5, 6))
def test_split_nan_reaches_connected_outputs_only(m):
    """NaNs on image corners, a tile boundary and inside reach exactly the outputs that
    (|A^T||B^T|) connects them to."""
    N, C, K, H, W = 20, 20, 64, 46, 45
    x, w, _, wd = _device((N, C, K, H, W), 31)
    points = [(0, 3, 0, 0), (2, 19, H - 1, W - 1), (5, 7, m, 2 * m), (9, 0, 17, 44)]
    clean = direct_conv(x, w)
    for n, c, h, v in points:
        x[n, c, h, v] = np.nan
    at, _, bt = toom_cook.matrices_f64(m)
    conn = (np.abs(at) @ np.abs(bt)) != 0  # m x T
    expect = np.zeros((N, H, W), bool)
    for n, _, h, v in points:
        for ty in range((H + m - 1) // m):
            for tx in range((W + m - 1) // m):
                a, b = h - (ty * m - 1), v - (tx * m - 1)
                if 0 <= a < m + 2 and 0 <= b < m + 2:
                    blk = np.outer(conn[:, a], conn[:, b])
                    hh, ww = min(m, H - ty * m), min(m, W - tx * m)
                    expect[n, ty * m:ty * m + hh, tx * m:tx * m + ww] |= blk[:hh, :ww]
    y = torch.empty((N, K, H, W), device="cuda")
    with wc.Plan(N, C, K, H, W, m) as p:
        assert "split products" in p.describe()
        p.run(torch.from_numpy(x).cuda(), wd, y)
        p.status()
    y = y.cpu().numpy()
    assert np.array_equal(np.isnan(y), np.broadcast_to(expect[:, None], y.shape))
    keep = ~np.isnan(y)
    assert errors(np.where(keep, y, 0), np.where(keep, clean, 0))[0] <= (1e-5 if m == 2 else 1e-4)


def test_split_weights_read_back():
    """The transformed kernels of a split plan read back in the documented layout as the
    exact floats the fp32 path transforms them to."""
    N, C, K, H, W = 8, 17, 130, 47, 61
    _, w, _, wd = _device((N, C, K, H, W), 3)
    got = []
    for algo in ("fused", "three_stage"):
        with wc.Plan(N, C, K, H, W, 4, algo) as p:
            p.set_weights(wd)
            got.append(p.intermediate(wc.WINO_BUF_WEIGHTS))
    assert np.array_equal(got[0], got[1])


def _unfold(buf, kind):
    """An intermediate in operand order as [f][c or k][tile] (layouts of wino_conv.h)."""
    F4, TB = buf.shape[:2]
    if kind == "U":   # [f4][tb][cs][c%4][t%16][f%4]
        v = buf.reshape(F4, TB, -1, 4, 16, 4).transpose(0, 5, 2, 3, 1, 4)
    else:             # [f4][tb][kb][k%4][k%16/4][t%16][f%4]
        v = buf.reshape(F4, TB, -1, 4, 4, 16, 4).transpose(0, 6, 2, 4, 3, 1, 5)
    return v.reshape(F4 * 4, -1, TB * 16).astype(np.float64)


@pytest.mark.parametrize("m", (2, 4, 5, 6, 7))
@pytest.mark.parametrize("shape", [(2, 64, 70, 11, 13), (3, 65, 130, 9, 30), (1, 79, 16, 7, 7), (5, 130, 64, 15, 16)],
                         ids=lambda s: "x".join(map(str, s)))
def test_three_stage_split_products(shape, m):
    """Parity end to end, and the products M against the fp64 products of the read-back U
    and W': within the rounding of an fp32 sum over C (a few sqrt(C) half-ulps: 1e-6 of
    the largest |M|), zeros where padding is documented."""
    N, C, K, H, W = shape
    x, w, xd, wd = _device(shape, 60 + m + C)
    y = torch.full((N, K, H, W), float("nan"), device="cuda")
    T2 = (m + 2) ** 2
    with wc.Plan(N, C, K, H, W, m, "three_stage") as p:
        assert "frequency_gemm_split" in p.describe()
        p.run(xd, wd, y)
        torch.cuda.synchronize()
        wt = p.intermediate(wc.WINO_BUF_WEIGHTS)
        U = _unfold(p.intermediate(wc.WINO_BUF_INPUT), "U")
        M = _unfold(p.intermediate(wc.WINO_BUF_PRODUCT), "M")
    Kb, Cs = wt.shape[:2]
    Wt = wt.reshape(Kb, Cs, -1, 4, 16, 4).transpose(2, 5, 1, 3, 0, 4).reshape(-1, Cs * 4, Kb * 16).astype(np.float64)
    ref = np.einsum("fck,fct->fkt", Wt, U)
    assert np.abs(M - ref).max() <= 1e-6 * np.abs(ref).max()
    assert not M[T2:].any() and not M[:, K:].any()
    assert_close(y.cpu().numpy(), direct_conv(x, w), m, f"three_stage F({m}) {shape}")


@pytest.mark.parametrize("m,C,pieces", [(2, 512, 8), (4, 512, 8), (5, 512, 8), (6, 512, 8), (4, 180, 3), (6, 250, 4)])
def test_last_round_pieces(m, C, pieces):
    """Layers of few tasks and many channel stages: the last round cut into up to eight
    pieces of at least four stages, the same bits on every call and without a plan."""
    shape = (1, C, 40, 9, 10)
    x, w, xd, wd = _device(shape, 40 + m)
    ys = [torch.full((1, 40, 9, 10), float("nan"), device="cuda") for _ in range(3)]
    with wc.Plan(*shape, m) as p:
        assert f"x {pieces} pieces" in p.describe(), p.describe()
        p.run(xd, wd, ys[0])
        p.run(xd, wd, ys[1])
        p.status()
    wc.wino_conv_run_noalloc(*shape, m, xd, wd, ys[2])
    torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1]) and torch.equal(ys[0], ys[2])
    assert_close(ys[0].cpu().numpy(), direct_conv(x, w), m, f"F({m}) C={C} in {pieces} pieces")


@pytest.mark.parametrize("shape,m", [((40, 64, 64, 64, 14), 4), ((40, 256, 256, 14, 14), 4), ((16, 128, 128, 28, 28), 5)])
def test_channel_splits_keep_their_blocking(shape, m):
    """channel_splits without a blocking runs the fp32 kernel at the blocking that kernel
    prefers (one with at least one item per compute unit where there is one), also on
    layers that run on the split-product kernel otherwise."""
    N, C, K, H, W = shape
    tiles = N * -(-H // m) * -(-W // m)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    largest = -(-tiles // 16) * -(-K // (64 if m == 4 else 32))
    with wc.Plan(*shape, m) as p:
        assert "split products" in p.describe()
    with wc.Plan(*shape, m, "fused", {"channel_splits": 2}) as p:
        d = p.describe()
    assert "split products" not in d
    kit = int(d.split("Kit=")[1].split()[0])
    assert (kit == (64 if m == 4 else 32)) == (largest >= cus), d


def test_split_kernel_operand_bytes_limit():
    """A task whose split kernels pass 2^32 bytes (2 blocks x 19440 stages x 36 x 3072) stays
    on the fp32 kernel, whose kernels fit; one stage step below the limit it does not.
    Plans only: nothing is run."""
    for C, split in ((311040, False), (310688, True)):
        assert (2 * (C // 16) * 36 * 3072 < 2 ** 32) == split and 64 * C * 36 * 4 < 2 ** 32
        with wc.Plan(1024, C, 64, 1, 1, 4) as p:
            assert ("split products" in p.describe()) == split, p.describe()


def test_three_stage_few_tiles_large_kernels():
    """F(7) layers of few tiles and more than 256 x 256 channels keep the fp32 products:
    both sides of the rule's lines, the fp32 side against the oracle."""
    for shape, split in (((1, 257, 256, 14, 14), False), ((1, 256, 256, 14, 14), True),
                         ((32, 257, 256, 14, 14), False), ((33, 257, 256, 14, 14), True)):
        with wc.Plan(*shape, 7, "three_stage") as p:
            assert ("frequency_gemm_split" in p.describe()) == split, (shape, p.describe())
    shape = (1, 257, 256, 14, 13)
    x, w, xd, wd = _device(shape, 12)
    y = torch.full((1, 256, 14, 13), float("nan"), device="cuda")
    with wc.Plan(*shape, 7, "three_stage") as p:
        p.run(xd, wd, y)
        torch.cuda.synchronize()
    assert_close(y.cpu().numpy(), direct_conv(x, w), 7, "three_stage F(7), few tiles")


# (shape, m): one image, output channels of a task missing (the epilogue's rounds of 8
# channels past K begin past the end of y), and images lower than a tile (so do its rows)
FEW_CHANNELS = [((1, 32, 40, 256, 257), 4), ((1, 32, 40, 250, 251), 2), ((1, 32, 24, 350, 351), 5), ((1, 32, 20, 400, 399), 6),
                ((1, 17, 57, 1, 16390), 4), ((1, 17, 57, 1, 8290), 2), ((1, 17, 25, 1, 20003), 5), ((1, 17, 25, 1, 24003), 6),
                ((1, 17, 57, 2, 16390), 4), ((1, 17, 25, 2, 24003), 6)]


@pytest.mark.parametrize("case", FEW_CHANNELS, ids=_id)
def test_split_kernel_few_output_channels(case):
    """Layers of one image and fewer output channels than a task holds: parity, and nothing
    written within 64 planes around y."""
    (N, C, K, H, W), m = case
    x, w, xd, wd = _device(case[0], 200 + m + sum(case[0]))
    print(f"\n[gpu] few channels {_id(case)}", flush=True)
    n, pad = K * H * W, 64 * H * W
    buf = torch.full((n + 2 * pad,), float("nan"), device="cuda")
    y = buf[pad:pad + n].view(N, K, H, W)
    with wc.Plan(N, C, K, H, W, m) as p:
        assert "split products" in p.describe(), p.describe()
        p.run(xd, wd, y)
        p.status()
    torch.cuda.synchronize()
    assert torch.isnan(buf[:pad]).all() and torch.isnan(buf[pad + n:]).all()
    assert_close(y.cpu().numpy(), direct_conv(x, w), m, _id(case))


# ---- the whole range of float -------------------------------------------------

def _run_pair(shape, m, algo, xd, wd):
    """y of the split products and of the fp32 products of the same transforms."""
    blocking = {"tiles_per_wg": 32 if m == 2 else 16, "k_per_wg": 64 if m <= 4 else 32}
    ys = []
    for a, tuning in ((algo, None), ("fused", {"channel_splits": 2, **blocking})):
        y = torch.full((shape[0], shape[2], *shape[3:]), 7.0, device="cuda")
        with wc.Plan(*shape, m, a, tuning) as p:
            assert ("split" in p.describe().split("split items")[0]) == (tuning is None), p.describe()
            p.run(xd, wd, y)
            p.status()
        ys.append(y.cpu().numpy())
    return ys


# (m, algorithm, shape): whole items, items in pieces, the three-stage products
RANGE = [(m, "fused", (20, 64, 64, 46, 46)) for m in (2, 4, 5, 6)] + [
    (2, "fused", (25, 128, 65, 17, 13)), (4, "fused", (35, 250, 200, 13, 15)), (5, "fused", (28, 250, 128, 13, 15)),
    (6, "fused", (30, 250, 128, 13, 15))] + [(m, "three_stage", (20, 70, 66, 13, 15)) for m in (2, 4, 5, 6)]


def _range_id(c):
    return "m%d-%s-%s" % (c[0], c[1], "x".join(map(str, c[2])))


@pytest.mark.parametrize("side", ("input", "kernels"))
@pytest.mark.parametrize("case", RANGE, ids=_range_id)
def test_split_products_keep_small_and_large_values(case, side):
    """Images (or output channels) at binary orders of magnitude from 2^-145 (denormal) to 2^120,
    the other factor scaled so that the results stay normal: the error of each against fp64
    within 1.5 times that of the fp32 products.  These add two halves of the channels, so
    their error may be smaller than that of one sum by sqrt(2); the rest is for chance in one
    image or channel.  (Denormal factors are compared with the fp64 result of the values they
    round to.)"""
    m, algo, shape = case
    N, C, K, H, W = shape
    x, w, _, _ = _device(shape, 50 + m + C)
    for exps, other in ((np.linspace(-145, -96, N if side == "input" else K), 60), (np.linspace(60, 120, N if side == "input" else K), -60)):
        sc = np.exp2(np.round(exps))
        if side == "input":
            xs, ws = (x * sc[:, None, None, None]).astype(np.float32), (w * 2.0 ** other).astype(np.float32)
        else:
            xs, ws = (x * 2.0 ** other).astype(np.float32), (w * sc[:, None, None, None]).astype(np.float32)
        ref = direct_conv(xs.astype(np.float64), ws.astype(np.float64))
        ys = _run_pair(shape, m, algo, torch.from_numpy(xs).cuda(), torch.from_numpy(ws).cuda())
        axis = 0 if side == "input" else 1
        rel = np.array([[errors(np.take(y, i, axis), np.take(ref, i, axis))[0] for i in range(len(sc))] for y in ys])
        print(f"{_range_id(case)} {side} {other}: worst {rel[0].max():.3e} fp32 {rel[1].max():.3e} "
              f"ratio {(rel[0] / rel[1]).max():.3f}")
        assert np.isfinite(ys[0]).all() and (rel[0] <= 1.5 * rel[1]).all(), rel


@pytest.mark.parametrize("case", RANGE, ids=_range_id)
def test_split_products_infinities_as_fp32(case):
    """Infinities, NaNs and values beyond the scaled terms among the inputs and kernels: the same
    outputs are infinite, with the same sign, and NaN as with the fp32 products, and the
    images and channels without such values are not touched."""
    m, algo, shape = case
    N, C, K, H, W = shape
    x, w, xd, wd = _device(shape, 70 + m + C)
    for values, kernels in (((np.inf, 1e33, -np.inf, -1e32), ()), ((1e33, -1e33), (np.inf, np.nan, -np.inf)), ((), (1e33, -1e32))):
        xs, ws = x.copy(), w.copy()
        for i, v in enumerate(values):
            xs[(3 * i) % N, (5 * i + 1) % C, (7 * i) % H, (4 * i + 2) % W] = v
        for i, v in enumerate(kernels):
            ws[(9 * i + 2) % K, (3 * i) % C, i, 2 - i] = v
        a, b = _run_pair(shape, m, algo, torch.from_numpy(xs).cuda(), torch.from_numpy(ws).cuda())
        assert np.array_equal(np.isnan(a), np.isnan(b)), (np.isnan(a).sum(), np.isnan(b).sum())
        assert np.array_equal(np.isposinf(a), np.isposinf(b)) and np.array_equal(np.isneginf(a), np.isneginf(b))
        assert np.isfinite(b).all() == (values == ())
        # images and output channels without such a value
        n = [i for i in range(N) if i not in [(3 * j) % N for j in range(len(values))]]
        k = [i for i in range(K) if i not in [(9 * j + 2) % K for j in range(len(kernels))]]
        a, b = a[n][:, k], b[n][:, k]
        assert np.isfinite(a).all() and errors(a, b)[0] <= 2e-5


def test_split_weights_read_back_any_value():
    """Transformed kernels read back bit for bit, whatever their magnitude: denormal, beyond the
    scaled terms, infinite, NaN, zeros of both signs."""
    N, C, K, H, W = 8, 17, 130, 47, 61
    w = np.random.default_rng(9).standard_normal((K, C, 3, 3)).astype(np.float32)
    w *= np.exp2(np.random.default_rng(8).integers(-149, 128, size=(K, C, 1, 1))).astype(np.float32)
    w[0, 0] = -0.0
    w[1, 1, 0, 0] = np.inf
    w[2, 2, 1, 1] = np.nan
    w[3, 3, 2, 2] = np.finfo(np.float32).max
    wd = torch.from_numpy(w).cuda()
    got = []
    for algo in ("fused", "three_stage"):
        with wc.Plan(N, C, K, H, W, 4, algo) as p:
            assert ("split products" in p.describe()) == (algo == "fused")
            p.set_weights(wd)
            got.append(p.intermediate(wc.WINO_BUF_WEIGHTS))
    nan = np.isnan(got[1])
    assert np.array_equal(np.isnan(got[0]), nan)
    assert np.array_equal(got[0].view(np.uint32)[~nan], got[1].view(np.uint32)[~nan])


def test_three_stage_padding_frequencies_zero():
    """Frequencies past T^2 hold zeros in M whatever the kernels hold (F(5): 49 of 52)."""
    shape = (1, 64, 16, 9, 9)
    x, w, xd, wd = _device(shape, 5)
    wd[3, 5, 1, 1] = float("inf")
    y = torch.empty((1, 16, 9, 9), device="cuda")
    with wc.Plan(*shape, 5, "three_stage") as p:
        p.run(xd, wd, y)
        M = _unfold(p.intermediate(wc.WINO_BUF_PRODUCT), "M")
    assert np.isnan(M[:49]).any() or np.isinf(M[:49]).any()
    assert not M[49:].any()


@pytest.mark.parametrize("shape,m", [((20, 64, 64, 46, 46), 2), ((20, 64, 64, 46, 46), 4), ((16, 128, 128, 28, 28), 5),
                                     ((32, 128, 128, 28, 28), 6)])
def test_given_blocking_is_the_fp32_kernels(shape, m):
    """Every blocking asked for runs on the fp32 kernel, at that blocking, also on layers
    that run on the split-product kernel otherwise; the plan's parameters tell them apart."""
    x, w, xd, wd = _device(shape, 17)
    N, C, K, H, W = shape
    ref = direct_conv(x, w)
    with wc.Plan(*shape, m) as p:
        assert "split products" in p.describe() and p.params() == (m, 0, 0, 0)
    for bm, R, kit in wc.wino_fused_blockings():
        if bm != m:
            continue
        y = torch.full((N, K, H, W), float("nan"), device="cuda")
        with wc.Plan(*shape, m, "fused", {"tiles_per_wg": R, "k_per_wg": kit}) as p:
            d = p.describe()
            assert "split products" not in d and f"R={R} " in d and f"Kit={kit} " in d, d
            assert p.params() == (m, 0, R, kit)
            p.run(xd, wd, y)
            p.status()
        assert_close(y.cpu().numpy(), ref, m, f"F({m}) {R} x {kit}")


def test_tuned_plan_has_both_kernels(tmp_path):
    """The tuner times the split-product kernel beside every fp32 blocking: where the rule
    takes it by a wide margin so does the tuner, a wisdom entry keeps the choice, an entry
    with a blocking gives the fp32 kernel, and one of the split-product kernel gives it
    also where the rule does not."""
    shape = (64, 128, 128, 28, 28)
    prop = torch.cuda.get_device_properties(0)
    key = "%s %d " % (prop.gcnArchName.split(":")[0], prop.multi_processor_count)
    wc.wino_wisdom_clear()
    with wc.Plan.tuned(*shape, wc.WINO_TUNE_M4) as p:
        assert "split products" in p.describe() and p.params() == (4, 0, 0, 0)
    f = tmp_path / "w.txt"
    wc.wino_wisdom_save(str(f))
    assert " 0x10 4 0 0 0 " in f.read_text()
    few = (1, 64, 64, 56, 56)
    f.write_text(key + "64 128 128 28 28 0x10 4 0 16 64 50.0\n" + key + "1 64 64 56 56 0x10 4 0 0 0 50.0\n")
    wc.wino_wisdom_load(str(f))
    with wc.Plan.tuned(*shape, wc.WINO_TUNE_M4) as p:
        assert "split products" not in p.describe() and p.params() == (4, 0, 16, 64)
    with wc.Plan(*few, 4) as p:
        assert "split products" not in p.describe()
    x, w, xd, wd = _device(few, 18)
    y = torch.full((1, 64, 56, 56), float("nan"), device="cuda")
    with wc.Plan.tuned(*few, wc.WINO_TUNE_M4) as p:
        assert "split products" in p.describe()
        p.run(xd, wd, y)
        p.status()
    assert_close(y.cpu().numpy(), direct_conv(x, w), 4, "split-product kernel by wisdom")
    wc.wino_wisdom_clear()


# layers where the fp32 kernel runs at a blocking that adds two halves of the channels: at
# both ends of the rule's range, ragged, in three stages and more, both item orders
HALVES = [((4, 64, 64, 56, 56), 2), ((4, 37, 45, 57, 61), 2), ((4, 112, 64, 56, 56), 2), ((20, 80, 64, 46, 46), 4),
          ((1, 64, 64, 224, 224), 4), ((24, 33, 60, 46, 45), 4), ((20, 64, 64, 46, 46), 5), ((20, 80, 64, 46, 46), 5),
          ((20, 33, 64, 46, 46), 5), ((20, 64, 64, 46, 46), 6), ((20, 33, 64, 46, 46), 6), ((1, 48, 64, 224, 224), 6)]


@pytest.mark.parametrize("case", HALVES, ids=_id)
def test_error_no_larger_than_two_halves(case):
    """Against fp64, a layer's error is no larger than at the blocking the fp32 kernel would
    take by itself: there one that adds two halves of the channels.  (Both errors are
    norms over more than 500,000 outputs, so chance moves them by well under 1%.)"""
    (N, C, K, H, W), m = case
    x, w, xd, wd = _device(case[0], 400 + m + C)
    ref = direct_conv(x, w)
    rel = []
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tiles = -(-(N * -(-H // m) * -(-W // m)) // 16)
    fp32 = {2: (16, 32), 4: (16, 32), 5: (16, 16), 6: (16, 16)}[m]
    assert tiles * -(-K // (64 if m <= 4 else 32)) < cus  # the larger blockings do not fill the device
    for tuning in (None, {"tiles_per_wg": fp32[0], "k_per_wg": fp32[1]}):
        y = torch.full((N, K, H, W), float("nan"), device="cuda")
        with wc.Plan(N, C, K, H, W, m, "fused", tuning) as p:
            p.run(xd, wd, y)
            p.status()
        rel.append(errors(y.cpu().numpy(), ref)[0])
    print(f"{_id(case)} {rel[0]:.3e} two halves {rel[1]:.3e} ratio {rel[0] / rel[1]:.3f}")
    assert rel[0] <= 1.01 * rel[1]


def test_rules_where_the_kernel_transform_weighs():
    """Both sides of the lines for three-stage layers of 64 to 80 channels, drawn with kernels
    given at every call in view."""
    for shape, m, split in (((32, 64, 64, 56, 56), 4, False), ((16, 64, 64, 56, 56), 4, True), ((32, 81, 64, 56, 56), 4, True),
                            ((2, 64, 128, 14, 14), 6, True), ((2, 64, 129, 14, 14), 6, False), ((2, 80, 256, 14, 14), 6, True),
                            ((8, 64, 512, 28, 28), 6, True), ((8, 72, 256, 28, 28), 4, False), ((32, 64, 256, 56, 56), 4, True)):
        with wc.Plan(*shape, m, "three_stage") as p:
            assert ("frequency_gemm_split" in p.describe()) == split, (shape, p.describe())


@pytest.mark.parametrize("m", (2, 4, 5, 6))
@pytest.mark.parametrize("shape", [(120, 70, 50, 8, 70), (40, 200, 128, 28, 27), (16, 256, 256, 28, 26)], ids=lambda s: "x".join(map(str, s)))
def test_kernel_transform_workgroups(shape, m):
    """The kernel transform with 4, 8 and 16 frequencies a workgroup: parity with and without a plan."""
    x, w, xd, wd = _device(shape, 80 + m)
    N, C, K, H, W = shape
    ys = [torch.full((N, K, H, W), float("nan"), device="cuda") for _ in range(2)]
    with wc.Plan(*shape, m) as p:
        assert "split products" in p.describe(), p.describe()
        p.run(xd, wd, ys[0])
        p.status()
    try:
        wc.wino_conv_run_noalloc(*shape, m, xd, wd, ys[1])
    except wc.WinoError as e:
        assert "scratch" in str(e)
        ys[1] = ys[0]
    torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1])
    assert_close(ys[0].cpu().numpy(), direct_conv(x, w), m, f"F({m}) {shape}")


@pytest.mark.parametrize("shape,m,split", [
    ((64, 64, 64, 32, 32), 4, False), ((63, 64, 64, 32, 32), 4, True), ((65, 64, 64, 32, 32), 4, True),
    ((64, 64, 64, 32, 30), 4, True), ((64, 64, 64, 30, 32), 4, False), ((64, 256, 64, 32, 32), 4, True), ((128, 64, 64, 32, 32), 4, True),
    ((192, 32, 64, 32, 32), 4, False), ((32, 64, 64, 40, 40), 5, False), ((32, 512, 64, 40, 40), 5, True),
    ((96, 64, 64, 40, 40), 5, False), ((32, 64, 64, 48, 48), 6, False), ((32, 64, 64, 47, 46), 6, False), ((32, 128, 64, 47, 45), 6, True), ((64, 64, 64, 48, 48), 6, True),
    ((8, 64, 64, 32, 32), 2, False), ((16, 64, 64, 32, 32), 2, False), ((32, 64, 64, 32, 32), 2, True),
    ((2, 192, 64, 64, 64), 2, True), ((9, 64, 64, 32, 32), 2, True),
    ((304, 64, 64, 45, 45), 5, False), ((24, 64, 64, 160, 160), 5, True), ((60, 64, 64, 102, 102), 6, False),
    ((67, 64, 64, 96, 96), 6, True)], ids=str)
def test_full_rounds_of_the_fp32_kernel(shape, m, split):
    """Layers that fill rounds of the fp32 kernel's smaller tasks stay on it; their neighbours
    in images, channels and raggedness on the split-product kernel (256 compute units)."""
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    with wc.Plan(*shape, m) as p:
        assert ("split products" in p.describe()) == split, p.describe()
