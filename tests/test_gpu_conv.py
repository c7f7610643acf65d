"""The convolution kernels on the GPU, one convolution at a time
(lipz_test_conv), at sizes that leave tiles, slices and splits partly filled:
against torch's fp64 convolutions on the CPU, and the wide fp32 tiles bit for
bit against the 64 x 64 ones; weights split beforehand bit for bit
against weights split on the way; infinities and NaNs of the bf16 kernel
against fp32 products."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU, skipped there
    pytest.skip("no GPU", allow_module_level=True)

import torch.nn.functional as F  # noqa: E402

import paper_1811_12843_amd as L  # noqa: E402

ANY, WIDE, SPLIT, PRE, SUM = 0, 1, 2, 3, 4
SLOPE = 0.2
KINDS = ["conv", "convT", "conv_dgrad", "convT_dgrad", "conv_wgrad", "convT_wgrad"]
# (images, log2 side, c_in, c_out): channels a multiple of 32 (a slice within one tap) and not, one and several
# 128- and 64-wide column tiles, whole and partial rows, last splits of a few positions
SHAPES = [(3, 3, 32, 64), (1, 2, 36, 132), (5, 2, 20, 68), (2, 4, 64, 128), (9, 3, 44, 192), (7, 1, 128, 20)]
TILES = [(128, 128), (128, 64), (64, 64)]


def _nchw(t):
    return t.permute(0, 3, 1, 2)


def _reference(kind, x, w, aux, bias):
    """fp64 results of a kind in lipz_test_conv's layout, and the sums of |a b| that bound their rounding."""
    out = []
    for f in (lambda t: t, torch.abs):
        X, W = f(x), f(w)
        ci, co = W.shape[-2], W.shape[-1]
        if kind == "conv":
            y = F.conv2d(_nchw(X), W.view(4, 4, ci, co).permute(3, 2, 0, 1), f(bias), stride=2, padding=1)
        elif kind == "convT":
            y = F.conv_transpose2d(_nchw(X), W.view(4, 4, ci, co).permute(2, 3, 0, 1), stride=2, padding=1)
        elif kind == "conv_dgrad":
            y = F.conv_transpose2d(_nchw(X), W.view(4, 4, ci, co).permute(3, 2, 0, 1), stride=2, padding=1)
        else:
            y = F.conv2d(_nchw(X), W.view(4, 4, ci, co).permute(2, 3, 0, 1), stride=2, padding=1)
        out.append(y.permute(0, 2, 3, 1).contiguous())
    if kind in ("conv_dgrad", "convT_dgrad"):
        out = [y * torch.where(aux > 0, 1.0, SLOPE) for y in out]
    elif kind == "conv":
        out[0] = torch.where(out[0] > 0, out[0], SLOPE * out[0])
    return out


def _wgrad_reference(kind, x, dy):
    out = []
    for f in (lambda t: t, torch.abs):
        X, D = f(x), f(dy)
        small, big = (D, X) if kind == "conv_wgrad" else (X, D)  # the big map is gathered by the 16 taps
        n, S = small.shape[0], small.shape[1]
        cols = F.unfold(_nchw(big), 4, stride=2, padding=1).view(n, big.shape[3], 16, S * S)  # [n][c][tap][pos]
        sm = small.reshape(n, S * S, -1)
        g = torch.stack([sum(cols[i, :, t] @ sm[i] for i in range(n)) for t in range(16)])  # [tap][big c][small c]
        if kind == "conv_wgrad":
            out.append(torch.cat([g.reshape(-1, g.shape[2]), D.sum((0, 1, 2))[None]]))
        else:
            out.append(g.transpose(1, 2).reshape(-1, g.shape[1]))
    return out


def _problem(kind, shape, seed):
    n, h, ci, co = shape
    rng = np.random.default_rng(seed)
    t = {k: torch.from_numpy(rng.standard_normal(s).astype(np.float32)) for k, s in dict(
        big=(n, 2 << h, 2 << h, co), inp=(n, 1 << h, 1 << h, ci), half=(n, max(1, 1 << h >> 1), max(1, 1 << h >> 1), co),
        w=(16, ci, co), bias=(co,), aux=(n, 1 << h, 1 << h, ci)).items()}
    x = {"conv": "inp", "convT": "inp", "conv_dgrad": "half", "convT_dgrad": "big", "conv_wgrad": "inp", "convT_wgrad": "inp"}
    w = {"conv_wgrad": "half", "convT_wgrad": "big"}
    return t[x[kind]], t[w.get(kind, "w")], t["bias"], t["aux"]


def _run(kind, shape, kernel, tile, x, w, bias, aux, pieces_tail=0):
    n, h, ci, co = shape
    K = KINDS.index(kind)
    splits = -(-(n << (2 * (h - 1 if kind == "conv_wgrad" else h))) // 1024)
    size = {"conv": (n, 1 << h >> 1, 1 << h >> 1, co), "convT": (n, 2 << h, 2 << h, co), "conv_dgrad": (n, 1 << h, 1 << h, ci),
            "convT_dgrad": (n, 1 << h, 1 << h, ci), "conv_wgrad": (splits, 16 * ci + 1, co),
            "convT_wgrad": (splits, 16 * ci, co)}[kind]
    if kernel == PRE:
        aux = torch.full((24 * ci * (-(-co // 32) + pieces_tail) * 32,), float("nan"))  # the weights' pieces
    dx, dw, db, da = (t.cuda().contiguous() for t in (x, w, bias, aux))
    out = torch.full(size, float("nan"), device="cuda")
    desc = torch.zeros(2048, dtype=torch.uint8, device="cuda")
    L.lipz_test_conv(torch.cuda.current_stream().cuda_stream, desc.data_ptr(), K, n, h, ci, co, dx.data_ptr(),
                     dw.data_ptr(), out.data_ptr(), db.data_ptr() if kind == "conv" else None, da.data_ptr(),
                     L.ACTS["lrelu"], SLOPE, kernel, *tile)
    torch.cuda.synchronize()
    return out.cpu()


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("shape", SHAPES)
def test_kernels_match_fp64(kind, shape):
    x, w, bias, aux = _problem(kind, shape, seed=sum(shape) * 7 + KINDS.index(kind))
    if kind.endswith("wgrad"):
        ref, mag = _wgrad_reference(kind, x.double(), w.double())
    else:
        ref, mag = _reference(kind, x.double(), w.double(), aux.double(), bias.double())
    n, h, ci, co = shape
    depth = {"conv": 16 * ci, "convT": 4 * ci, "conv_dgrad": 4 * co, "convT_dgrad": 16 * co}.get(kind, n << (2 * h))
    # a chain of fp32 multiply-adds over K products is off by at most K 2^-24 of the sum of |a b|; then bias,
    # activation and the sum of splits
    bound = (depth + 8) * 2.0 ** -24 * mag + 1e-30
    if (co if kind in ("conv", "convT", "conv_wgrad", "convT_wgrad") else ci) <= 16:
        pytest.skip("no wide tile is that narrow")
    base = None
    split = [(SPLIT, t) for t in TILES] if kind in ("conv", "convT") else []
    for kernel, tile in [(ANY, (0, 0))] + [(WIDE, t) for t in TILES] + split:
        print(f"[case] {kind} {shape} kernel {kernel} tile {tile}", flush=True)
        got = _run(kind, shape, kernel, tile, x, w, bias, aux)
        full = got.double().sum(0) if kind.endswith("wgrad") else got.double()
        assert torch.all((full - ref).abs() <= bound), (kernel, tile, float(((full - ref).abs() / bound).max()))
        if kernel == ANY:
            base = got
        elif kernel == WIDE:
            assert torch.equal(got, base), (tile, float((got - base).abs().max()))
        elif kernel == SPLIT and ci % 32 == 0:
            pre = _run(kind, shape, PRE, tile, x, w, bias, aux)
            assert torch.equal(pre, got), (tile, float((pre - got).abs().max()))


@pytest.mark.parametrize("kind", ["conv", "convT"])
@pytest.mark.parametrize("shape", [(9, 3, 32, 64), (17, 2, 36, 132), (9, 3, 64, 132)])
def test_split_kernel_keeps_infinities_and_nans(kind, shape):
    """Operands with infinities, NaNs, zeros and a value next to fp32's largest: the same outputs are infinite (with
    the same sign) and NaN as with fp32 products, and the others agree."""
    x, w, bias, aux = _problem(kind, shape, seed=3)
    f = x.view(-1)
    f[::53] = 0.0
    f[5], f[f.numel() // 2], f[f.numel() // 3] = float("inf"), float("-inf"), float("nan")
    f[f.numel() // 4] = 3.395e38  # finite, but bf16 rounds it to infinity
    w.view(-1)[::31] = 0.0
    w.view(-1)[7] = float("inf")
    print(f"[case] non-finite {kind} {shape}", flush=True)
    # the finite outputs are sums without those operands; both sides are within the rounding of their K products
    zeroed = [torch.nan_to_num(t, 0.0, 0.0, 0.0).double() for t in (x, w, aux, bias)]
    bound = 2 * (16 * shape[2] + 8) * 2.0 ** -24 * _reference(kind, *zeroed)[1] + 1e-30
    base = _run(kind, shape, ANY, (0, 0), x, w, bias, aux)
    inf, fin = torch.isinf(base), torch.isfinite(base)
    assert fin.any() and inf.any() and torch.isnan(base).any()
    for tile in TILES:
        got = _run(kind, shape, SPLIT if shape[2] % 32 else PRE, tile, x, w, bias, aux)
        assert torch.equal(torch.isnan(got), torch.isnan(base)), tile
        assert torch.equal(torch.isinf(got), inf), tile
        assert torch.equal(got[inf], base[inf]), tile
        assert torch.all((got[fin].double() - base[fin].double()).abs() <= bound[fin]), tile


@pytest.mark.parametrize("kind", ["conv", "convT"])
@pytest.mark.parametrize("shape", [(1, 3, 32, 64), (1, 3, 36, 20), (4, 3, 64, 128), (3, 4, 32, 132), (1, 2, 8, 64)])
@pytest.mark.parametrize("plant", ["one", "huge", "weights"])
def test_split_tiles_with_a_non_finite_sum_keep_fp32_precision(kind, shape, plant):
    """A tile with an infinite or NaN sum has the fp32 kernel's sums bit for bit, its finite ones too; the others are
    as without the planted values.  (Tiles whole and cut, one slice and many, and networks that are NaN all over.)"""
    n, h, ci, co = shape
    x, w, bias, aux = _problem(kind, shape, seed=11)
    clean = _run(kind, shape, PRE if ci % 32 == 0 else SPLIT, (64, 64), x, w, bias, aux)
    if plant == "weights":
        w[:] = float("nan")
    else:
        x[0, x.shape[1] // 2, x.shape[2] // 2, ci // 3] = float("inf") if plant == "one" else 3.395e38
    base = _run(kind, shape, ANY, (0, 0), x, w, bias, aux)
    assert plant == "huge" or not torch.isfinite(base).all()
    for kernel in [SPLIT] + ([PRE] if ci % 32 == 0 else []):
        for tile in TILES:
            print(f"[case] again {kind} {shape} {plant} kernel {kernel} tile {tile}", flush=True)
            got = _run(kind, shape, kernel, tile, x, w, bias, aux)
            same = (got.view(torch.int32) == base.view(torch.int32)) | (torch.isnan(got) & torch.isnan(base))
            # outputs are rows of positions (of a parity class each, for the transposed kind) in tiles of tile[0] rows
            g = x.shape[1] >> 1 if kind == "conv" else x.shape[1]
            q = torch.arange(n * g * g).view(n, g, g)
            if kind == "convT":
                q = torch.stack([torch.stack([q + (2 * r + s) * 65536 for s in (0, 1)], -1) for r in (0, 1)], 2).reshape(
                    n, 2 * g, 2 * g)
            row = (q // 65536 * 65536 + q % 65536 // tile[0]).reshape(-1)
            col = torch.arange(co) // tile[1]
            f, s, u = got.reshape(-1, co), same.reshape(-1, co), clean.reshape(-1, co)
            redone = 0
            for r in row.unique():
                for c in col.unique():
                    at = (row == r)[:, None] & (col == c)[None]
                    if not s[at].all():
                        assert torch.equal(f[at], u[at]), (kernel, tile, int(r), int(c))
                    else:
                        redone += 1
            assert redone > 0


@pytest.mark.parametrize("kind", ["conv", "convT"])
@pytest.mark.parametrize("ex,ew", [(-112, 0), (0, -118), (-122, 40), (40, -126), (-130, 30), (-60, -60)])
def test_split_kernel_on_tiny_operands(kind, ex, ew):
    """Operands whose bf16 pieces would be subnormal, and subnormal operands: against fp64, no further off than fp32
    products are (root mean square; the split's is about a third of theirs)."""
    shape = (8, 3, 32, 64)
    x, w, bias, aux = _problem(kind, shape, seed=5)
    x, w, bias = torch.ldexp(x, torch.tensor(ex)), torch.ldexp(w, torch.tensor(ew)), torch.zeros_like(bias)
    ref = _reference(kind, x.double(), w.double(), aux.double(), bias.double())[0]

    def rms(kernel, tile):
        got = _run(kind, shape, kernel, tile, x, w, bias, aux)
        return float((got.double() - ref).pow(2).mean().sqrt() / ref.pow(2).mean().sqrt())

    base = rms(ANY, (0, 0))
    for kernel in (SPLIT, PRE):
        print(f"[case] tiny {kind} 2^{ex} 2^{ew} kernel {kernel}", flush=True)
        assert rms(kernel, (64, 64)) <= base


@pytest.mark.parametrize("kind", ["conv", "convT"])
@pytest.mark.parametrize("shape", [(3, 3, 32, 20), (3, 3, 32, 96), (1, 3, 64, 132)])
def test_split_weights_are_read_within_their_extent(kind, shape):
    """Columns of a tile past the last whole block of weights: NaNs behind the weights' pieces (a tile's whole width of
    them) never reach a sum, which would send its tile to fp32 and change its bits."""
    x, w, bias, aux = _problem(kind, shape, seed=17)
    for tile in TILES:
        print(f"[case] extent {kind} {shape} tile {tile}", flush=True)
        got = _run(kind, shape, PRE, tile, x, w, bias, aux, pieces_tail=4)
        assert torch.equal(got, _run(kind, shape, SPLIT, tile, x, w, bias, aux)), tile


# (images, log2 side): one split and several of 1024 positions, a last one of a few, splits that start inside an
# image, grids 32 wide (one grid row per slice)
@pytest.mark.parametrize("kind,shape", [("convT_wgrad", (5, 4, 32, 64)), ("conv_wgrad", (17, 4, 32, 64)),
                                        ("conv_wgrad", (3, 6, 8, 36)), ("convT_wgrad", (3, 5, 12, 20)),
                                        ("convT_wgrad", (67, 2, 36, 132)), ("conv_wgrad", (2051, 1, 8, 20))])
def test_weight_gradients_of_several_splits(kind, shape):
    x, w, bias, aux = _problem(kind, shape, seed=23)
    ref, mag = _wgrad_reference(kind, x.double(), w.double())
    n, h, ci, co = shape
    pos = n << (2 * (h - 1 if kind == "conv_wgrad" else h))
    assert pos > 1024
    print(f"[case] splits {kind} {shape} kernel 0", flush=True)
    base = _run(kind, shape, ANY, (0, 0), x, w, bias, aux)
    assert torch.all((base.double().sum(0) - ref).abs() <= (1024 + pos / 1024 + 8) * 2.0 ** -24 * mag + 1e-30)
    for tile in TILES:
        print(f"[case] splits {kind} {shape} kernel 1 tile {tile}", flush=True)
        assert torch.equal(_run(kind, shape, WIDE, tile, x, w, bias, aux), base), tile


@pytest.mark.parametrize("n,h,co", [(1, 1, 1), (3, 3, 3), (5, 5, 3), (1, 6, 64), (3, 6, 64), (9, 5, 20), (33, 3, 17)])
def test_column_sums_match_the_gemm_tile(n, h, co):
    """The bias gradient as column sums: the tile kernel's sums bit for bit (one position to several splits of 4096, a
    last one of a few; one to 64 columns, where a split takes many passes through LDS)."""
    x = torch.from_numpy(np.random.default_rng(n * co).standard_normal((n, 1 << h, 1 << h, co)).astype(np.float32)).cuda()
    splits = -(-(n << (2 * h)) // 4096)
    out = []
    for kernel in (ANY, SUM):
        print(f"[case] sums {n} {h} {co} kernel {kernel}", flush=True)
        o = torch.full((splits, co), float("nan"), device="cuda")
        desc = torch.zeros(2048, dtype=torch.uint8, device="cuda")
        L.lipz_test_conv(torch.cuda.current_stream().cuda_stream, desc.data_ptr(), 6, n, h, 1, co, x.data_ptr(),
                         x.data_ptr(), o.data_ptr(), kernel=kernel)
        torch.cuda.synchronize()
        out.append(o.cpu())
    ref = x.cpu().double().reshape(-1, co)
    assert torch.all((out[0].double().sum(0) - ref.sum(0)).abs() <= (4096 + splits) * 2.0 ** -24 * ref.abs().sum(0))
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("kind", ["conv", "convT"])
@pytest.mark.parametrize("shape", [(8, 3, 8, 64), (8, 3, 32, 64), (8, 3, 64, 128), (3, 2, 512, 64), (3, 2, 1024, 32)])
@pytest.mark.parametrize("signs", ["both", "one"])
def test_split_kernel_is_as_accurate_as_fp32_products(kind, shape, signs):
    """Against fp64, from 32 to 16384 products a sum: the bf16 pieces' rms error is no larger than the fp32 MFMAs',
    and their mean error (they drop bits towards minus infinity) is a fraction of it, on sums of one sign too.  (The
    worst-case bounds above leave room for a kernel without its smaller products.)"""
    x, w, bias, aux = _problem(kind, shape, seed=31)
    bias = torch.zeros_like(bias)
    if signs == "one":
        x, w = x.abs(), w.abs()
    ref = _reference(kind, x.double(), w.double(), aux.double(), bias.double())[0]
    scale = ref.pow(2).mean().sqrt()

    def error(kernel, tile):
        e = (_run(kind, shape, kernel, tile, x, w, bias, aux).double() - ref) / scale
        if kind == "conv":  # the activation's slope on negative sums would fold their errors
            e = e[ref > 0]
        return float(e.pow(2).mean().sqrt()), float(e.mean())

    base = error(ANY, (0, 0))
    for kernel in [SPLIT] + ([PRE] if shape[2] % 32 == 0 else []):
        for tile in TILES:
            rms, mean = error(kernel, tile)
            print(f"[case] accuracy {kind} {shape} {signs} kernel {kernel} tile {tile} rms {rms:.2e} mean {mean:.1e} "
                  f"fp32 {base[0]:.2e} {base[1]:.1e}", flush=True)
            assert rms <= base[0], (kernel, tile)
            assert abs(mean) <= 0.25 * base[0], (kernel, tile)
