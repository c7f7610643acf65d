"""The grouped GEMM's loads at any alignment and size (lipz_test_gemm): what lies
around an operand's elements (the ends of its rows, the rest of its buffer)
never reaches a result, and a problem's sums do not depend on where its
operands lie."""
import numpy as np
import pytest
import torch

from paper_1811_12843_amd import lipz as L

pytestmark = pytest.mark.gpu

# K below, at and past a slice of 32 and its 16-deep halves, quads cut by the end of a row, one row and column;
# tiles of 32 and 64 rows, whole and cut
SHAPES = [(1, 1, 1), (33, 65, 37), (100, 256, 64), (65, 31, 18), (32, 64, 33), (200, 100, 515), (37, 70, 784)]


def _operand(rows, cols, pad, shift, g):
    """A [rows][cols] operand with row stride cols + pad in a buffer of NaNs, `shift` floats past a 16-byte boundary."""
    ld = cols + pad
    x = g.standard_normal((rows, cols)).astype(np.float32)
    buf = torch.full((shift + rows * ld + 64,), float("nan"), device="cuda")
    view = buf[shift:shift + rows * ld].view(rows, ld)
    view[:, :cols] = torch.from_numpy(x).cuda()
    return x, buf, view, ld


def _run(M, N, K, a_trans, b_trans, pad, shift, tile_rows, variant, seed):
    g = np.random.default_rng(seed)
    A, abuf, a, lda = _operand(*((K, M) if a_trans else (M, K)), pad, shift, g)
    B, bbuf, b, ldb = _operand(*((N, K) if b_trans else (K, N)), pad, shift, g)
    C = torch.full((M + 1, N + pad), 7.0, device="cuda")
    desc = torch.zeros(256, dtype=torch.uint8, device="cuda")
    L.lipz_test_gemm(torch.cuda.current_stream().cuda_stream, desc.data_ptr(), M, N, K, a.data_ptr(), lda, a_trans, -1,
                     b.data_ptr(), ldb, b_trans, C.data_ptr(), N + pad, 0, 0, 0.2, tile_rows=tile_rows, variant=variant)
    torch.cuda.synchronize()
    out = C.cpu().numpy()
    assert np.all(out[M] == 7.0) and np.all(out[:, N:] == 7.0), "written outside the result"
    return (A.T if a_trans else A), (B.T if b_trans else B), out[:M, :N]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0)])
def test_any_alignment_gives_the_same_sums(shape, trans):
    M, N, K = shape
    base = {}
    for tile_rows in (32, 64):
        # row strides and bases that are a multiple of 16 bytes, or not
        for pad_to4, shift in ((True, 0), (False, 0), (False, 1), (False, 3)):
            rows_len = (M if trans[0] else K, K if trans[1] else N)
            pad = 0
            if pad_to4:
                while any((r + pad) % 4 for r in rows_len) and pad < 8:
                    pad += 1
                if any((r + pad) % 4 for r in rows_len):
                    continue  # no common padding aligns both
            variants = (1, 2, 3) if pad_to4 else (0,)
            for v in variants:
                print(f"[case] {shape} {trans} tile {tile_rows} pad {pad} shift {shift} variant {v}", flush=True)
                A, B, out = _run(M, N, K, *trans, pad, shift, tile_rows, v, seed=M + N + K)
                ref = A.astype(np.float64) @ B.astype(np.float64)
                mag = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)
                # at most K + 3 roundings of partial sums
                assert np.all(np.abs(out - ref) <= (K + 3) * 2.0 ** -24 * mag + 1e-30), (tile_rows, pad, shift, v)
                # one chain, or four: the same bits from every kernel, layout and place
                aligned = not any((r + pad) % 4 for r in rows_len) and shift == 0
                chains = 4 if v in (2, 3) or (v == 0 and aligned and K >= 512) else 1
                assert np.array_equal(base.setdefault(chains, out), out), (tile_rows, pad, shift, v)


@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0)])
def test_deep_products_take_four_chains_on_any_kernel(trans):
    """Depths and tile counts on either side of the rule between the two four-chain kernels: the library's choice has
    the bits of both."""
    for M, N, K in ((64, 64, 4064), (64, 64, 4096), (1088, 1024, 4064), (1088, 1024, 4096)):
        print(f"[case] deep {M} {N} {K} {trans}", flush=True)
        out = [_run(M, N, K, *trans, 0, 0, 32, v, seed=K)[2] for v in (0, 2, 3)]
        assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])


@pytest.mark.parametrize("outlier", [1e10, 1e-30, float("inf"), float("nan")])
@pytest.mark.parametrize("rows,fi,fo", [(100, 64, 64), (37, 45, 70)])
def test_adam_short_and_full_divisions_agree(rows, fi, fo, outlier):
    """The weight gradient's Adam step with moments in the range of the short division sequence, and with one element
    per wave and pass outside it (the full sequence for the whole pass): every other element comes out the same."""
    g = np.random.default_rng(rows)
    X = torch.from_numpy(g.standard_normal((rows, fi)).astype(np.float32)).cuda()
    dY = torch.from_numpy((g.standard_normal((rows, fo)) * 1e-2).astype(np.float32)).cuda()
    P0 = g.standard_normal((fi + 1, fo)).astype(np.float32)
    # magnitudes over the whole range, zeros among them
    m0 = (g.standard_normal((fi + 1, fo)) * 10.0 ** g.uniform(-20, 3, (fi + 1, fo))).astype(np.float32)
    v0 = (10.0 ** g.uniform(-25, 3, (fi + 1, fo))).astype(np.float32)
    m0[::3, ::5] = 0.0
    v0[::3, ::5] = 0.0
    at = np.zeros((fi + 1, fo), bool)
    at[::8, ::32] = True
    out = []
    for plant in (False, True):
        m, v = m0.copy(), v0.copy()
        if plant:
            (v if outlier == 1e-30 else m)[at] = np.float32(outlier) * (1e-5 if outlier == 1e-30 else 1.0)
        dX, dYp = X.clone(), dY.clone()
        if outlier == 1e-30:  # no gradient in those rows, so that the moment stays as small
            dX[:, ::8] = 0.0
        t = [torch.from_numpy(a).cuda() for a in (P0.copy(), m, v)]
        lr = torch.tensor([3e-4], device="cuda")
        step = torch.tensor([6], dtype=torch.int32, device="cuda")
        desc = torch.zeros(256, dtype=torch.uint8, device="cuda")
        print(f"[case] adam {rows} {fi} {fo} outlier {outlier} planted {plant}", flush=True)
        L.lipz_test_gemm(torch.cuda.current_stream().cuda_stream, desc.data_ptr(), fi + 1, fo, rows, dX.data_ptr(), fi, 1,
                         fi, dYp.data_ptr(), fo, 0, t[0].data_ptr(), fo, 3, 0, 0.2, d_m=t[1].data_ptr(),
                         d_v=t[2].data_ptr(), d_lr=lr.data_ptr(), d_t=step.data_ptr(), step_local=0, tile_rows=32)
        torch.cuda.synchronize()
        out.append([x.cpu().numpy() for x in t])
    for a, b in zip(*out):
        assert np.isfinite(a).all()
        assert np.array_equal(a[~at], b[~at])


@pytest.mark.parametrize("ends", [False, True])
def test_adam_has_the_bits_of_ieee_divisions(ends):
    """Adam's step without a gradient against numpy's fp32 division and root, bit for bit: moments over the range of
    the short sequences or at its ends (2^-80, 2^-100, 2^20), zeros of both signs, parameters of both zeros."""
    g = np.random.default_rng(int(ends))
    fi, fo, rows, f = 64, 64, 40, np.float32
    shape = (fi + 1, fo)

    def powers(lo, hi):
        e = g.choice([lo, hi - 1], shape) if ends else g.integers(lo, hi, shape)
        near = g.choice([0, 0, 1, 2, (1 << 23) - 1], shape) if ends else g.integers(0, 1 << 23, shape)
        return np.ldexp(1.0 + near * 2.0 ** -23, e).astype(f)

    m, v = powers(-80, 20) * g.choice([-1, 1], shape).astype(f), powers(-100, 20)
    p = g.standard_normal(shape).astype(f) * (m * 0 + g.choice([1, 1e-30], shape).astype(f))
    m[::7, ::3], v[::5, ::4], p[::3, ::5], p[1::3, ::5] = f(0.0), f(0.0), f(0.0), f(-0.0)
    m0, v0 = m * f(2), v * f(2)  # halved exactly by beta = 0.5
    below = np.zeros(shape, bool)
    below[8:24, 32:] = g.random((16, 32)) < 0.3
    p[8:24, 32:48] = f(-0.0)
    m0[below], m[below] = f(-2.0 ** -149), f(-0.0)  # half the smallest subnormal rounds to -0
    t = [torch.from_numpy(a.copy()).cuda() for a in (p, m0, v0)]
    X, dY = torch.zeros(rows, fi, device="cuda"), torch.zeros(rows, fo, device="cuda")
    lr, step = torch.tensor([3e-4], device="cuda"), torch.tensor([6], dtype=torch.int32, device="cuda")
    desc = torch.zeros(256, dtype=torch.uint8, device="cuda")
    print(f"[case] adam ieee ends {ends}", flush=True)
    L.lipz_test_gemm(torch.cuda.current_stream().cuda_stream, desc.data_ptr(), fi + 1, fo, rows, X.data_ptr(), fi, 1, fi,
                     dY.data_ptr(), fo, 0, t[0].data_ptr(), fo, 3, 0, 0.2, d_m=t[1].data_ptr(), d_v=t[2].data_ptr(),
                     d_lr=lr.data_ptr(), d_t=step.data_ptr(), beta1=0.5, beta2=0.5, tile_rows=32)
    torch.cuda.synchronize()
    out = [a.cpu().numpy() for a in t]
    bc = f(1.0 - 0.5 ** 7)
    want = p - f(3e-4) * (m / bc) / (np.sqrt(v / bc) + f(1e-8))
    assert want.dtype == f
    bits = [a.view(np.int32) for a in (out[0], out[1], out[2], want, m, v)]
    assert np.array_equal(bits[1], bits[4]) and np.array_equal(bits[2], bits[5])
    assert np.array_equal(bits[0], bits[3])
