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
