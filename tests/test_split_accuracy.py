"""Three bf16 pieces of an fp32 value (the evaluation's convolutions), emulated on
the CPU: what the pieces hold, what the products left out can be, and that a
comparison of rms errors with fp32 products notices a missing piece product."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

SCALE = 2.0 ** 16


def _pieces(x):
    """The bf16 pieces of fp32 values scaled by 2^16, as fp64."""
    r, out = x * np.float32(SCALE), []
    for _ in range(3):
        p = torch.from_numpy(r).bfloat16().float().numpy()
        out.append(p.astype(np.float64))
        r = r - p
    assert r.dtype == np.float32 and not r.any()
    return out


@pytest.mark.parametrize("exponent", [0, 90, -60, -110, -125, -140])
def test_pieces_hold_every_bit(exponent):
    x = np.ldexp(np.random.default_rng(exponent + 200).standard_normal(20000), exponent).astype(np.float32)
    p = _pieces(x)
    v = np.abs(x.astype(np.float64)) * SCALE
    assert np.array_equal(p[0] + p[1] + p[2], x.astype(np.float64) * SCALE)
    assert np.all(np.abs(p[1]) <= 2.0 ** -8 * v) and np.all(np.abs(p[2]) <= 2.0 ** -17 * v)


@pytest.mark.parametrize("K", [80, 512, 4096])
def test_a_missing_piece_product_shows_in_the_rms_error(K):
    g = np.random.default_rng(K)
    A, B = g.standard_normal((64, K)).astype(np.float32), g.standard_normal((K, 64)).astype(np.float32)
    a, b = _pieces(A), _pieces(B)
    ref = A.astype(np.float64) @ B.astype(np.float64)
    left = sum(np.abs(a[i]) @ np.abs(b[j]) for i in range(3) for j in range(3) if i + j > 2) / SCALE ** 2
    assert np.all(left <= (2.0 ** -24 + 2.0 ** -34) * (np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)))
    chain = np.zeros((64, 64), np.float32)
    for k in range(K):  # a fused multiply-add's sum: the product is exact in fp64
        chain = (chain.astype(np.float64) + A[:, k, None].astype(np.float64) * B[k].astype(np.float64)).astype(np.float32)

    def rms(c):
        return np.sqrt(np.mean((c - ref) ** 2))

    pairs = [(i, j) for i in range(3) for j in range(3) if i + j <= 2]
    assert rms(sum(a[i] @ b[j] for i, j in pairs) / SCALE ** 2) < 0.5 * rms(chain)
    for missing in pairs:
        part = sum(a[i] @ b[j] for i, j in pairs if (i, j) != missing) / SCALE ** 2
        assert rms(part) > 1.2 * rms(chain), missing
