"""The float64 reference kernel at the edges of its tiles: more than
256 whole 128 x 128 tiles with K steps of 16 take the kernel with 16-byte
loads, anything else (fewer tiles, a remainder in any dimension, a
misaligned operand) the one with guarded loads."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SHAPES = [(128, 16, 128), (128, 48, 256), (384, 32, 128), (128, 17, 128), (129, 16, 128),
          (128, 16, 127), (1, 1, 1), (3, 70, 260), (257, 33, 131), (2048, 32, 2048), (2176, 16, 2048),
          (2176, 48, 2176)]


@pytest.mark.parametrize("M,K,N", SHAPES)
@pytest.mark.parametrize("shift", [0, 1])
def test_reference_tiles(M, K, N, shift):
    from paper_2609_39816_amd import fm
    rng = np.random.default_rng(M * 7 + K * 3 + N)
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = rng.standard_normal((K, N)).astype(np.float32)

    def device(X):  # shift 1: contiguous, 4 bytes off a 16-byte boundary
        t = torch.empty(X.size + 1, dtype=torch.float32, device="cuda")[shift:shift + X.size]
        t.copy_(torch.from_numpy(X).reshape(-1))
        return t.reshape(X.shape)
    out = fm.reference_f64(device(A), device(B)).cpu().numpy()
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    # products are exact in float64; K additions, each within half an ulp of
    # a partial sum, on either side
    bound = 2 * K * 2.0 ** -53 * (np.abs(A64) @ np.abs(B64))
    assert (np.abs(out - A64 @ B64) <= bound).all()
