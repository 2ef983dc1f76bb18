"""The integer quantizer and the classical operator at the edges of their
kernels, bit for bit against the oracle: every group length's kernel, an
operand off a 16-byte boundary, a last wave that is partly empty, groups of
zeros; products in one group per K step and in several."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("rows,K,g", [(1, 64, 64), (5, 192, 64), (3, 128, 128), (17, 640, 128),
                                      (9, 768, 256), (2, 192, 192), (4, 1024, 512), (33, 256, 256)])
def test_quantizer(rows, K, g, shift):
    from paper_2609_39816_amd import fm
    rng = np.random.default_rng([rows, K, g])
    X = (rng.standard_normal((rows, K)) * 3).astype(np.float32)
    X[rows // 2, :g] = 0.0
    X[0, 0] = 1000.0
    t = torch.empty(X.size + 1, dtype=torch.float32, device="cuda")[shift:shift + X.size]
    t.copy_(torch.from_numpy(X).reshape(-1))
    for b in (31, 127):
        codes, d = fm.int8_quantize(t.reshape(X.shape), g, b)
        oc, od = oracle.int8_quantize_a(X, g, b)
        assert np.array_equal(codes.cpu().numpy(), oc)
        got, want = d.cpu().numpy(), np.asarray(od, np.float32)
        want = want if want.shape == got.shape else want.T
        assert np.array_equal(got.view(np.uint32), np.ascontiguousarray(want).view(np.uint32))


@pytest.mark.parametrize("M,N,K,g", [(4, 4, 128, 128), (256, 128, 256, 128), (260, 132, 384, 128),
                                     (300, 260, 512, 256), (64, 516, 1024, 512)])
def test_classical(M, N, K, g):
    from paper_2609_39816_amd import fm
    rng = np.random.default_rng([M, N, K])
    A = rng.standard_normal((M, K)).astype(np.float32)
    BT = rng.standard_normal((N, K)).astype(np.float32)
    ac, da = fm.int8_quantize(torch.from_numpy(A).cuda(), g, 127)
    bc, db = fm.int8_quantize(torch.from_numpy(BT).cuda(), g, 127)
    got = fm.int8_matmul_classical(ac, da, bc, db, g).cpu().numpy()
    a, b = ac.cpu().numpy().astype(np.int64), bc.cpu().numpy().astype(np.int64)
    dA, dB = da.cpu().numpy(), db.cpu().numpy()
    out = np.zeros((M, N), np.float32)
    for i in range(K // g):  # (P dA) dB in fp32, added in fp32, group by group
        k = slice(g * i, g * i + g)
        p = (a[:, k] @ b[:, k].T).astype(np.float32)
        out = out + (p * dA[i][:, None]) * dB[i][None, :]
    assert np.array_equal(got.view(np.uint32), out.view(np.uint32))
