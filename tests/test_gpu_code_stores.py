"""One-level Strassen orbits with few rows and long B rows, whose codes are
stored 16 bytes at a time as fast as the memory takes them: every error is
that of the realization's own output, whose B codes other kernels form."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synthetic as sy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["e4m3", "e5m2"])
@pytest.mark.parametrize("mode", ["tensor", "rowcol", "group"])
@pytest.mark.parametrize("gauge,G,chunk", [("gl", 64, 0), ("gl", 48, 0), ("gl", 64, 32), ("gl", 64, 8),
                                           ("sign", 8, 0), ("sign", 8, 2)])
def test_orbit_of_few_rows(gauge, G, chunk, mode, fmt):
    from paper_2609_39816_amd import fm
    M, K, N = 16, 1024, 1024
    rng = np.random.default_rng(3)
    A = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).cuda()
    B = torch.from_numpy(rng.standard_normal((K, N)).astype(np.float32)).cuda()
    if gauge == "gl":
        gs = sy.gl_gauges(2, 2, 2, G, 4)
    else:
        gs = [(np.diag(d), np.diag(e), np.diag(f)) for d, e, f in sy.sample_sign_orbit(2, 2, 2, G, 4)]
    orbit = fm.Scheme.base("strassen").gauge_orbit(gs)
    sm = {"tensor": fm.SCALE_TENSOR, "rowcol": fm.SCALE_ROWCOL, "group": fm.SCALE_GROUP}[mode]
    f = fm.FMTS[fmt]
    Cref = fm.reference_f64(A, B)
    ws = fm.workspace(fm.workspace_size(orbit[0], M, N, K, 1, G, chunk, sm))
    errs = fm.orbit_eval(orbit, A, B, Cref, 1, f, ws=ws, scale_mode=sm)
    want = np.array([fm.error_stats(fm.matmul_lowp(s, A, B, 1, f, scale_mode=sm), Cref)["rel_fro"]
                     for s in orbit])
    assert np.all(np.abs(errs / want - 1) <= 1e-9), (errs, want)
