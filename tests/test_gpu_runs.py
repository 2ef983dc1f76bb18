"""Chunks that hold gauges of several kernel families: each run of one family
goes to its own kernels, a chunk of short runs to the generic ones.  Either
way every gauge's error has the bits it has alone."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synthetic as sy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["tensor", "rowcol", "group", "group+rows+weights"])
@pytest.mark.parametrize("scheme,ids,chunk", [
    ("strassen", {0}, 0), ("strassen", {0, 12}, 0), ("strassen", {0, 2, 4, 6, 8}, 0),
    ("strassen", {0, 23}, 12), ("laderman", {5}, 0)])
def test_runs_of_families(scheme, ids, chunk, mode):
    from paper_2609_39816_amd import fm
    n = 2 if scheme == "strassen" else 3
    G = 24
    A, B = sy.operands(sy.scaled(sy.WORKLOADS["strassen1_256_gl64"], 128 * n, 128 * n, 128 * n))
    At, Bt = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    dense = sy.gl_gauges(n, n, n, G, 11)
    gauges = [(np.eye(n),) * 3 if i in ids else dense[i] for i in range(G)]
    orbit = fm.Scheme.base(scheme).gauge_orbit(gauges)
    sm = {"tensor": fm.SCALE_TENSOR, "rowcol": fm.SCALE_ROWCOL, "group": fm.SCALE_GROUP,
          "group+rows+weights": fm.SCALE_GROUP | fm.REPAIR_ROWS | fm.REPAIR_WEIGHTS}[mode]
    Cref = fm.reference_f64(At, Bt)
    M = 128 * n
    ws = fm.workspace(fm.workspace_size(orbit[0], M, M, M, 1, G, chunk, sm))
    errs = fm.orbit_eval(orbit, At, Bt, Cref, 1, ws=ws, scale_mode=sm)
    alone = [fm.orbit_eval([s], At, Bt, Cref, 1, scale_mode=sm)[0] for s in orbit]
    assert np.array_equal(errs.view(np.uint64), np.array(alone).view(np.uint64))


@pytest.mark.parametrize("fmt", ["e4m3", "e5m2"])
@pytest.mark.parametrize("chunk", [0, 12])
@pytest.mark.parametrize("scheme,Mb,Kb,Nb", [
    ("strassen", 512, 128, 256), ("strassen", 512, 64, 128), ("strassen", 256, 128, 128),
    ("laderman", 512, 128, 256)])
def test_runs_in_the_tiled_layout(scheme, Mb, Kb, Nb, chunk, fmt):
    """The identity before dense gauges where the products are whole tiles
    (256 x 256, 512 x 128 and 256 x 128) and go to the reconstruction tile by
    tile: every error is that of the realization's own output, whose products
    are stored by rows (the same output bits, sums in another order)."""
    from paper_2609_39816_amd import fm
    n, G = (2 if scheme == "strassen" else 3), 24
    rng = np.random.default_rng([Mb, Kb, Nb, n])
    A = torch.from_numpy(rng.standard_normal((Mb * n, Kb * n)).astype(np.float32)).cuda()
    B = torch.from_numpy(rng.standard_normal((Kb * n, Nb * n)).astype(np.float32)).cuda()
    orbit = fm.Scheme.base(scheme).gauge_orbit([(np.eye(n),) * 3] + sy.gl_gauges(n, n, n, G - 1, 11))
    f = fm.FMTS[fmt]
    Cref = fm.reference_f64(A, B)
    ws = fm.workspace(fm.workspace_size(orbit[0], Mb * n, Nb * n, Kb * n, 1, G, chunk))
    errs = fm.orbit_eval(orbit, A, B, Cref, 1, f, ws=ws)
    for g, s in enumerate(orbit):
        st = fm.error_stats(fm.matmul_lowp(s, A, B, 1, f), Cref)
        assert abs(errs[g] / st["rel_fro"] - 1) <= 1e-9, (g, errs[g], st["rel_fro"])
