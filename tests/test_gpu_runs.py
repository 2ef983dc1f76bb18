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
