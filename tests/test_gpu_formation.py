"""Operand formation at the edges of its tiles, bit for bit against the
oracle: block-row lengths that are one lane's worth, part of a wave, a wave
and several workgroups, odd row counts, one block of scales and several, and
orbits whose gauges share a workgroup.  B's side both straight from B and from
its transposed copy, which orbits form it from."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from oracle import scheme_ops as so
from oracle import schemes as osch
import synthetic as sy

pytestmark = pytest.mark.gpu


def gauge(base, levels, seed):
    n = {"strassen": 2, "laderman": 3, "classical": 1}[base]
    if base == "strassen" and levels > 1:
        d, e, f = sy.sample_sign_orbit(n ** levels, n ** levels, n ** levels, 3, seed)[2]
        return (np.diag(d), np.diag(e), np.diag(f)), True
    return (sy.gl_gauges(n, n, n, 1, seed)[0] if base != "classical" else (np.eye(1),) * 3), False


CASES = [(b, l, m, Mb, Kb, Nb)
         for b, l, m, shapes in [
             ("strassen", 1, "rowcol", [(1, 16, 3), (7, 48, 37), (37, 64, 2), (5, 1040, 66)]),
             ("strassen", 2, "rowcol", [(1, 16, 2), (33, 48, 67), (7, 32, 130), (65, 64, 6),
                                        (3, 128, 257), (2, 1040, 3), (4, 2304, 34)]),
             ("strassen", 3, "rowcol", [(3, 16, 5), (17, 48, 2)]),
             ("laderman", 1, "rowcol", [(5, 16, 4), (9, 144, 65)]),
             ("classical", 1, "rowcol", [(9, 80, 33)]),
             ("strassen", 1, "group", [(4, 128, 128), (132, 384, 256)]),
             ("strassen", 2, "group", [(4, 128, 128), (36, 256, 384)]),
             ("strassen", 3, "group", [(4, 128, 128), (12, 256, 256)]),
             ("laderman", 1, "group", [(8, 256, 128)]),
             ("strassen", 1, "tensor", [(1, 16, 1), (5, 48, 35), (33, 144, 66)]),
             ("strassen", 2, "tensor", [(1, 16, 2), (9, 48, 33), (2, 272, 130)]),
             ("laderman", 1, "tensor", [(3, 16, 3), (7, 144, 34)]),
             ("classical", 1, "tensor", [(5, 16, 7), (130, 272, 34)])]
         for Mb, Kb, Nb in shapes]


def off_boundary(B):
    """B off an 8-byte boundary: one scheme's operand is then formed from the
    transposed copy, by the kernels orbits use."""
    t = torch.empty(B.numel() + 1, dtype=torch.float32, device=B.device)[1:]
    t.copy_(B.reshape(-1))
    return t.reshape(B.shape)


@pytest.mark.parametrize("fmt", ["e4m3", "e5m2"])
@pytest.mark.parametrize("base,levels,mode,Mb,Kb,Nb", CASES)
def test_operands(base, levels, mode, Mb, Kb, Nb, fmt):
    from paper_2609_39816_amd import fm
    n = {"strassen": 2, "laderman": 3, "classical": 1}[base] ** levels
    M, K, N = Mb * n, Kb * n, Nb * n
    rng = np.random.default_rng([Mb, Kb, Nb, levels])
    A = rng.standard_normal((M, K)).astype(np.float32)
    A[:, rng.integers(0, K, 3)] *= 50.0
    A[M // 2] = 0.0  # a row of zeros: scale 1
    B = (0.02 * rng.standard_normal((K, N))).astype(np.float32)
    g, flat = gauge(base, levels, 5)
    hb, ob = fm.Scheme.base(base), osch.BASE_SCHEMES[base]()
    if flat:
        h, o, lv = hb.kron(levels).gauge(*g), so.gauge(so.power(ob, levels), *g), 1
    else:
        h, o, lv = hb.gauge(*g), so.power(so.gauge(ob, *g), levels), levels
    tabs, (gm, gk, gn, R) = oracle.flatten_f32(o)
    sm = {"tensor": 0, "rowcol": 1, "group": 2}[mode]
    ho, oo = ((fm.E4M3, oracle.E4M3) if fmt == "e4m3" else (fm.E5M2, oracle.E5M2))
    om = [oracle.SCALE_TENSOR, oracle.SCALE_ROWCOL, oracle.SCALE_GROUP][sm]
    Tq, Sq, dT, dS = fm.form_operands(h, torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), lv,
                                      ho, scale_mode=sm)
    tq, dt = oracle.form_operands(A, gm, gk, tabs[0], oo, scale_mode=om, side=0)
    sq, ds = oracle.form_operands(B, gk, gn, tabs[1], oo, scale_mode=om, side=1)
    assert np.array_equal(dT.cpu().numpy().view(np.uint32).reshape(-1), dt.view(np.uint32).reshape(-1))
    assert np.array_equal(dS.cpu().numpy().view(np.uint32).reshape(-1), ds.view(np.uint32).reshape(-1))
    assert np.array_equal(Tq.cpu().numpy(), tq)
    assert np.array_equal(Sq.cpu().numpy(), sq.transpose(0, 2, 1))
    _, Sq, _, dS = fm.form_operands(h, torch.from_numpy(A).cuda(),
                                    off_boundary(torch.from_numpy(B).cuda()), lv, ho, scale_mode=sm)
    assert np.array_equal(dS.cpu().numpy().view(np.uint32).reshape(-1), ds.view(np.uint32).reshape(-1))
    assert np.array_equal(Sq.cpu().numpy(), sq.transpose(0, 2, 1))


@pytest.mark.parametrize("levels,mode,shape,G", [
    (2, "rowcol", (36, 64, 40), 70), (2, "rowcol", (128, 128, 128), 33), (1, "rowcol", (64, 96, 10), 40),
    (2, "group", (512, 1024, 1536), 40), (1, "group", (264, 256, 256), 130),
    (1, "group", (16, 1024, 1024), 64), (2, "group", (16, 1024, 2048), 128)])
def test_orbit_gauges_share_workgroups(levels, mode, shape, G):
    """Every gauge's error has the bits it has alone.  The last two have so
    many 128 x 128 blocks that a workgroup takes a whole one (alone: an
    eighth)."""
    from paper_2609_39816_amd import fm
    M, K, N = shape
    rng = np.random.default_rng(3)
    A = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).cuda()
    B = torch.from_numpy(rng.standard_normal((K, N)).astype(np.float32)).cuda()
    n = 2 ** levels
    if levels == 1:
        gs = sy.gl_gauges(2, 2, 2, G, 4)
    else:
        gs = [(np.diag(d), np.diag(e), np.diag(f)) for d, e, f in sy.sample_sign_orbit(n, n, n, G, 4)]
    orbit = fm.Scheme.base("strassen").kron(levels).gauge_orbit(gs) if levels > 1 else \
        fm.Scheme.base("strassen").gauge_orbit(gs)
    sm = {"rowcol": 1, "group": 2}[mode]
    Cref = fm.reference_f64(A, B)
    errs = fm.orbit_eval(orbit, A, B, Cref, 1, scale_mode=sm)
    for g in (0, 1, G // 2, G - 1):
        alone = fm.orbit_eval([orbit[g]], A, B, Cref, 1, scale_mode=sm)
        assert alone.view(np.uint64)[0] == errs.view(np.uint64)[g], g


@pytest.mark.parametrize("K", [128, 896, 1024, 2048, 3968, 4096, 4224, 8192, 8320])
def test_row_repair_lengths(K):
    """Rows shorter than, as long as and longer than the 4096 values a
    workgroup loads at once, with squares that sum to a power of two and one unit beside it."""
    from paper_2609_39816_amd import fm
    rng = np.random.default_rng(K)
    M, N = 24, 128
    A = (rng.standard_normal((M, K)) * np.exp2(rng.integers(-6, 7, (M, 1)))).astype(np.float32)
    A[3] = 0.0
    A[4] = 0.25  # mean square exactly 2^-4
    A[5] = 0.25
    A[5, K - 1] = np.nextafter(np.float32(0.25), np.float32(1))
    B = (0.02 * rng.standard_normal((K, N))).astype(np.float32)
    k = oracle.row_exponents(A)
    As = (A * np.exp2(-k.astype(np.float64))[:, None]).astype(np.float32)
    s = fm.Scheme.base("classical")
    Tq, _, dT, _ = fm.form_operands(s, torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), 1,
                                    scale_mode=fm.SCALE_GROUP | fm.REPAIR_ROWS)
    tabs, (gm, gk, _, _) = oracle.flatten_f32(osch.BASE_SCHEMES["classical"]())
    tq, dt = oracle.form_operands(As, gm, gk, tabs[0], oracle.E4M3, scale_mode=oracle.SCALE_GROUP,
                                  side=0)
    assert np.array_equal(dT.cpu().numpy().view(np.uint32).reshape(-1), dt.view(np.uint32).reshape(-1))
    assert np.array_equal(Tq.cpu().numpy(), tq)
