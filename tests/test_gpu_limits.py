"""Calls beyond the limits of one launch's grid."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from oracle import schemes as osch
import synthetic as sy

pytestmark = pytest.mark.gpu


def test_more_gauges_than_grid_slices():
    """Per-row maxima of 128 block-sum rows take one gauge per slice: more
    than 65535 gauges in one chunk.  Two schemes in turn: every error has the
    bits of the orbit of the two."""
    from paper_2609_39816_amd import fm
    M, K, N, G = 512, 64, 4, 65600
    rng = np.random.default_rng(8)
    A = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).cuda()
    B = torch.from_numpy(rng.standard_normal((K, N)).astype(np.float32)).cuda()
    gs = [(np.diag(d), np.diag(e), np.diag(f)) for d, e, f in sy.sample_sign_orbit(4, 4, 4, 2, 4)]
    pair = fm.Scheme.base("strassen").kron(2).gauge_orbit(gs)
    Cref = fm.reference_f64(A, B)
    want = fm.orbit_eval(pair, A, B, Cref, 1, scale_mode=fm.SCALE_ROWCOL)
    errs = fm.orbit_eval(list(pair) * (G // 2), A, B, Cref, 1, scale_mode=fm.SCALE_ROWCOL)
    assert np.array_equal(errs.view(np.uint64).reshape(-1, 2),
                          np.broadcast_to(want.view(np.uint64), (G // 2, 2)))


def test_more_repaired_rows_than_one_grid_row():
    """The row repair takes a workgroup per row: more than 2^24 rows.  Codes
    and scales of the first and last rows are those of a call of them alone."""
    from paper_2609_39816_amd import fm
    M, K, N, n = (1 << 24) + 8, 128, 128, 16
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    A = torch.randn((M, K), generator=g, device="cuda")
    A[-n:] *= torch.exp2(torch.arange(n, device="cuda") - 8.0)[:, None]
    B = torch.randn((K, N), generator=g, device="cuda")
    s = fm.Scheme.base("classical")
    mode = fm.SCALE_GROUP | fm.REPAIR_ROWS
    Tq, _, dT, _ = fm.form_operands(s, A, B, 1, scale_mode=mode)
    for rows in (slice(0, n), slice(M - n, M)):
        tq, _, dt, _ = fm.form_operands(s, A[rows].contiguous(), B, 1, scale_mode=mode)
        assert torch.equal(Tq[:, rows], tq)
        assert torch.equal(dT[:, :, rows].view(torch.int32), dt.view(torch.int32))


def test_inner_length_beyond_the_direct_formation():
    """B's operand is formed from the transposed copy where its rows are more
    strips than the direct kernels' grid holds."""
    from paper_2609_39816_amd import fm
    M, K, N = 1, (1 << 23) + 128, 2
    rng = np.random.default_rng(9)
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = (0.02 * rng.standard_normal((K, N))).astype(np.float32)
    Tq, Sq, dT, dS = fm.form_operands(fm.Scheme.base("classical"), torch.from_numpy(A).cuda(),
                                      torch.from_numpy(B).cuda())
    tabs, (gm, gk, gn, _) = oracle.flatten_f32(osch.BASE_SCHEMES["classical"]())
    tq, dt = oracle.form_operands(A, gm, gk, tabs[0], oracle.E4M3, side=0)
    sq, ds = oracle.form_operands(B, gk, gn, tabs[1], oracle.E4M3, side=1)
    assert np.array_equal(dT.cpu().numpy(), dt.reshape(-1))
    assert np.array_equal(dS.cpu().numpy(), ds.reshape(-1))
    assert np.array_equal(Tq.cpu().numpy(), tq)
    assert np.array_equal(Sq.cpu().numpy(), sq.transpose(0, 2, 1))


def test_more_small_products_than_one_grid_row():
    """A wave per product: more than 2^26 of them.  The first and last are
    those of a call of them alone."""
    from paper_2609_39816_amd import fm
    batch, Kb, n = (1 << 26) + 8, 128, 16
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    T, S = (torch.randint(0, 0x78, (batch, 1, Kb), generator=g, dtype=torch.uint8, device="cuda")
            for _ in range(2))
    dT, dS = (torch.rand(batch, generator=g, device="cuda") + 0.5 for _ in range(2))
    out = torch.full((batch, 1, 1), float("nan"), device="cuda")
    fm.block_products(T, S, dT, dS, out=out)
    for b in (slice(0, n), slice(batch - n, batch)):
        alone = fm.block_products(T[b].contiguous(), S[b].contiguous(), dT[b].contiguous(),
                                  dS[b].contiguous())
        assert torch.isfinite(alone).all()
        assert torch.equal(out[b].view(torch.int32), alone.view(torch.int32))
