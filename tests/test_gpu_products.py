"""Block products at the edges of every kernel's tiles: rows and columns that
are whole tiles, one more, one less or part of one, either side the longer,
column counts that are no multiple of 4, inner lengths of every kernel."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import synthetic as sy

pytestmark = pytest.mark.gpu

SHAPES = [(128, 256, 128), (128, 1024, 256), (100, 300, 128), (4, 512, 384), (256, 128, 128),
          (250, 260, 128), (100, 301, 128), (255, 129, 128), (257, 132, 256), (301, 136, 128), (129, 514, 128),
          (256, 256, 64), (512, 256, 64), (256, 512, 192), (512, 128, 128), (512, 384, 64),
          (768, 256, 128), (32, 32, 32), (33, 31, 48), (1, 4, 16), (64, 64, 16), (60, 20, 272),
          (16, 200, 80), (3, 3, 128), (128, 128, 128), (2, 640, 128)]


def codes(rng, shape, fmt):
    c = rng.integers(0, 256, shape).astype(np.uint8)
    bad = (c & 0x7f) == 0x7f if fmt == oracle.E4M3 else (c & 0x7f) >= 0x7c
    c[bad] = 0x38
    return c


@pytest.mark.parametrize("mode", ["tensor", "rowcol", "group"])
@pytest.mark.parametrize("Mb,Nb,Kb", SHAPES)
def test_products(Mb, Nb, Kb, mode):
    from paper_2609_39816_amd import fm
    if mode == "group" and (Kb % 128 or Nb % 128 or Mb % 4):
        pytest.skip("group scales need whole groups")
    batch = 5
    rng = np.random.default_rng([Mb, Nb, Kb])
    fmt = "e5m2" if (Mb + Nb) % 3 == 0 else "e4m3"
    fo, fh = (oracle.E4M3, fm.E4M3) if fmt == "e4m3" else (oracle.E5M2, fm.E5M2)
    T, S = codes(rng, (batch, Mb, Kb), fo), codes(rng, (batch, Nb, Kb), fo)
    ng = max(1, Kb // 128)
    shp = {"tensor": ((batch,), (batch,)), "rowcol": ((batch, Mb), (batch, Nb)),
           "group": ((batch, ng, Mb), (batch, ng, max(1, Nb // 128)))}[mode]
    dT = rng.uniform(0.5, 2.0, shp[0]).astype(np.float32)
    dS = rng.uniform(0.5, 2.0, shp[1]).astype(np.float32)
    sm = {"tensor": fm.SCALE_TENSOR, "rowcol": fm.SCALE_ROWCOL, "group": fm.SCALE_GROUP}[mode]
    out = torch.full((batch, Mb, Nb), float("nan"), device="cuda")
    out = fm.block_products(*(torch.from_numpy(x).cuda() for x in (T, S, dT, dS)), fh, out=out,
                            scale_mode=sm).cpu().numpy().astype(np.float64)
    t, s = (oracle.fp8_decode(x, fo).astype(np.float64) for x in (T, S))
    for b in range(batch):
        if mode == "group":
            want = np.zeros((Mb, Nb))
            size = np.zeros((Mb, Nb))
            for g in range(ng):
                k = slice(128 * g, 128 * g + 128)
                d = dT[b, g].astype(np.float64)[:, None] * np.repeat(dS[b, g].astype(np.float64), 128)
                want += (t[b][:, k] @ s[b][:, k].T) * d
                size += (np.abs(t[b][:, k]) @ np.abs(s[b][:, k]).T) * d
            # the fp32 sums, then half a bf16 step
            bound = 2.0 ** -8 * np.abs(want) + 1.01 * (Kb + 8) * 2.0 ** -24 * size
        else:
            d = (dT[b].reshape(-1, 1) * np.ones((Mb, 1))) .astype(np.float64) * dS[b].astype(np.float64)
            want = (t[b] @ s[b].T) * d
            # products are exact; Kb fp32 additions and two scalings
            bound = (Kb + 4) * 2.0 ** -24 * (np.abs(t[b]) @ np.abs(s[b]).T) * d + 1e-30
        assert (np.abs(out[b] - want) <= bound).all(), b


def scaled_codes(rng, shape, fmt):
    return torch.from_numpy(codes(rng, shape, fmt)).cuda()


@pytest.mark.parametrize("mode", ["tensor", "rowcol"])
@pytest.mark.parametrize("batch,Mb,Nb,Kb,pipelined", [
    (5, 256, 512, 1024, True), (7, 768, 1024, 256, True), (3, 256, 256, 896, True),
    (16, 256, 2048, 896, True), (16, 256, 2048, 640, True), (17, 256, 2048, 640, True),
    (17, 256, 2048, 768, False), (43, 768, 256, 1024, False)])
def test_rows_of_odd_256s(batch, Mb, Nb, Kb, pipelined, mode):
    """Up to 128 square tiles the products of an odd number of 256 rows are
    the pipelined kernel's, as those of 128 rows always are: the same sums to
    the bit.  Beyond, from inner lengths of 768 on, they are the wide
    kernel's, as those of 512 rows always are."""
    from paper_2609_39816_amd import fm
    rng = np.random.default_rng([batch, Mb, Nb, Kb])
    T, S = scaled_codes(rng, (batch, Mb, Kb), oracle.E4M3), scaled_codes(rng, (batch, Nb, Kb), oracle.E4M3)
    dT = torch.from_numpy(rng.uniform(0.5, 2, (batch, Mb)).astype(np.float32)).cuda()
    dS = torch.from_numpy(rng.uniform(0.5, 2, (batch, Nb)).astype(np.float32)).cuda()
    sm = fm.SCALE_TENSOR if mode == "tensor" else fm.SCALE_ROWCOL
    sT, sS = (dT[:, 0].contiguous(), dS[:, 0].contiguous()) if mode == "tensor" else (dT, dS)
    out = fm.block_products(T, S, sT, sS, scale_mode=sm)
    rows = 128 if pipelined else 512  # the rows of one kernel's products
    Tp = T[:, :rows] if rows <= Mb else torch.cat([T, T], 1)[:, :rows]
    dp = sT if mode == "tensor" else (dT[:, :rows] if rows <= Mb else torch.cat([dT, dT], 1)[:, :rows])
    part = fm.block_products(Tp.contiguous(), S, dp.contiguous(), sS, scale_mode=sm)
    n = min(rows, Mb)
    assert torch.equal(out[:, :n].view(torch.int32), part[:, :n].view(torch.int32))


@pytest.mark.parametrize("M,K,N,G", [(1024, 1024, 2048, 7), (1024, 3072, 3072, 3), (1024, 4352, 3072, 3)])
def test_a_gauges_bits_do_not_depend_on_the_others(M, K, N, G):
    """Two-level orbits whose products are an odd number of 256 rows, on
    either side of the rule: every error has the bits it has alone, and is
    that of the realization's own output."""
    from paper_2609_39816_amd import fm
    rng = np.random.default_rng([M, K, N])
    A = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).cuda()
    B = torch.from_numpy(rng.standard_normal((K, N)).astype(np.float32)).cuda()
    gs = [(np.diag(d), np.diag(e), np.diag(f)) for d, e, f in sy.sample_sign_orbit(4, 4, 4, G, 4)]
    orbit = fm.Scheme.base("strassen").kron(2).gauge_orbit(gs)
    Cref = fm.reference_f64(A, B)
    errs = fm.orbit_eval(orbit, A, B, Cref, 1)
    for g, s in enumerate(orbit):
        alone = fm.orbit_eval([s], A, B, Cref, 1)
        assert alone.view(np.uint64)[0] == errs.view(np.uint64)[g], g
        st = fm.error_stats(fm.matmul_lowp(s, A, B, 1), Cref)
        assert abs(errs[g] / st["rel_fro"] - 1) <= 1e-9


@pytest.mark.parametrize("Mb,Nb,Kb,tile", [
    (64, 64, 496, False), (64, 64, 528, True), (64, 64, 1040, True), (64, 64, 1024, False),
    (33, 33, 976, False), (33, 33, 1008, True), (64, 32, 1008, False), (64, 32, 1040, True),
    (32, 32, 2032, False), (32, 32, 2064, True), (20, 64, 1360, True)])
def test_small_products_by_inner_length(Mb, Nb, Kb, tile):
    """Beyond 128 KB of loads a product of at most 64 x 64 is a 128 x 128
    tile's, as those of more than 64 rows always are: the same sums to the
    bit."""
    from paper_2609_39816_amd import fm
    rng = np.random.default_rng([Mb, Nb, Kb])
    batch = 3
    T, S = scaled_codes(rng, (batch, Mb, Kb), oracle.E4M3), scaled_codes(rng, (batch, Nb, Kb), oracle.E4M3)
    dT, dS = (torch.from_numpy(rng.uniform(0.5, 2, batch).astype(np.float32)).cuda() for _ in range(2))
    out = fm.block_products(T, S, dT, dS)
    more = torch.cat([T] * (65 // Mb + 1), 1).contiguous()  # more than 64 rows
    part = fm.block_products(more, S, dT, dS)[:, :Mb]
    assert torch.equal(out.view(torch.int32), part.contiguous().view(torch.int32)) == tile
