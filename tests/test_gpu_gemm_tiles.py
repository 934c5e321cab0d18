"""Every tile of the matrix products, launched directly (a plan's choice moves when its constants do), with sizes one below,
at and one above the tile's, against 64-bit products of the same fp16 operands."""
import pytest

from tests import gemm_calls as gc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def lib():
    from paper_2609_34045_amd import stage
    return stage.load_library()


@pytest.mark.parametrize("tile,rows", [(0, 32), (1, 64)])
def test_row_tiles_take_k_in_one_order(torch, lib, tile, rows):
    """Equal rows of A in different row tiles get the same bits: a tile's start in K depends on its columns alone."""
    n, k = 384, 320
    g = torch.Generator(device="cuda").manual_seed(3)
    a = torch.randn(rows, k, generator=g, device="cuda").half().repeat(128 // rows, 1).contiguous()
    w = torch.randn(n, k, generator=g, device="cuda").half()
    c, err = torch.zeros(128, n, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    assert gc.launch_gemm(lib, gc.RESID, tile, 1, a, w, None, 128, n, k, c, None, err, None) == 0
    torch.cuda.synchronize()
    for r in range(rows, 128, rows):
        assert torch.equal(c[r:r + rows], c[:rows]), r


MARK = 77.0  # outputs past the last row


def operands(torch, m, n, k, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.randn(m, k, generator=g, device="cuda").half()
    w = torch.randn(n, k, generator=g, device="cuda").half()
    return a, w, a.double() @ w.double().T, 2 * k * 2.0 ** -24 * (a.double().abs() @ w.double().abs().T)


def steps(tile):
    """Depths in 64-deep K steps: 1 to 5 and, once past every ring, 9."""
    return [1, 2, 3, 4, 5, 9] if tile in (0, 2, 4, 8) else [1, 3, 4, 5, 9]


@pytest.mark.parametrize("tile", gc.BUILT[gc.RESID])
def test_residual_and_partial_sums(torch, lib, tile):
    """C += A W^T, and the K slices of the same product.  fp32 sums of k products are within 2 k 2^-24 sum |a w| of exact ones
    (each product is added with at most two roundings)."""
    tm, tn = gc.TILES[tile]
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    for nk in steps(tile):
        for m, n in ((tm - 1, tn + 1), (tm, tn), (tm + 1, tn - 1), (1, 2 * tn + 33), (2 * tm + 5, 31)):
            k = 64 * nk
            a, w, ref, tol = operands(torch, m, n, k, 1000 * nk + m)
            c = torch.full((m + 1, n), MARK, device="cuda")
            c[:m] = 3.0
            assert gc.launch_gemm(lib, gc.RESID, tile, 1, a, w, None, m, n, k, c, None, err, None) == 0
            assert ((c[:m].double() - 3.0 - ref).abs() <= tol + 2.0 ** -22 * (3.0 + ref.abs())).all(), (m, n, nk)
            assert (c[m:] == MARK).all(), (m, n, nk)
            for slices in range(1, min(nk, gc.MAX_SLICES) + 1):
                part = torch.full((slices * m + 1, n), MARK, device="cuda")
                assert gc.launch_gemm(lib, gc.PARTIAL, tile, slices, a, w, None, m, n, k, part, None, err, None) == 0
                assert ((part[:-1].view(slices, m, n).double().sum(0) - ref).abs() <= tol).all(), (m, n, nk, slices)
                assert (part[-1] == MARK).all(), (m, n, nk, slices)
    assert err.item() == 0


@pytest.mark.parametrize("tile", gc.BUILT[gc.SWIGLU])
def test_swiglu(torch, lib, tile):
    """silu(gate) up in fp16.  An error d in the gate moves silu by at most 1.1 d; the result rounds to 2^-11 of itself, and
    expf and the division add a few 2^-24."""
    tm, tn = gc.TILES[tile]
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    for nk in steps(tile):
        for m, n in ((tm - 1, tn + 32), (tm, tn), (tm + 1, tn - 32), (1, 2 * tn + 64)):
            k, nout = 64 * nk, n // 2
            a, w, _, _ = operands(torch, m, n, k, 2000 * nk + m)
            a *= 0.1
            ad = a.double()
            g, u = ad @ w[:nout].double().T, ad @ w[nout:].double().T
            tol = 2 * k * 2.0 ** -24 * (ad.abs() @ w.double().abs().T)
            out = torch.full((m + 1, nout), MARK, dtype=torch.half, device="cuda")
            assert gc.launch_gemm(lib, gc.SWIGLU, tile, 1, a, w[:nout], w[nout:], m, n, k, None, out, err, None) == 0
            ref = torch.nn.functional.silu(g) * u
            bound = 1.1 * tol[:, :nout] * u.abs() + torch.nn.functional.silu(g).abs() * tol[:, nout:]
            assert ((out[:m].double() - ref).abs() <= bound + 1.01 * 2.0 ** -11 * ref.abs() + 2.0 ** -24).all(), (m, n, nk)
            assert (out[m:] == MARK).all(), (m, n, nk)
    assert err.item() == 0


@pytest.mark.parametrize("io,rows", [(io, r) for io in ("float32", "bfloat16")
                                     for r in (5, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256)] +
                         [("bfloat16", 257), ("bfloat16", 511)])
def test_logits(torch, lib, io, rows):
    """Every tile gives the same bits, near 64-bit sums: 2^-23 for the operands' two parts and the few roundings of sums that
    are carried, on random rows 4e-7 of a row's logits in the 2-norm (one part alone: 1e-4)."""
    parts = 2 if io == "float32" else 1
    gen = torch.Generator(device="cuda").manual_seed(rows)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    for n, k in ((127, 64), (129, 192), (257, 256), (225, 320), (479, 576), (300, 2048), (33, 2112)):
        x = torch.randn(rows, k, generator=gen, device="cuda").to(getattr(torch, io))
        w = torch.randn(n, k, generator=gen, device="cuda").half()
        a = torch.empty(2 * gc.HEAD_CHUNK, k, dtype=torch.half, device="cuda")
        scale = torch.empty(2 * gc.HEAD_CHUNK, 3, device="cuda")
        xd = x.double()
        ref = xd / (xd.square().mean(1, keepdim=True) + 1e-5).sqrt() @ w.double().T
        first = None
        for tile in gc.BUILT[gc.LOGITS if parts == 1 else gc.LOGITS_SPLIT]:
            y = torch.full((rows + 1, n), MARK, device="cuda")
            assert gc.launch_head_logits(lib, x, None, w, rows, n, k, 1e-5, a, scale, y, err, None, tile) == 0
            first = y if first is None else first
            assert torch.equal(y, first), (n, k, tile)
        assert ((first[:rows].double() - ref).norm(dim=1) <= 4e-7 * ref.norm(dim=1)).all(), (n, k)
        assert (first[rows:] == MARK).all(), (n, k)
    assert err.item() == 0


def test_tiles_that_are_not_built_are_refused(torch, lib):
    t = torch.zeros(256, 256, device="cuda")
    h = torch.zeros(2 * gc.HEAD_CHUNK, 64, dtype=torch.half, device="cuda")
    for x, built in ((t[:8, :64].contiguous(), gc.BUILT[gc.LOGITS_SPLIT]),
                     (t[:8, :64].bfloat16().contiguous(), gc.BUILT[gc.LOGITS])):
        for tile in range(10):
            got = gc.launch_head_logits(lib, x, None, h, 8, 32, 64, 1e-5, h, t, t, t, None, tile)
            assert (got == 0) == (tile in built), tile
    torch.cuda.synchronize()
