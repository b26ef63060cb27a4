"""The short-product GEMM at every tile height, unsplit and split, with every epilogue and operand layout it serves, against 64-bit
products: the plan is given, not picked (which plans the layers' own products get is in test_gemm_dispatch.py)."""
import pytest

from tests import internal as I

pytestmark = pytest.mark.gpu

K = 1056                                     # 33 slabs of 32: uneven shares for every split
GUARD = 40                                   # rows behind an output that have to stay as they were


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def _slab(t):
    """[rows, K] -> [K / 32][rows][32], flat."""
    rows, k = t.shape
    return t.reshape(rows, k // 32, 32).permute(1, 0, 2).contiguous()


def _unslab(t, rows, cols):
    return t.reshape(cols // 32, rows, 32).permute(1, 0, 2).reshape(rows, cols)


def _key_slot(key):
    return (key & ~12) | ((key & 4) << 1) | ((key & 8) >> 1)


class Product:
    """Operands, 64-bit products and their error bounds: an fp32 sum of K products in any order, one rounding to bf16."""

    def __init__(self, torch, M, N, seed, gather, a_slab, b_slab, second=0):
        g = torch.Generator(device="cuda").manual_seed(seed)
        rnd = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
        self.torch, self.M, self.N = torch, M, N
        src = M + 7 if gather else M
        self.A = rnd(src, K).bfloat16()
        self.idx = torch.sort(torch.randperm(src, generator=g, device="cuda")[:M]).values.int() if gather else None
        self.B = [(rnd(n, K) / K ** 0.5).bfloat16() for n in (N, second) if n]
        a = (self.A[self.idx.long()] if gather else self.A).double()
        self.sums = [a @ b.double().t() for b in self.B]
        self.slack = [K * 2.0 ** -24 * (a.abs() @ b.double().abs().t()) for b in self.B]
        self.keep = [_slab(self.A) if a_slab else self.A] + [_slab(b) if b_slab else b for b in self.B]
        self.args = I.GemmArgs(A=self.keep[0].data_ptr(), lda=K, B0=self.keep[1].data_ptr(), ldb=K, M=M, N=N, K=K, a_slab=int(a_slab),
                               b_slab=int(b_slab), b_rows=N)
        if gather:
            self.args.a_idx, self.args.a_rows = self.idx.data_ptr(), src
        if second:
            self.args.B1 = self.keep[2].data_ptr()

    def out(self, rows, cols):
        return self.torch.full((rows + GUARD, cols), float("nan"), dtype=self.torch.bfloat16, device="cuda")

    def run(self, tm, ksplit):
        torch, a = self.torch, self.args
        part = torch.full((max(1, I.small_part_bytes(a, tm, ksplit) // 4) + 64,), float("nan"), device="cuda")
        a.part32 = part.data_ptr()
        assert I.small_supported(a)
        assert I.launch_small(a, tm, ksplit, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        assert torch.isnan(part[-64:]).all()


def _close(torch, got, want, slack):
    err = (got.double() - want).abs()
    assert bool((err <= slack + 2.0 ** -8 * want.abs() + 1e-30).all()), float((err - slack - 2.0 ** -8 * want.abs()).max())


def _rows(tm):
    return (1, tm - 1, tm + 1, 2 * tm + 33)


CASES = [pytest.param(tm, ks, slab, id=f"tm{tm}_split{ks}_{'slab' if slab else 'rows'}") for tm in (64, 128, 192) for ks in (1, 2, 5) for slab in (False, True)]


@pytest.mark.parametrize("tm,ksplit,slab", CASES)
def test_store_and_stacked_store(torch, tm, ksplit, slab):
    for M in _rows(tm):
        p = Product(torch, M, 256, M, not slab, slab, slab)           # plain, with the transposed copy of the values
        ldct = (M + 255) // 256 * 256
        c, ct = p.out(M, 256), torch.full((256, ldct), float("nan"), dtype=torch.bfloat16, device="cuda")
        p.args.C, p.args.ldc, p.args.Ct, p.args.ldct = c.data_ptr(), 256, ct.data_ptr(), ldct
        p.run(tm, ksplit)
        _close(torch, c[:M], p.sums[0], p.slack[0])
        assert torch.isnan(c[M:]).all()
        slots = torch.tensor([_key_slot(i) for i in range(M)], device="cuda")
        assert torch.equal(ct[:, slots].t(), c[:M])
        assert torch.isfinite(ct[:, :(M + 63) // 64 * 64]).all()       # the attention multiplies the padding of its last tile by zero
        p = Product(torch, M, 256, M + 1, not slab, slab, slab, second=256)   # columns [256, 512) from a second matrix
        p.args.N, p.args.epi = 512, I.EPI_STORE
        c = p.out(M, 512)
        p.args.C, p.args.ldc, p.args.c_slab = c.data_ptr(), 512, int(slab)
        p.run(tm, ksplit)
        got = _unslab(c.reshape(-1)[:M * 512], M, 512) if slab else c[:M]
        _close(torch, got, torch.cat(p.sums, 1), torch.cat(p.slack, 1))
        assert torch.isnan(c.reshape(-1)[M * 512:]).all()


@pytest.mark.parametrize("tm,ksplit,slab", CASES)
def test_silu_of_gate_times_up(torch, tm, ksplit, slab):
    for M in _rows(tm):
        p = Product(torch, M, 384, M, not slab, slab, slab, second=384)
        c = p.out(M, 384)
        p.args.epi, p.args.C, p.args.ldc, p.args.c_slab = I.EPI_SILU_MUL, c.data_ptr(), 384, int(slab)
        p.run(tm, ksplit)
        (g, u), (dg, du) = p.sums, p.slack
        silu = g * torch.sigmoid(g)
        got = _unslab(c.reshape(-1)[:M * 384], M, 384) if slab else c[:M]
        # |silu'| <= 1.1; the exponential and the reciprocal are good to 2^-21 of silu(g)
        _close(torch, got, silu * u, 1.1 * dg * u.abs() + du * silu.abs() + dg * du + 2.0 ** -20 * (silu * u).abs())
        assert torch.isnan(c.reshape(-1)[M * 384:]).all()


@pytest.mark.parametrize("tm,ksplit,slab", CASES)
def test_residual_into_scattered_rows(torch, tm, ksplit, slab):
    for M in _rows(tm):
        p = Product(torch, M, 512, M, False, slab, slab)
        g = torch.Generator(device="cuda").manual_seed(M)
        rows = torch.sort(torch.randperm(M + 9, generator=g, device="cuda")[:M]).values.int()
        x = (4 * torch.randn((M + 9, 512), generator=g, device="cuda")).bfloat16()
        c = x.clone()
        p.args.epi, p.args.C, p.args.ldc, p.args.c_idx = I.EPI_RESIDUAL, c.data_ptr(), 512, rows.data_ptr()
        p.run(tm, ksplit)
        _close(torch, c[rows.long()], x[rows.long()].double() + p.sums[0], p.slack[0])
        rest = torch.ones(M + 9, dtype=torch.bool, device="cuda")
        rest[rows.long()] = False
        assert torch.equal(c[rest], x[rest])


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("tm,ksplit,slab", CASES)
def test_rotary_alone_and_beside_a_stored_product(torch, tm, ksplit, slab, d):
    for M in _rows(tm):
        for second in (0, 256):
            p = Product(torch, M, 512, M, not slab, slab, slab, second=second)
            ang = torch.rand((M + 5, d // 2), generator=torch.Generator(device="cuda").manual_seed(d), device="cuda") * 6.28
            table = torch.stack([torch.cos(ang), torch.sin(ang)], -1).contiguous()
            at = (torch.arange(M, device="cuda") + 5).flip(0).int()
            q, scale = p.out(M, 512), 0.125
            a = p.args
            a.epi, a.C, a.ldc, a.rope, a.rope_idx, a.head_dim, a.rope_scale = I.EPI_ROPE, q.data_ptr(), 512, table.data_ptr(), at.data_ptr(), d, scale
            if second:
                ldct = (M + 255) // 256 * 256
                v, vt = p.out(M, 256), torch.full((256, ldct), float("nan"), dtype=torch.bfloat16, device="cuda")
                a.epi, a.N, a.n_split, a.C2, a.ldc2, a.Ct, a.ldct, a.b_rows1 = I.EPI_ROPE_STORE, 768, 512, v.data_ptr(), 256, vt.data_ptr(), ldct, 256
            p.run(tm, ksplit)
            s, e = p.sums[0].reshape(M, -1, 2, d // 2), p.slack[0].reshape(M, -1, 2, d // 2)
            cs, sn = (table[at.long(), :, i].double()[:, None, :] for i in (0, 1))
            want = torch.stack([s[:, :, 0] * cs - s[:, :, 1] * sn, s[:, :, 1] * cs + s[:, :, 0] * sn], 2).reshape(M, 512) * scale
            slack = (e.sum(2, keepdim=True) + 2.0 ** -22 * s.abs().sum(2, keepdim=True)).expand_as(s).reshape(M, 512) * scale
            _close(torch, q[:M], want, slack)
            assert torch.isnan(q[M:]).all()
            if second:
                _close(torch, v[:M], p.sums[1], p.slack[1])
                assert torch.isnan(v[M:]).all()
                slots = torch.tensor([_key_slot(i) for i in range(M)], device="cuda")
                assert torch.equal(vt[:, slots].t(), v[:M]) and torch.isfinite(vt[:, :(M + 63) // 64 * 64]).all()


@pytest.mark.parametrize("k", [992, 1024, 4096])
def test_unsplit_sums_are_those_of_the_256_wide_tiles(torch, k):
    """Both kernels add a row's products in the same order when K is not split: which one takes a product does not show in its result."""
    M, N = 300, 512
    g = torch.Generator(device="cuda").manual_seed(k)
    A, B = (torch.randn((n, k), generator=g, device="cuda").bfloat16() for n in (M, N))
    want = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
    a = I.GemmArgs(A=A.data_ptr(), lda=k, B0=B.data_ptr(), ldb=k, ldc=N, M=M, N=N, K=k, C=want.data_ptr())
    stream = torch.cuda.current_stream().cuda_stream
    assert I.mfma_supported(a) and I.launch_wide(a, stream) == 0
    for tm in (64, 128, 192):
        got = torch.zeros_like(want)
        a.C = got.data_ptr()
        assert I.launch_small(a, tm, 1, stream) == 0
        assert torch.equal(got, want), tm


@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("slabs,ksplit", [(95, 1), (96, 1), (97, 1), (98, 1), (99, 1), (101, 1), (193, 2), (195, 2), (292, 3)])
@pytest.mark.parametrize("tm", [64, 192])
def test_long_shares_of_row_major_rows(torch, monkeypatch, tm, slabs, ksplit, gather):
    """Two slabs of A at a time: shares just below and from the length on that takes them, even and odd (a last pair of one slab, the end of the last
    row at the end of the operand), shares that begin in the middle of a line."""
    monkeypatch.setitem(globals(), "K", 32 * slabs)
    for M in _rows(tm):
        p = Product(torch, M, 384, M, gather, False, True, second=384)
        c = p.out(M, 384)
        p.args.epi, p.args.C, p.args.ldc = I.EPI_SILU_MUL, c.data_ptr(), 384
        p.run(tm, ksplit)
        (g, u), (dg, du) = p.sums, p.slack
        silu = g * torch.sigmoid(g)
        _close(torch, c[:M], silu * u, 1.1 * dg * u.abs() + du * silu.abs() + dg * du + 2.0 ** -20 * (silu * u).abs())
        assert torch.isnan(c[M:]).all()
        p = Product(torch, M, 256, M + 1, gather, False, False)
        c = p.out(M, 256)
        p.args.C, p.args.ldc = c.data_ptr(), 256
        p.run(tm, ksplit)
        _close(torch, c[:M], p.sums[0], p.slack[0])
        assert torch.isnan(c[M:]).all()
