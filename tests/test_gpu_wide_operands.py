"""The 256-wide GEMM with operands that travel 64 of K at a time, at K around the lengths of its ring and of its unrolled loop (a stage is a pair
of slabs, 3 stages of A, 2 of B or 4 of its slabs; 6 pairs a turn), whole and in uneven shares of K, against 64-bit products."""
import pytest

from tests import internal as I

pytestmark = pytest.mark.gpu

PAIRS = (1, 2, 3, 4, 7, 8, 9, 13, 14, 21)


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def _slab(t):
    """[rows, K] -> [K / 32][rows][32], flat."""
    rows, k = t.shape
    return t.reshape(rows, k // 32, 32).permute(1, 0, 2).contiguous()


def _operands(torch, M, N, K, matrices, b_slab, seed):
    """Arguments of a gathered product, what they point at, and the 64-bit products with their error bound (an fp32 sum in any order)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.randn((M + 5, K), generator=g, device="cuda").bfloat16()
    idx = torch.sort(torch.randperm(M + 5, generator=g, device="cuda")[:M]).values.int()
    B = [(torch.randn((N, K), generator=g, device="cuda") / K ** 0.5).bfloat16() for _ in range(matrices)]
    a = A[idx.long()].double()
    keep = [A, idx] + [_slab(b) if b_slab else b for b in B]
    args = I.GemmArgs(A=A.data_ptr(), lda=K, a_idx=idx.data_ptr(), a_rows=M + 5, B0=keep[2].data_ptr(), ldb=K, M=M, N=N, K=K, b_slab=int(b_slab), b_rows=N)
    if matrices > 1:
        args.B1 = keep[3].data_ptr()
    return args, keep, [a @ b.double().t() for b in B], [K * 2.0 ** -24 * (a.abs() @ b.double().abs().t()) for b in B]


def _run(torch, args):
    assert I.mfma_supported(args)
    assert I.launch_wide(args, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()


def _close(got, want, slack):
    err = (got.double() - want).abs()
    assert bool((err <= slack + 2.0 ** -8 * want.abs() + 1e-30).all()), float((err - slack - 2.0 ** -8 * want.abs()).max())


@pytest.mark.parametrize("b_slab", [False, True], ids=["rows", "slabs"])
@pytest.mark.parametrize("pairs", PAIRS)
def test_stored_product_whole_and_split(torch, pairs, b_slab):
    for M in (1, 300):
        for ks in (1, 2, 3, 5):
            if ks > pairs:
                continue
            args, keep, (want,), (slack,) = _operands(torch, M, 256, 64 * pairs, 1, b_slab, pairs)
            c = torch.full((M + 9, 256), float("nan"), dtype=torch.bfloat16, device="cuda")
            part = torch.full(((M + 255) // 256 * ks * 65536 + 64,), float("nan"), device="cuda")
            args.C, args.ldc, args.epi, args.part32 = c.data_ptr(), 256, I.EPI_STORE, part.data_ptr()
            if ks > 1:
                args.ksplit, args.nfull = ks, 0
            _run(torch, args)
            _close(c[:M], want, slack)
            assert torch.isnan(c[M:]).all() and torch.isnan(part[-64:]).all()


@pytest.mark.parametrize("epi,b_slab", [(I.EPI_SILU_MUL, False), (I.EPI_SILU_MUL, True), (I.EPI_SILU_MUL_T, False), (I.EPI_SILU_MUL_T, True)],
                         ids=["rows", "slabs", "transposed_rows", "transposed_slabs"])
@pytest.mark.parametrize("pairs", PAIRS)
def test_silu_of_gate_times_up(torch, pairs, epi, b_slab):
    M, N = 300, 128
    args, keep, (g, u), (dg, du) = _operands(torch, M, N, 64 * pairs, 2, b_slab, pairs)
    flip = epi == I.EPI_SILU_MUL_T
    c = torch.full((N, 512) if flip else (M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    args.C, args.ldc, args.epi = c.data_ptr(), c.shape[1], epi
    _run(torch, args)
    silu = g * torch.sigmoid(g)
    # |silu'| <= 1.1; the exponential and the reciprocal are good to 2^-21 of silu(g)
    _close(c[:, :M].t() if flip else c, silu * u, 1.1 * dg * u.abs() + du * silu.abs() + dg * du + 2.0 ** -20 * (silu * u).abs())
