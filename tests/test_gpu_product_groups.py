"""Independent products in one launch: the same bits as each product in a launch of its own, whatever the mix of sizes, splits and epilogues."""
import ctypes as C

import pytest

from paper_2601_13155_amd import binding, runtime, synth
from tests import internal as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def _fn(mangled, *args):
    f = getattr(binding.load(), mangled)
    f.restype, f.argtypes = C.c_int, args
    return f


def _small_group(args, plans, stream):
    n = len(args)
    return _fn("_ZN4spts23launch_gemm_small_groupEPKNS_8GemmArgsEPKNS_13GemmSmallPlanEiP12ihipStream_t", C.POINTER(I.GemmArgs), C.POINTER(I.SmallPlan),
               C.c_int, C.c_void_p)((I.GemmArgs * n)(*args), (I.SmallPlan * n)(*[I.SmallPlan(*p) for p in plans]), n, stream)


def _tile32_group(args, bf16, stream):
    n = len(args)
    return _fn("_ZN4spts24launch_gemm_tile32_groupEPKNS_8GemmArgsEibP12ihipStream_t", C.POINTER(I.GemmArgs), C.c_int, C.c_bool, C.c_void_p)((I.GemmArgs * n)(*args), n, bf16, stream)


def _product(torch, M, N, K, epi, dtype, seed, d=64):
    """Arguments with an output of NaNs, and what keeps the memory alive."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.randn((M, K), generator=g, device="cuda").to(dtype)
    B = (torch.randn((N, K), generator=g, device="cuda") / K ** 0.5).to(dtype)
    ang = torch.rand((M, d // 2), generator=g, device="cuda") * 6.28
    table = torch.stack([torch.cos(ang), torch.sin(ang)], -1).contiguous()
    c = torch.full((M + 3, N), float("nan"), dtype=dtype, device="cuda")
    ct = torch.full((N, (M + 255) // 256 * 256), float("nan"), dtype=dtype, device="cuda")
    a = I.GemmArgs(A=A.data_ptr(), lda=K, B0=B.data_ptr(), ldb=K, C=c.data_ptr(), ldc=N, M=M, N=N, K=K, epi=epi, rope=table.data_ptr(), head_dim=d, rope_scale=0.5)
    if epi == I.EPI_STORE:
        a.Ct, a.ldct = ct.data_ptr(), ct.shape[1]
    return a, c, ct, (A, B, table)


SPLITS = [(1, 1, 1), (3, 1, 2), (1, 4, 1), (2, 2, 5), (1, 2), (3, 1)]


@pytest.mark.parametrize("splits", SPLITS, ids=lambda s: "_".join(map(str, s)))
@pytest.mark.parametrize("tm", [64, 128, 192])
def test_short_products(torch, tm, splits):
    stream = torch.cuda.current_stream().cuda_stream
    shapes = [(tm + 1, 512, I.EPI_ROPE), (33, 1024, I.EPI_ROPE), (2 * tm, 256, I.EPI_STORE)]
    got = []
    for together in (True, False):
        made = [_product(torch, M, N, 1056, epi, torch.bfloat16, i) for i, (M, N, epi) in enumerate(shapes[:len(splits)])]
        parts = []
        for (a, *_), ks in zip(made, splits):
            parts.append(torch.full((max(1, I.small_part_bytes(a, tm, ks) // 4) + 64,), float("nan"), device="cuda"))
            a.part32 = parts[-1].data_ptr()
            assert I.small_supported(a)
        if together:
            assert _small_group([m[0] for m in made], [(tm, ks) for ks in splits], stream) == 0
        else:
            for (a, *_), ks in zip(made, splits):
                assert I.launch_small(a, tm, ks, stream) == 0
        torch.cuda.synchronize()
        assert all(torch.isnan(p[-64:]).all() for p in parts)
        got.append([t for m in made for t in m[1:3]])
    for x, y in zip(*got):
        assert torch.equal(torch.nan_to_num(x, nan=7.0), torch.nan_to_num(y, nan=7.0))
    for (M, N, epi), c in zip(shapes, got[0][::2]):
        assert torch.isfinite(c[:M]).all() and torch.isnan(c[M:]).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [1, 2, 3])
def test_32x32_tiles(torch, n, dtype):
    stream, t = torch.cuda.current_stream().cuda_stream, {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    shapes = [(65, 128, I.EPI_ROPE), (31, 200, I.EPI_STORE), (100, 64, I.EPI_ROPE)]
    got = []
    for together in (True, False):
        made = [_product(torch, M, N, 104, epi, t, i, d=32) for i, (M, N, epi) in enumerate(shapes[:n])]
        if together:
            assert _tile32_group([m[0] for m in made], dtype == "bf16", stream) == 0
        else:
            for m in made:
                assert I.launch_generic(m[0], dtype == "bf16", stream) == 0
        torch.cuda.synchronize()
        got.append([x for m in made for x in m[1:3]])
    for x, y in zip(*got):
        assert torch.equal(torch.nan_to_num(x, nan=7.0), torch.nan_to_num(y, nan=7.0))
    for (M, N, epi), c in zip(shapes, got[0][::2]):
        assert torch.isfinite(c[:M]).all() and torch.isnan(c[M:]).all()


@pytest.mark.parametrize("K", [256, 260, 512, 516, 772, 1028, 2052])
@pytest.mark.parametrize("rows", [(65, 31, 100), (1500, 900, 64)], ids=["eight_wavefronts", "four_wavefronts"])
def test_32x32_tiles_of_long_fp32_sums(torch, rows, K):
    """Plain products of K > 256, eight partial sums, with a rotary product of four between them: K at and just beyond a group of every wavefront and of
    half of them, few tiles (eight wavefronts) and many (four).  In one launch, in launches of their own and for 33 of the rows alone the same bits."""
    stream = torch.cuda.current_stream().cuda_stream
    shapes = [(rows[0], 512, I.EPI_STORE), (rows[1], 128, I.EPI_ROPE), (rows[2], 200, I.EPI_STORE)]
    got = []
    for together in (True, False):
        made = [_product(torch, M, N, K, epi, torch.float32, i, d=32) for i, (M, N, epi) in enumerate(shapes)]
        if together:
            assert _tile32_group([m[0] for m in made], False, stream) == 0
        else:
            for m in made:
                assert I.launch_generic(m[0], False, stream) == 0
        torch.cuda.synchronize()
        got.append([x for m in made for x in m[1:3]])
    for x, y in zip(*got):
        assert torch.equal(torch.nan_to_num(x, nan=7.0), torch.nan_to_num(y, nan=7.0))
    for (M, N, epi), (a, c, ct, (A, B, _)) in zip(shapes, made):
        assert torch.isnan(c[M:]).all()
        if epi != I.EPI_STORE:
            assert torch.isfinite(c[:M]).all()
            continue
        ref = A.double() @ B.double().t()
        bound = A.double().abs() @ B.double().abs().t()
        assert bool(((c[:M].double() - ref).abs() <= (K / 8 + 8) * 2.0 ** -24 * bound).all())   # eight chains of K / 8 fused terms, their sum
        whole = c[:M].clone()
        few = min(33, M)
        a.M, a.Ct = few, None
        c.fill_(float("nan"))
        assert I.launch_generic(a, False, stream) == 0
        assert torch.equal(c[:few], whole[:few]) and torch.isnan(c[few:]).all()


def test_products_of_different_kernels_stay_apart(torch):
    """A dense layer with 128 key columns, which the 256-wide tiles do not take, and 512 query columns, which they do: the queries do not
    follow the keys into the 32x32 tiles' launch."""
    shape = synth.ModelShape(D=256, H=4, Hkv=1, d=128, Dff=256, dtype="bf16")
    ctx = runtime.make_context(shape, 300, 1, 16, shape.Dff)
    dw = runtime.upload_layer(synth.make_layer(3, 0, shape, 16), shape, 16)
    ctx.spts_profile_begin()
    runtime.run_layer(ctx, synth.hidden_states(3, 300, shape.D, "bf16"), synth.positions(300), dw, shape, skip=0, probe_len=1, m_attn=300, m_ffn=300)
    assert ctx.spts_profile_end()["q_proj"][1] == 1
