"""Row norms of a split product, taken from its shares: against the norms of the stored bf16 product of the same plan."""
import ctypes as C

import pytest

from paper_2601_13155_amd import binding
from tests import internal as I

pytestmark = pytest.mark.gpu

K = 2112   # 66 slabs of 32, 33 pairs: uneven shares


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def _launch_norm(a, plan, s_mha, c, s, stream):
    f = getattr(binding.load(), "_ZN4spts16launch_gemm_normERKNS_8GemmArgsEPKNS_13GemmSmallPlanEPKfPfS8_P12ihipStream_t")
    f.restype, f.argtypes = C.c_int, [C.POINTER(I.GemmArgs), C.POINTER(I.SmallPlan), C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p]
    return f(a, plan, s_mha, c, s, stream)


@pytest.mark.parametrize("tm,ksplit", [(64, 2), (64, 5), (128, 2), (192, 3), (256, 2), (256, 7)])
def test_norms_are_those_of_the_stored_product(torch, tm, ksplit):
    stream = torch.cuda.current_stream().cuda_stream
    for M in (1, 15, tm - 1, tm, tm + 17, 9 * tm + 5):   # 9 row tiles: more than one group of the short tiles' numbering
        g = torch.Generator(device="cuda").manual_seed(M)
        A = torch.randn((M, K), generator=g, device="cuda").bfloat16()
        B = (torch.randn((256, K), generator=g, device="cuda") / K ** 0.5).bfloat16()
        s_mha = torch.rand(M, generator=g, device="cuda")
        z = torch.full((M, 256), float("nan"), dtype=torch.bfloat16, device="cuda")
        a = I.GemmArgs(A=A.data_ptr(), lda=K, B0=B.data_ptr(), ldb=K, C=z.data_ptr(), ldc=256, M=M, N=256, K=K, epi=I.EPI_STORE)
        wide = tm == 256
        floats = (M + 255) // 256 * ksplit * 65536 if wide else I.small_part_bytes(a, tm, ksplit) // 4
        part = torch.full((floats + 64,), float("nan"), device="cuda")
        a.part32 = part.data_ptr()
        if wide:
            a.ksplit, a.nfull = ksplit, 0
        assert (I.launch_wide(a, stream) if wide else I.launch_small(a, tm, ksplit, stream)) == 0
        torch.cuda.synchronize()
        want = z.double().norm(dim=1)
        z.fill_(float("nan"))
        part.fill_(float("nan"))
        c, s = (torch.full((M + 40,), float("nan"), device="cuda") for _ in range(2))
        plan = None if wide else I.SmallPlan(tm, ksplit)
        assert _launch_norm(a, plan, s_mha.data_ptr(), c.data_ptr(), s.data_ptr(), stream) == 0
        torch.cuda.synchronize()
        assert torch.isnan(z).all() and torch.isnan(c[M:]).all() and torch.isnan(s[M:]).all() and torch.isnan(part[-64:]).all()
        # 256 squares summed in fp32 in some order, a square root and a product: 256 * 2^-24 is far above what that loses
        assert bool(((c[:M].double() - want).abs() <= 2.0 ** -16 * want).all())
        assert bool(((s[:M].double() - want * s_mha.double()).abs() <= 2.0 ** -16 * want).all())
        assert _launch_norm(a, plan, None, None, s.data_ptr(), stream) == 0   # no S^MHA: the norm itself
        torch.cuda.synchronize()
        assert torch.equal(s[:M], c[:M])
