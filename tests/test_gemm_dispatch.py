"""Host side of the GEMM dispatch (no kernel runs here)."""
import ctypes as C
import os
import re

import pytest

from paper_2601_13155_amd import binding
from tests import internal as I

HIP_INVALID_VALUE = 1
A16 = 1 << 20   # an aligned address that is never read


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__ as g
        g.build()
    return binding.load()


def test_argument_struct_has_the_fields_of_the_header():
    """Names and order of tests.internal.GemmArgs against the declaration it mirrors."""
    src = open(os.path.join(os.path.dirname(binding.LIB_PATH), "csrc", "spts_internal.h")).read()
    body = re.sub(r"//[^\n]*", "", re.search(r"struct GemmArgs \{(.*?)\n\};", src, re.S).group(1))
    names, size = [], {"*": 8, "int64_t": 8, "int32_t": 4, "float": 4}
    for decl in filter(str.strip, body.split(";")):
        t, rest = re.match(r"\s*(?:const\s+)?(\w+)(.*)", decl, re.S).groups()
        for n in rest.split(","):
            names.append((n.replace("*", "").strip(), size["*" if "*" in rest else t]))
    assert names == [(n, C.sizeof(t)) for n, t in I.GemmArgs._fields_]


@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "f32"])
def test_general_gemm_refuses_the_channel_major_epilogue(bf16):
    """Only the 256-wide matrix-core kernel stores channel-major: the kernels for any shape would take the product for a plain one and
    write rows at the channels' pitch."""
    for K in (64, 62):   # whole 16-byte chunks, and the element-wise kernel's rows
        a = I.GemmArgs(A=A16, lda=K, B0=A16, B1=A16, ldb=K, C=A16, ldc=256, M=40, N=128, K=K, epi=I.EPI_SILU_MUL_T)
        assert not I.tile32_supported(a, bf16)
        assert I.launch_generic(a, bf16) == HIP_INVALID_VALUE


def test_groups_of_32x32_tiles_are_no_larger_than_a_launch():
    """2^23 workgroups of 256 threads: larger products keep their own launches instead of failing in one."""
    f = getattr(binding.load(), "_ZN4spts27gemm_tile32_group_supportedEPKNS_8GemmArgsEib")
    f.restype, f.argtypes = C.c_bool, [C.POINTER(I.GemmArgs), C.c_int, C.c_bool]
    for M, fits in ((32 << 15, True), ((32 << 15) + 1, False)):   # 128 and 128 column tiles: plain, and rotary pairs of twice the columns
        two = [I.GemmArgs(A=A16, lda=64, B0=A16, ldb=64, C=A16, ldc=n, M=M, N=n, K=64, epi=epi, head_dim=64, rope=A16)
               for n, epi in ((4096, I.EPI_STORE), (8192, I.EPI_ROPE))]
        assert all(I.tile32_supported(a, False) for a in two)
        assert f((I.GemmArgs * 2)(*two), 2, False) == fits


@pytest.mark.parametrize("M,N,K,waves", [(256, 1024, 512, 8), (257, 1024, 512, 4), (1500, 512, 688, 4), (6000, 256, 1376, 8), (6000, 256, 1024, 4), (6000, 260, 2052, 4),
                                         (3000, 256, 2752, 4), (64, 64, 260, 8), (64, 64, 256, 4)])
def test_plain_fp32_products_of_many_tiles_keep_four_wavefronts(M, N, K, waves):
    """Eight where every tile has a CU for itself (256 tiles), and for very long sums of many rows to few columns."""
    f = getattr(binding.load(), "_ZN4spts17gemm_tile32_wavesERKNS_8GemmArgsEb")
    f.restype, f.argtypes = C.c_int, [C.POINTER(I.GemmArgs), C.c_bool]
    for epi in (I.EPI_STORE, I.EPI_RESIDUAL):
        a = I.GemmArgs(A=A16, lda=K, B0=A16, ldb=K, C=A16, ldc=N, M=M, N=N, K=K, epi=epi)
        assert f(a, False) == waves and f(a, True) == 4
    a.epi, a.head_dim, a.rope = I.EPI_ROPE, 4, A16
    assert f(a, False) == 4


def _layer_products(D, QD, KV, Dff, r, d, N, Ma, Mf, P):
    """The products of one skip layer over N rows with Ma / Mf active ones, as the layer call sets them up (row-major weights)."""
    def g(M, n, k, epi, **kw):
        return I.GemmArgs(A=A16, lda=k, B0=A16, ldb=k, C=A16, ldc=n, M=M, N=n, K=k, epi=epi, head_dim=d, rope=A16, **kw)
    return {"k": g(N, KV, D, I.EPI_ROPE), "probe_q": g(P, QD, D, I.EPI_ROPE),
            "qv": g(Ma, QD + KV, D, I.EPI_ROPE_STORE, n_split=QD, B1=A16, C2=A16, ldc2=KV, Ct=A16, ldct=(Ma + 255) // 256 * 256, a_idx=A16, a_rows=N),
            "o": g(Ma, D, QD, I.EPI_RESIDUAL, c_idx=A16), "proxy_in": g(N, 2 * r, D, I.EPI_STORE, B1=A16), "z": g(N, r, Dff, I.EPI_STORE),
            "gate_up": g(Mf, Dff, D, I.EPI_SILU_MUL, B1=A16, a_idx=A16, a_rows=N), "down": g(Mf, D, Dff, I.EPI_RESIDUAL, c_idx=A16)}


def test_short_prompts_reach_every_tile_height_and_both_splits():
    """Plans of the products of short prompts (8B shape): each tile height is taken unsplit and split, the rotary, merged and
    residual products are split; a product of many rows stays with the 256-wide tiles.  What the plans compute is in
    test_gpu_short_products.py."""
    seen = {}
    for N in (65, 250, 333, 600, 1025, 2000):
        for name, a in _layer_products(4096, 4096, 1024, 14336, 256, 128, N, int(0.4 * N), int(0.4 * N), 64).items():
            assert I.small_supported(a), name
            plan = I.small_pick(a, 64 << 20)
            if plan:
                tm, ks = plan
                assert tm in (64, 128, 192) and 1 <= ks <= 16 and (ks == 1 or a.K // ks >= 1024) and I.small_part_bytes(a, tm, ks) <= 64 << 20
                seen.setdefault((tm, ks > 1), set()).add(name)
    assert {tm for tm, split in seen if not split} == {64, 128, 192} and {tm for tm, split in seen if split} == {64, 128, 192}, seen
    assert {"k", "qv", "o", "down"} <= set.union(*(names for (_, split), names in seen.items() if split)), seen
    for name, a in _layer_products(4096, 4096, 1024, 14336, 256, 128, 32768, 13107, 13107, 64).items():
        if name in ("qv", "o", "gate_up", "down"):
            assert I.small_pick(a, 64 << 20) is None, name


# products that were measured to be faster on the 256-wide tiles: us there / on the small tiles that a model without the epilogues chose
@pytest.mark.parametrize("epi,M,N,K", [
    pytest.param(I.EPI_STORE, 20011, 256, 512, id="16.6_18.4"), pytest.param(I.EPI_STORE, 2643, 4096, 128, id="11.5_16.4"),
    pytest.param(I.EPI_STORE, 14414, 1280, 256, id="23.3_28.9"), pytest.param(I.EPI_RESIDUAL, 23422, 512, 256, id="20.1_23.7"),
    pytest.param(I.EPI_RESIDUAL, 1620, 5120, 256, id="19.0_23.0"),
    pytest.param(I.EPI_ROPE, 38805, 512, 128, id="31.6_37.6"), pytest.param(I.EPI_SILU_MUL, 10405, 512, 128, id="9.8_12.1"),
    pytest.param(I.EPI_SILU_MUL, 2896, 2816, 128, id="16.5_19.0")])
def test_products_that_the_wide_tiles_finish_sooner_stay_with_them(epi, M, N, K):
    a = I.GemmArgs(A=A16, lda=K, B0=A16, ldb=K, C=A16, ldc=N, M=M, N=N, K=K, epi=epi, head_dim=128, rope=A16)
    if epi == I.EPI_SILU_MUL:
        a.B1 = A16
    assert I.small_supported(a)
    assert I.small_pick(a, 512 << 20) is None
