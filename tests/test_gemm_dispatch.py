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
