"""The rotary table that the first RMSNorm's launch makes: against 64-bit values, and against the row that a decode step makes for the same
position, for every base that a context takes (a base below 1 turns positions into angles that fp64 cannot hold to a radian)."""
import ctypes as C

import numpy as np
import pytest

from paper_2601_13155_amd import binding

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


def _table(torch, pos, d, base, D=8, fill=1.0):
    """(table [N, d/2, 2], the copy of pos, the normalised rows of `fill`)."""
    N, vp = len(pos), C.c_void_p
    x, gamma = torch.full((N, D), fill, device="cuda"), torch.ones(D, device="cuda")
    out, table, copy = torch.zeros_like(x), torch.zeros((N, d // 2, 2), device="cuda"), torch.full_like(pos, -1)
    f = _fn("_ZN4spts19launch_rmsnorm_ropeEPKvS1_fPvliPKiifP15HIP_vector_typeIfLj2EEPibP12ihipStream_t",
            vp, vp, C.c_float, vp, C.c_int64, C.c_int, vp, C.c_int, C.c_float, vp, vp, C.c_bool, vp)
    stream = torch.cuda.current_stream().cuda_stream
    assert f(x.data_ptr(), gamma.data_ptr(), 0.0, out.data_ptr(), N, D, pos.data_ptr(), d, base, table.data_ptr(), copy.data_ptr(), False, stream) == 0
    torch.cuda.synchronize()
    return table, copy, out


POS = np.array([0, 1, 2, 31, 4095, 131071, 10 ** 6, 2 ** 24 + 1, 2 ** 31 - 1, -1, -77777, -2 ** 31] + list(range(1000, 1023)), np.int32)


@pytest.mark.parametrize("base", [1e6, 500000.0, 10000.0, 1.0, 0.5, 2.0 ** -19, 2.0 ** -20, 1e-7, 1e-12, 1e-30])
@pytest.mark.parametrize("d", [2, 64, 88, 256])
def test_rows_are_rotations_and_those_of_a_decode_step(torch, d, base):
    table, copy, out = _table(torch, torch.from_numpy(POS).cuda(), d, base)
    assert np.array_equal(copy.cpu().numpy(), POS) and bool((out - 1.0).abs().max() <= 2.0 ** -20)
    t = table.double()
    # (cos, sin) rounded to fp32 each: the squares sum to 1 within 4 * 2^-24
    assert bool(((t ** 2).sum(-1) - 1.0).abs().max() <= 2.0 ** -22)
    row = torch.zeros((d // 2, 2), device="cuda")
    f = _fn("_ZN4spts22launch_decode_rope_rowEiifP15HIP_vector_typeIfLj2EEP12ihipStream_t", C.c_int, C.c_int, C.c_float, C.c_void_p, C.c_void_p)
    for i, p in enumerate(POS):
        assert f(int(p), d, base, row.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
        # the same fp64 angle, its cosine and sine rounded to fp32: the same value, or its neighbour in a halfway case
        assert bool((row - table[i]).abs().max() <= 2.0 ** -24), (int(p), base)
    # against 64 bits: a frequency and an angle rounded to fp64 (a few 2^-53 of the angle each), the result to fp32
    j = np.arange(d // 2)
    ang = POS[:, None].astype(np.float64) * np.exp2(j * (-2.0 / d * np.log2(np.float64(np.float32(base)))))
    known = np.abs(ang) < 2.0 ** 40
    want = np.stack([np.cos(ang), np.sin(ang)], -1)
    bound = 2.0 ** -25 + 2.0 ** -48 * np.abs(ang)[..., None]
    assert (np.abs(t.cpu().numpy() - want) <= bound)[known].all()


def test_more_rows_than_a_launch_has_threads_for(torch):
    """15.8 million rows: with a workgroup of 256 threads a row and one of the table behind every 16, more than 2^32 threads."""
    N, d = 15_800_000, 2
    pos = torch.arange(N, dtype=torch.int32, device="cuda")
    table, copy, out = _table(torch, pos, d, 10000.0, D=4)
    assert torch.equal(copy, pos) and bool((out - 1.0).abs().max() <= 2.0 ** -20)
    want = torch.stack([torch.cos(pos.double()), torch.sin(pos.double())], -1)[:, None]
    assert bool((table.double() - want).abs().max() <= 2.0 ** -24)
