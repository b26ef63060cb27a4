"""Decode attention over several sequences of very different lengths, with as little scratch as it accepts and with plenty, against 64 bits."""
import ctypes as C

import pytest

from paper_2601_13155_amd import binding

pytestmark = pytest.mark.gpu


class DecodeBatch(C.Structure):
    """spts::DecodeBatch of csrc/spts_internal.h."""
    _fields_ = [("k", C.c_void_p * 16), ("v", C.c_void_p * 16), ("cache_pos", C.c_void_p * 16), ("count", C.c_int64 * 16), ("pos", C.c_int32 * 16), ("n", C.c_int32)]


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available()
    return torch


@pytest.mark.parametrize("pairs", [(1,), (1, 2), (1, 20000), (63, 64, 65, 66), (5000, 300, 17), (129,) * 16, (9000,) + (1,) * 14 + (3000,)], ids=lambda p: f"{len(p)}_{max(p)}")
@pytest.mark.parametrize("H,Hkv,d,dtype", [(8, 8, 64, "bf16"), (8, 2, 128, "bf16"), (7, 1, 128, "bf16"), (4, 2, 16, "f32")])
def test_ragged_lengths(torch, pairs, H, Hkv, d, dtype):
    t, n, stream = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype], len(pairs), torch.cuda.current_stream().cuda_stream
    f = getattr(binding.load(), "_ZN4spts26launch_decode_attn_batchedEPKvRKNS_11DecodeBatchEiiiPfmPvbP12ihipStream_t")
    f.restype, f.argtypes = C.c_int, [C.c_void_p, C.POINTER(DecodeBatch), C.c_int, C.c_int, C.c_int, C.c_void_p, C.c_size_t, C.c_void_p, C.c_bool, C.c_void_p]
    g = torch.Generator(device="cuda").manual_seed(sum(pairs))
    q = torch.randn((n, H, d), generator=g, device="cuda").to(t)
    kv = [[torch.randn((m, Hkv, d), generator=g, device="cuda").to(t) for _ in range(2)] for m in pairs]
    db = DecodeBatch(n=n)
    for b, (k, v) in enumerate(kv):
        db.k[b], db.v[b], db.count[b] = k.data_ptr(), v.data_ptr(), pairs[b] - 1
    least = n * Hkv * 8 * (d + 2)
    for floats in (least, least + Hkv * 8 * (d + 2) * 512):
        part = torch.full((floats + 64,), float("nan"), device="cuda")
        out = torch.full((n + 1, H, d), float("nan"), dtype=t, device="cuda")
        assert f(q.data_ptr(), db, H, Hkv, d, part.data_ptr(), floats, out.data_ptr(), dtype == "bf16", stream) == 0
        torch.cuda.synchronize()
        assert torch.isnan(part[-64:]).all() and torch.isnan(out[n]).all()
        for b, (k, v) in enumerate(kv):
            k, v = (x.double().repeat_interleave(H // Hkv, 1) for x in (k, v))
            w = torch.softmax((q[b].double()[None] * k).sum(-1) / d ** 0.5, 0)
            want = (w[..., None] * v).sum(0)
            # fp32 logits (128 products of about one: within 2^-14), probabilities and sums of at most 20000 of them; one rounding of the result
            slack = 2.0 ** -12 * float(v.abs().max()) + (2.0 ** -8 if dtype == "bf16" else 0.0) * want.abs()
            assert bool(((out[b].double() - want).abs() <= slack).all())
