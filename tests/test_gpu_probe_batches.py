"""The matrix-core probe over batches, at every chunk length and on both sides of the 32 chunks up to which its second pass combines the
statistics itself (the longest sequence decides): the bits of every sequence probed alone, which has chunks of its own length, and the scores
of the CPU oracle."""
import ctypes as C

import numpy as np
import pytest

from oracle import spts_oracle as orc
from paper_2601_13155_amd import binding, runtime, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def _chunk_keys(N, P, heads, Hkv):
    f = getattr(binding.load(), "_ZN4spts16probe_chunk_keysEliii")
    f.restype, f.argtypes = C.c_int, [C.c_int64, C.c_int, C.c_int, C.c_int]
    return f(N, P, heads, Hkv)


# kv heads, query heads, probe rows, lengths, keys a chunk, chunks of the longest sequence
CASES = [
    (2, 4, 40, (2049, 65, 300), 64, 33),
    (2, 4, 40, (333, 64, 700, 2048), 64, 32),
    (8, 16, 40, (127, 128, 129, 4000, 40), 128, 32),
    (8, 16, 40, (4097, 129, 255), 128, 33),
    (8, 16, 40, (255, 256, 257, 511, 8000), 256, 32),
    (8, 16, 40, (257, 8193, 511, 64), 256, 33),
    (1, 7, 80, (640, 1300, 81, 2500), 64, 40),       # 560 probe rows: two groups of them
    (1, 3, 96, (1025, 2049, 96), 64, 33),            # 288 probe rows: three blocks a wavefront
    (1, 1, 8, (16700, 12001, 11500), 128, 131),      # more groups of 256 keys than lanes
]


IDS = lambda v: "_".join(map(str, v)) if isinstance(v, tuple) else str(v)   # noqa: E731


class ProbeArgs(C.Structure):
    """spts::ProbeArgs of csrc/spts_internal.h, field by field."""
    _fields_ = [("qp", C.c_void_p), ("k", C.c_void_p), ("S", C.c_void_p), ("stats", C.c_void_p), ("partial", C.c_void_p), ("N", C.c_int64),
                ("P", C.c_int32), ("H", C.c_int32), ("Hkv", C.c_int32), ("d", C.c_int32), ("q_scale", C.c_float)]


class ProbeSegments(C.Structure):
    _fields_ = [("off", C.c_void_p), ("chunk", C.c_void_p), ("n", C.c_int32), ("chunks", C.c_int64), ("max_chunks", C.c_int64), ("chunk_keys", C.c_int32)]


def _fn(mangled, res, *args):
    f = getattr(binding.load(), mangled)
    f.restype, f.argtypes = res, args
    return f


def _probe(torch, q, k, heads, seg=None):
    """Scores of the keys k [N, Hkv, d] by the queries q [.., P, H, d], through the single or the batched launch."""
    (N, Hkv, d), P, stream = k.shape, q.shape[-3], torch.cuda.current_stream().cuda_stream
    S = torch.full((N + 64,), float("nan"), device="cuda")
    a = ProbeArgs(qp=q.data_ptr(), k=k.data_ptr(), S=S.data_ptr(), N=N, P=P, H=heads, Hkv=Hkv, d=d)
    pa, ps = C.POINTER(ProbeArgs), C.POINTER(ProbeSegments)
    floats = (_fn("_ZN4spts20probe_scratch_floatsEliii", C.c_size_t, C.c_int64, C.c_int, C.c_int, C.c_int)(N, P, heads, Hkv) if seg is None else
              _fn("_ZN4spts26probe_batch_scratch_floatsERKNS_9ProbeArgsERKNS_13ProbeSegmentsE", C.c_size_t, pa, ps)(a, seg))
    part = torch.full((floats + 64,), float("nan"), device="cuda")
    a.partial = part.data_ptr()
    if seg is None:
        assert _fn("_ZN4spts17launch_probe_mfmaERKNS_9ProbeArgsEP12ihipStream_t", C.c_int, pa, C.c_void_p)(a, stream) == 0
    else:
        assert _fn("_ZN4spts25launch_probe_mfma_batchedERKNS_9ProbeArgsERKNS_13ProbeSegmentsEP12ihipStream_t", C.c_int, pa, ps, C.c_void_p)(a, seg, stream) == 0
    torch.cuda.synchronize()
    assert torch.isnan(S[N:]).all() and torch.isnan(part[-64:]).all() and torch.isfinite(S[:N]).all()
    return S[:N]


@pytest.mark.parametrize("Hkv,heads,P,lens,keys,chunks", CASES, ids=IDS)
def test_a_batch_has_the_bits_of_its_sequences(torch, Hkv, heads, P, lens, keys, chunks):
    d, n, offs = 64 if heads != 7 else 128, len(lens), np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    N = int(offs[-1])
    assert _chunk_keys(N, P, heads, Hkv) == keys and -(-max(lens) // keys) == chunks
    g = torch.Generator(device="cuda").manual_seed(N)
    k = torch.randn((N, Hkv, d), generator=g, device="cuda").bfloat16()
    k[offs[1] // 2] *= 6.0                                       # a key that dominates some rows
    q = torch.randn((n, P, heads, d), generator=g, device="cuda").bfloat16()
    counts = np.concatenate([[0], np.cumsum([-(-m // keys) for m in lens])]).astype(np.int64)
    off, chunk = torch.from_numpy(offs).cuda(), torch.from_numpy(counts).cuda()
    S = _probe(torch, q, k, heads, ProbeSegments(off.data_ptr(), chunk.data_ptr(), n, int(counts[-1]), chunks, keys))
    for b, m in enumerate(lens):
        alone = _probe(torch, q[b].contiguous(), k[offs[b]:offs[b + 1]].contiguous(), heads)
        got = S[offs[b]:offs[b + 1]]
        assert bool((got == alone).all()), (m, float(((got - alone).abs() / alone).max()))


@pytest.mark.parametrize("Hkv,heads,P,lens,keys,chunks", CASES, ids=IDS)
def test_a_batched_layer_has_the_scores_of_the_oracle(torch, Hkv, heads, P, lens, keys, chunks):
    shape = synth.ModelShape(D=256, H=heads, Hkv=Hkv, d=64 if heads != 7 else 128, Dff=256, dtype="bf16")
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    N = int(offs[-1])
    w = synth.make_layer(7, 0, shape, 16)
    dw = runtime.upload_layer(w, shape, 16)
    xs = [synth.hidden_states(11 + b, n, shape.D, shape.dtype) for b, n in enumerate(lens)]
    ps = [(synth.positions(n) * 2 + b).astype(np.int32) for b, n in enumerate(lens)]
    ctx = runtime.make_context(shape, N, P, 16, shape.Dff)
    s = torch.zeros(N, device="cuda")
    ctx.spts_layer_prefill_batched(runtime.to_device(np.concatenate(xs), "bf16"), torch.from_numpy(np.concatenate(ps)).cuda(), offs, dw, P,
                                   [0] * len(lens), [0] * len(lens), 1, None, s)
    for b, n in enumerate(lens):
        got = s[offs[b]:offs[b + 1]].cpu().numpy()
        _, S = orc.probe_attn(xs[b], ps[b], w, H.oracle_model(shape), P, H.rnd_for("bf16"))
        assert H.score_rel_err(got, S) <= H.TOL["bf16"]["score"], n
        assert abs(float(got.astype(np.float64).sum()) - 1.0) < 1e-3
