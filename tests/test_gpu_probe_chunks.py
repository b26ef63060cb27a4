"""The matrix-core probe at every chunk length, with the statistics combined inside its second pass (up to 32 chunks) and before it, against
the CPU oracle."""
import numpy as np
import pytest

from oracle import spts_oracle as orc
from paper_2601_13155_amd import runtime, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available()
    return torch


# 64 keys a chunk: one chunk, one key more, 32 and 33 chunks; 128 keys: 32 and 33 chunks; 256 keys: 32 and 33 chunks
@pytest.mark.parametrize("Hkv,N", [(2, 64), (2, 65), (2, 2048), (2, 2049), (8, 4096), (8, 4097), (8, 8192), (8, 8193)])
def test_chunk_lengths(torch, Hkv, N):
    P, limit = 40, 9000
    shape = synth.ModelShape(D=256, H=2 * Hkv, Hkv=Hkv, d=64, Dff=256, dtype="bf16")
    w, x = synth.make_layer(7, 0, shape, 16), synth.hidden_states(N, N, shape.D, shape.dtype)
    pos = (synth.positions(N) * 2 + 1).astype(np.int32)
    for most in (N, limit):   # scratch sized for this call alone, and for longer ones
        ctx = runtime.make_context(shape, most, P, 16, shape.Dff)
        dw = runtime.upload_layer(w, shape, 16)
        kd = torch.zeros((N, Hkv, shape.d), dtype=torch.bfloat16, device="cuda")
        sd = torch.zeros(N, dtype=torch.float32, device="cuda")
        ctx.spts_probe_attn(runtime.to_device(x, "bf16"), torch.from_numpy(pos).cuda(), N, dw, P, kd, sd)
        _, S = orc.probe_attn(x, pos, w, H.oracle_model(shape), P, H.rnd_for("bf16"))
        s = sd.cpu().numpy()
        assert H.score_rel_err(s, S) <= H.TOL["bf16"]["score"]
        assert abs(float(s.astype(np.float64).sum()) - 1.0) < 1e-3
