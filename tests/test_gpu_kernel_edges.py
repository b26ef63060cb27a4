"""Kernels at the sizes where their tiles, groups and splits begin and end, against the CPU oracle (through the C ABI)."""
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


def _mk(shape, N, r, seed):
    return (synth.make_layer(seed, 0, shape, r), synth.hidden_states(seed, N, shape.D, shape.dtype),
            (synth.positions(N) * 2 + 1).astype(np.int32))


# ------------------------------------------------------------------------------------------ probe row groups
# more than 512 probe rows per kv head: 513..1024 rows are two row groups (525: the second nearly empty), 1040 are three
@pytest.mark.parametrize("H_,Hkv,d,P,N", [(7, 1, 128, 75, 600), (14, 2, 128, 128, 1111), (7, 1, 64, 74, 74), (16, 2, 64, 130, 513)],
                         ids=["525rows", "896rows", "518rows_all_probe", "1040rows"])
def test_probe_row_groups(torch, H_, Hkv, d, P, N):
    shape = synth.ModelShape(D=512, H=H_, Hkv=Hkv, d=d, Dff=256, dtype="bf16")
    w, x, pos = _mk(shape, N, 16, 7)
    ctx = runtime.make_context(shape, N, P, 16, shape.Dff)
    dw = runtime.upload_layer(w, shape, 16)
    kd = torch.zeros((N, Hkv, d), dtype=torch.bfloat16, device="cuda")
    sd = torch.zeros(N, dtype=torch.float32, device="cuda")
    ctx.spts_probe_attn(runtime.to_device(x, "bf16"), torch.from_numpy(pos).cuda(), N, dw, P, kd, sd)
    _, S = orc.probe_attn(x, pos, w, H.oracle_model(shape), P, H.rnd_for("bf16"))
    s = sd.cpu().numpy()
    assert H.score_rel_err(s, S) <= H.TOL["bf16"]["score"]
    assert abs(float(s.astype(np.float64).sum()) - 1.0) < 1e-3


# ------------------------------------------------------------------------------------------ greedy head
@pytest.mark.parametrize("V", [16, 1008, 1024 * 32, 1024 * 32 + 16, 128256])   # (batched calls take multiples of 16)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_argmax_picks_the_lowest_id_of_equal_logits(torch, dtype, V):
    """Logits are whole numbers here (one non-zero state element, integer table): ties are exact and lie in different shares of
    the row; a row of all-equal logits gives id 0."""
    D, nb = 64, 3
    shape = synth.ModelShape(D=D, H=1, Hkv=1, d=64, Dff=64, dtype=dtype, rms_eps=0.0)
    ctx = runtime.make_context(shape, 16, 1, 1, 64)
    rng = np.random.default_rng(V)
    table = np.zeros((V, D), dtype=np.float32)
    table[:, :2] = rng.integers(-3, 3, (V, 2))
    best = sorted(rng.integers(0, V, 5).tolist())
    table[best, 0] = 4.0                      # row 0 of the batch: tie between these ids
    table[V - 1, 1] = 5.0                     # row 1: the very last id
    x = np.zeros((nb, D), dtype=np.float32)
    x[0, 0] = x[1, 1] = x[2, 5] = 1.0         # rows 2: every logit is zero
    td = runtime.to_device(table, dtype)
    xd, gd = runtime.to_device(x, dtype), runtime.to_device(np.ones(D, dtype=np.float32), dtype)
    tok = torch.full((nb,), -1, dtype=torch.int32, device="cuda")
    logits = torch.zeros((nb, V), dtype=torch.float32, device="cuda")
    nxt = torch.zeros_like(xd)
    ctx.spts_greedy_token_batched(xd, gd, td, V, nb, tok, logits, nxt)
    assert tok.cpu().tolist() == [best[0], V - 1, 0]
    assert torch.equal(nxt, td[tok.long()])
    one = torch.full((4,), -1, dtype=torch.int32, device="cuda")
    ctx.spts_greedy_token(xd[0], gd, td, V, one, logits[0], None)
    assert int(one[0]) == best[0]
