"""The phase timer counts what was launched, once, under the name of what the launch does."""
import pytest

from paper_2601_13155_amd import runtime, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def _phases(shape, N, skip, kv_mode=0):
    """{phase: launches} of one layer."""
    ctx = runtime.make_context(shape, N, 32, 16, shape.Dff)
    dw = runtime.upload_layer(synth.make_layer(3, 0, shape, 16), shape, 16)
    ctx.spts_profile_begin()
    runtime.run_layer(ctx, synth.hidden_states(3, N, shape.D, shape.dtype), synth.positions(N), dw, shape, skip=skip, probe_len=32,
                      m_attn=N // 2, m_ffn=N // 2, kv_mode=kv_mode)
    return {k: n for k, (_, n) in ctx.spts_profile_end().items()}


# products of one kernel: keys in one launch with the probe's queries and all values, or with a dense layer's values and queries
@pytest.mark.parametrize("skip,kv_mode,alone", [(1, 0, {"q_proj": 1, "v_proj": 1}), (1, 1, {"q_proj": 1}), (0, 0, {})],
                         ids=["active_pairs", "all_pairs", "dense"])
def test_shared_launch(torch, skip, kv_mode, alone):
    got = _phases(synth.TINY, 300, skip, kv_mode)
    assert {k: n for k, n in got.items() if k.endswith("_proj") or k == "probe_q"} == {"kqv_proj": 1, "o_proj": 1, **alone}


# 128 key columns, which the 256-wide tiles do not take, beside 512 query columns, which they do
@pytest.mark.parametrize("skip,kv_mode,alone", [(1, 0, {"probe_q": 1}), (1, 1, {"probe_q": 1}), (0, 0, {})], ids=["active_pairs", "all_pairs", "dense"])
def test_launches_of_their_own(torch, skip, kv_mode, alone):
    got = _phases(synth.ModelShape(D=256, H=4, Hkv=1, d=128, Dff=256, dtype="bf16"), 300, skip, kv_mode)
    assert {k: n for k, n in got.items() if k.endswith("_proj") or k == "probe_q"} == {"k_proj": 1, "q_proj": 1, "v_proj": 1, "o_proj": 1, **alone}
