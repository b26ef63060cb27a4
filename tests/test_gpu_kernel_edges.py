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


# ------------------------------------------------------------------------------------------ fp32 / odd-dimension layer
# head dimensions at and between the kernels' 32 / 64 / 128 / 256 (30: rows that are not whole 16-byte pieces), row lengths
# that are not whole chunks (D = 62: the element-wise GEMM), sequence lengths around the 32-row tiles and the 8 (4) x 32 keys that
# a workgroup's wavefronts take per round.  Tolerance: helpers.TOL (fp32 1e-4, derived there from K = 4096; K <= 256 here).
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D,H_,Hkv,d,Dff", [(64, 4, 2, 16, 96), (62, 3, 1, 30, 70), (96, 2, 2, 96, 100), (256, 2, 1, 128, 130), (80, 2, 1, 256, 44)],
                         ids=["d16", "d30", "d96", "d128", "d256"])
def test_layer_of_any_head_dimension(torch, dtype, D, H_, Hkv, d, Dff):
    shape = synth.ModelShape(D=D, H=H_, Hkv=Hkv, d=d, Dff=Dff, dtype=dtype)
    mdl, r = H.oracle_model(shape), 8
    ctx = runtime.make_context(shape, 300, 40, r, Dff)
    w = synth.make_layer(51, 0, shape, r)
    dw = runtime.upload_layer(w, shape, r)
    for N in (1, 31, 33, 129, 257, 300):
        x = synth.hidden_states(51 + N, N, D, dtype)
        pos = (synth.positions(N) * 3 + 5).astype(np.int32)
        P = min(37, N)
        dense = runtime.run_layer(ctx, x, pos, dw, shape, skip=0, probe_len=P, m_attn=0, m_ffn=0)
        H.lockstep_layer(dense, x, pos, w, mdl, orc.LayerCfg(0, P, N, N, 1, 0), dtype)
        for kv_mode, ma in ((0, max(1, (2 * N) // 3)), (1, max(1, N // 3))):
            mf = max(1, N // 2)
            skip = runtime.run_layer(ctx, x, pos, dw, shape, skip=1, probe_len=P, m_attn=ma, m_ffn=mf, kv_mode=kv_mode)
            H.lockstep_layer(skip, x, pos, w, mdl, orc.LayerCfg(1, P, ma, mf, 1, kv_mode), dtype)


# ------------------------------------------------------------------------------------------ short products
# row counts around one and two of the short-product GEMM's tiles, through the layer, with and without slab-major weights.  Products
# this small all take 64-row tiles, and only down and z are split; every tile height, split and epilogue is in
# test_gpu_short_products.py
@pytest.mark.parametrize("pack", [True, False], ids=["packed", "row_major"])
@pytest.mark.parametrize("H_,Hkv,d", [(8, 2, 128), (8, 4, 64)], ids=["d128", "d64"])
def test_layer_with_short_products(torch, H_, Hkv, d, pack):
    shape = synth.ModelShape(D=1024, H=H_, Hkv=Hkv, d=d, Dff=2048, dtype="bf16", rope_base=500000.0)
    mdl, r = H.oracle_model(shape), 256
    ctx = runtime.make_context(shape, 400, 40, r, shape.Dff)
    assert ctx.uses_mfma()
    w = synth.make_layer(61, 0, shape, r)
    dw = runtime.upload_layer(w, shape, r, pack=pack)
    for N in (63, 65, 128, 191, 193, 321, 385):
        x = synth.hidden_states(61 + N, N, shape.D, "bf16")
        pos = (synth.positions(N) * 3 + 5).astype(np.int32)
        dense = runtime.run_layer(ctx, x, pos, dw, shape, skip=0, probe_len=8, m_attn=0, m_ffn=0)
        H.lockstep_layer(dense, x, pos, w, mdl, orc.LayerCfg(0, 8, N, N, 1, 0), "bf16")
        for kv_mode, ma, mf in ((0, max(1, (2 * N) // 3), N // 2), (1, N // 3, N - 1)):
            skip = runtime.run_layer(ctx, x, pos, dw, shape, skip=1, probe_len=37, m_attn=ma, m_ffn=mf, kv_mode=kv_mode)
            H.lockstep_layer(skip, x, pos, w, mdl, orc.LayerCfg(1, 37, ma, mf, 1, kv_mode), "bf16")


# ------------------------------------------------------------------------------------------ batches in one launch per step
@pytest.mark.parametrize("name,shape,P", [
    ("d128_g4", synth.ModelShape(D=512, H=8, Hkv=2, d=128, Dff=1024, dtype="bf16", rope_base=500000.0), 8),
    ("d64_g2_p1", synth.ModelShape(D=512, H=8, Hkv=4, d=64, Dff=1024, dtype="bf16"), 1),
    ("d128_g7", synth.ModelShape(D=512, H=7, Hkv=1, d=128, Dff=1024, dtype="bf16"), 80),
], ids=lambda v: v if isinstance(v, str) else None)
def test_batch_with_sequences_around_chunks_and_tiles(torch, name, shape, P):
    """50 sequences (more than one launch of the cache fill takes) whose lengths and budgets lie around the probe's 64-key tiles (and
    chunks, which so few candidates leave at 64 keys; longer ones: test_gpu_probe_batches.py) and the attention's 64-key / 64 .. 256-query tiles, budgets of zero among them; skip and dense branch, every sequence
    lock-step against the oracle, caches included."""
    r, mdl = 64, H.oracle_model(shape)
    rng = np.random.default_rng(3)
    lens = [P, P + 1, 256, 257, 511] + [int(v) for v in rng.integers(P, 300, 45)]
    w = synth.make_layer(71, 0, shape, r)
    dw = runtime.upload_layer(w, shape, r)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ctx = runtime.make_context(shape, int(offs[-1]), P, r, shape.Dff)
    xs = [synth.hidden_states(200 + b, n, shape.D, "bf16") for b, n in enumerate(lens)]
    ps = [(synth.positions(n) * 2 + b).astype(np.int32) for b, n in enumerate(lens)]
    ma = [min(n, (63, 64, 65, 0, 256, 1)[b % 6]) for b, n in enumerate(lens)]
    mf = [max(1, n // 2) for n in lens]
    for skip in (1, 0):
        a_n = ma if skip else lens
        f_n = mf if skip else lens
        xd = runtime.to_device(np.concatenate(xs), "bf16")
        s = torch.zeros(int(offs[-1]), dtype=torch.float32, device="cuda")
        ia = torch.full((sum(a_n) + 1,), -1, dtype=torch.int32, device="cuda")
        iff = torch.full((sum(f_n) + 1,), -1, dtype=torch.int32, device="cuda")
        caches = [runtime.KVCache(shape, n) for n in a_n]
        kvs = [c.struct for c in caches]
        ctx.spts_layer_prefill_batched(xd, torch.from_numpy(np.concatenate(ps)).cuda(), offs, dw, P, ma, mf, 1, kvs, s, ia, iff, skip=skip)
        x_out, s_out, ia, iff = runtime.to_host(xd).astype(np.float64), s.cpu().numpy(), ia.cpu().numpy(), iff.cpu().numpy()
        oa = of = 0
        for b, n in enumerate(lens):
            r0 = int(offs[b])
            gpu = dict(x=x_out[r0:r0 + n], s_mha=s_out[r0:r0 + n], idx_attn=ia[oa:oa + a_n[b]] - r0, idx_ffn=iff[of:of + f_n[b]] - r0)
            cfg = orc.LayerCfg(skip, P, a_n[b], f_n[b], 1, 0)
            ref = H.lockstep_layer(gpu, xs[b], ps[b], w, mdl, cfg, "bf16")["ref"]
            assert kvs[b].count == a_n[b]
            if a_n[b]:
                k, v, p = caches[b].host()
                assert np.array_equal(p, ps[b][gpu["idx_attn"]] if skip else ps[b])
                assert H.row_rel_err(k.reshape(a_n[b], -1), ref.k_cache.reshape(a_n[b], -1)) <= H.TOL["bf16"]["hidden"]
                assert H.row_rel_err(v.reshape(a_n[b], -1), ref.v_cache.reshape(a_n[b], -1)) <= H.TOL["bf16"]["hidden"]
            oa += a_n[b]
            of += f_n[b]


# ------------------------------------------------------------------------------------------ channel scores
# calibration lengths around the wavefront kernel's 64 x 8 .. 64 x 128 (fp32: 64 x 64) registers and the GEMM's 256-row tiles
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [1, 63, 255, 257, 512, 513, 1025, 2047, 2049, 4096, 4097, 8192, 8200])
def test_channel_importance_lengths(torch, dtype, T):
    shape = synth.ModelShape(D=64, H=1, Hkv=1, d=64, Dff=128, dtype=dtype)
    w = synth.layer_weights(81, 0, shape)
    dw = runtime.upload_layer(w, shape, 0, pack=False)
    ctx = runtime.make_context(shape, T, 1, 1, shape.Dff)
    x = synth.calibration_states(81, T, shape.D, dtype)
    xd = runtime.to_device(x, dtype)
    for k in sorted({1, max(1, T // 5), T}):
        imp = torch.full((shape.Dff,), -1.0, dtype=torch.float32, device="cuda")
        ctx.spts_channel_importance(xd, T, dw, k, imp)
        ref = orc.channel_importance(x, w["Wgate"], w["Wup"], k, H.rnd_for(dtype))
        assert np.max(np.abs(imp.cpu().numpy() - ref)) <= H.TOL[dtype]["score"] * np.max(np.abs(ref)), k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [1, 5, 64, 511, 513, 1500, 2048, 4096])
def test_topk_mean_of_any_values(torch, dtype, n):
    """Rows whose quantiles a sample of them tells well, badly and not at all: smooth, few values, steps, many octaves, ascending, all zero, infinite."""
    from tests import internal as I
    rng = np.random.default_rng(n)
    z = rng.standard_normal(n)
    rows = [z, np.abs(z) ** 8, np.zeros(n), np.full(n, -0.75), np.where(rng.random(n) < 0.3, 2.0, -1.0), np.sort(z), -np.sort(-np.abs(z)), np.exp(20 * z),
            np.where(np.arange(n) % 64 == 5, 9.0, 1e-3 * z), np.where(np.arange(n) < n // 2, 0.0, z), np.round(3 * z), np.where(rng.random(n) < 0.01, np.inf, z)]
    v = torch.from_numpy(np.stack(rows).astype(np.float32)).cuda().to(torch.bfloat16 if dtype == "bf16" else torch.float32).contiguous()
    host = np.sort(np.abs(v.float().cpu().numpy().astype(np.float64)), axis=1)[:, ::-1]
    for k in sorted({1, 2, max(1, n // 50), max(1, n // 5), max(1, n // 2), max(1, n - 1), n} & set(range(1, n + 1))):
        out = torch.full((len(rows),), -1.0, dtype=torch.float32, device="cuda")
        assert I.topk_mean(v.data_ptr(), n, len(rows), n, k, out.data_ptr(), dtype == "bf16", torch.cuda.current_stream().cuda_stream) == 0
        ref = host[:, :k].mean(1)
        # a sum of k fp32 terms of one sign in any order, a product and a quotient
        assert np.allclose(out.cpu().numpy(), ref, rtol=(k + 4) * 2.0 ** -24, atol=0), k


def _topk_mean(torch, v, k, out):
    from tests import internal as I
    assert I.topk_mean(v.data_ptr(), v.shape[1], v.shape[0], v.shape[1], k, out.data_ptr(), v.dtype == torch.bfloat16, torch.cuda.current_stream().cuda_stream) == 0


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [64, 512, 513, 1024, 1025, 2048, 3000, 4096])
def test_topk_mean_of_few_values(torch, dtype, n):
    """Rows whose threshold lies among many equal or nearly equal values: one value, two, steps, values a few units of the last place apart, a tie below
    smooth values, a tie that the sample misses (every 64th value is another)."""
    rng = np.random.default_rng(100 + n)
    z = rng.standard_normal(n)
    u = rng.random(n)
    rows = [np.full(n, -0.3), np.full(n, 1e-30), np.where(u < 0.19, 2.0, 1.0), np.where(u < 0.5, 1.0 + 1e-6 * z, 1e-20), np.round(2 * z), 0.3 * np.round(2 * z),
            np.where(u < 0.15, 1.0 + np.abs(z), 0.7), np.where(u < 0.25, 1.0 + np.abs(z), 0.7), np.where(u < 0.6, 0.7, 0.7 * (1 - 1e-3 * u)), np.where(np.arange(n) % 64 < 13, 5.0, 4.0),
            np.where(u < 0.5, np.inf, 1.0), np.where(u < 0.3, 1e38, 1e-38 * u)]
    v = torch.from_numpy(np.stack(rows).astype(np.float32)).cuda().to(torch.bfloat16 if dtype == "bf16" else torch.float32).contiguous()
    host = np.sort(np.abs(v.float().cpu().numpy().astype(np.float64)), axis=1)[:, ::-1]
    for k in sorted({1, max(1, n // 50), n // 5, n // 3, n // 2, n - 1, n}):
        out = torch.full((len(rows),), -1.0, dtype=torch.float32, device="cuda")
        _topk_mean(torch, v, k, out)
        ref = host[:, :k].mean(1)
        # a sum of k fp32 terms of one sign in any order, a product and a quotient; sums beyond the largest fp32 number are infinite
        got = out.cpu().numpy().astype(np.float64)
        over = host[:, :k].sum(1) > 3.4e38
        assert np.allclose(got[~over], ref[~over], rtol=(k + 4) * 2.0 ** -24, atol=1e-45) and np.isinf(got[over]).all(), k


@pytest.mark.parametrize("n", [1000, 2048])
def test_topk_mean_of_equal_values_takes_little_longer(torch, n):
    """The search for the threshold of 14336 rows closes in on it from both sides; of equal fp32 values it does not go through all bits below the first that
    the sample tells (then 1.9 and 2 times the time of smooth rows, now 1.4 and 1.5)."""
    out = torch.empty(14336, device="cuda")
    smooth = torch.randn((14336, n), device="cuda") * torch.randn((14336, n), device="cuda")
    same = torch.full((14336, n), 0.25, device="cuda")
    times = [_best_us(torch, lambda v=v: _topk_mean(torch, v, n // 5, out)) for v in (smooth, same)]
    assert times[1] <= 1.7 * times[0], times


# ------------------------------------------------------------------------------------------ TopK of long rows of a batch
@pytest.mark.parametrize("n", [32772, 65536, 100004, 131068, 131072, 131076])
def test_long_row_topk_patterns(torch, n):
    """Rows that the one-sweep kernel takes by its bracket (smooth, sorted, periodic), and rows that make the bracket miss or overflow
    (equal scores, two values, a step at one place, values that the sample's positions never see); lengths around a wavefront's
    slices and the kernel's longest row (one length beyond it)."""
    rng = np.random.default_rng(n)
    base = np.exp(0.5 * rng.standard_normal(n)).astype(np.float32) / n
    unseen = base.copy()
    quads = n // 4
    seen = np.zeros(quads, bool)
    seen[(np.arange(2048, dtype=np.int64) * quads) // 2048] = True
    unseen[np.repeat(~seen, 4)[: n]] *= 7.0                       # the sample sees only the small ones
    step = base.copy(); step[: n // 3] += 1.0
    rows = {"smooth": base, "ascending": np.sort(base), "descending": np.sort(base)[::-1].copy(), "equal": np.full(n, 0.25, np.float32),
            "two_values": np.where(np.arange(n) % 3 == 0, 0.5, 0.125).astype(np.float32), "step": step, "unseen": unseen,
            "signed": rng.standard_normal(n).astype(np.float32), "octaves": np.exp(20 * rng.standard_normal(n)).astype(np.float32),
            "zeros": np.where(rng.random(n) < 0.9, -0.0, base).astype(np.float32)}
    s = np.stack(list(rows.values()))
    sd = torch.from_numpy(s).cuda()
    ctx = runtime.make_context(synth.TINY, n, 1, 1, synth.TINY.Dff)
    for k in (1, 2, 700, int(0.4 * n), n - 3, n):
        for protect in (0, 1):
            out = torch.full((len(rows), k), -7, dtype=torch.int32, device="cuda")
            ctx.spts_select_topk_batched(sd, n, k, protect, len(rows), out)
            got = out.cpu().numpy()
            for b, name in enumerate(rows):
                assert np.array_equal(got[b], orc.topk_select(s[b], k, protect)), (name, k, protect)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 333, 511, 512, 513, 1023, 1024, 1025])
def test_short_row_topk(torch, n):
    """Rows of up to a thousand scores, down to one."""
    rng = np.random.default_rng(n)
    rows = np.stack([np.exp(rng.standard_normal(n)), rng.standard_normal(n), np.full(n, 0.25), np.round(2 * rng.standard_normal(n)),
                     np.where(rng.random(n) < 0.5, -0.0, 0.0), np.full(n, -np.inf)]).astype(np.float32)
    sd = torch.from_numpy(rows).cuda()
    ctx = runtime.make_context(synth.TINY, n, 1, 1, synth.TINY.Dff)
    for k in sorted({1, max(1, n // 3), max(1, n - 1), n}):
        for protect in (0, 1):
            out = torch.full((len(rows) * k + 1,), -7, dtype=torch.int32, device="cuda")
            ctx.spts_select_topk_batched(sd, n, k, protect, len(rows), out)
            got = out.cpu().numpy()
            assert got[-1] == -7
            for b in range(len(rows)):
                assert np.array_equal(got[b * k:(b + 1) * k], orc.topk_select(rows[b], k, protect)), (b, k, protect)


@pytest.mark.parametrize("n", [32769, 32770, 32771, 65537, 98305, 100003, 131069, 131071, 131073, 262147])
def test_long_row_topk_of_rows_at_odd_addresses(torch, n):
    """Lengths that are no multiple of 4: rows at any 4-byte address, a last piece of one to three scores, one that begins a wavefront's slice;
    with the row's end among the largest, the smallest (minus infinity, so that padding ties with it) and the equal scores."""
    rng = np.random.default_rng(n)
    base = np.exp(0.5 * rng.standard_normal(n)).astype(np.float32) / n
    end = base.copy(); end[-3:] = (5.0, 4.0, 6.0)
    low = base.copy(); low[-5:] = -np.inf; low[rng.random(n) < 0.3] = -np.inf
    rows = np.stack([base, end, low, np.full(n, 0.25), np.full(n, -np.inf), np.sort(base), np.round(2 * rng.standard_normal(n)), rng.standard_normal(n)]).astype(np.float32)
    sd = torch.from_numpy(rows).cuda()
    ctx = runtime.make_context(synth.TINY, n, 1, 1, synth.TINY.Dff)
    for k in (1, n // 100, int(0.4 * n), n - n // 20, n - 1, n):
        for protect in (0, 1):
            out = torch.full((len(rows) * k + 1,), -7, dtype=torch.int32, device="cuda")
            ctx.spts_select_topk_batched(sd, n, k, protect, len(rows), out)
            got = out.cpu().numpy()
            assert got[-1] == -7
            for b in range(len(rows)):
                assert np.array_equal(got[b * k:(b + 1) * k], orc.topk_select(rows[b], k, protect)), (b, k, protect)


@pytest.mark.parametrize("n", [32769, 65538, 131071, 131073])
def test_long_row_topk_padding_is_below_every_score(torch, n):
    """Lengths that are no multiple of 4 with NaNs of either sign (a set sign bit comes below minus infinity), and with as many infinite scores as
    put the threshold's bracket across them and the finite ones: the places that fill the last piece up are never selected."""
    rng = np.random.default_rng(n)
    base = np.exp(0.5 * rng.standard_normal(n)).astype(np.float32) / n
    negative = np.array([0xFFC00000, 0xFF800001, 0xFFFFFFFF], dtype=np.uint32).view(np.float32)
    some = base.copy(); some[rng.random(n) < 0.3] = negative[0]; some[-1] = 1.0
    most = np.where(rng.random(n) < 0.98, rng.choice(negative, n), base); most[-2:] = (negative[1], 2.0)
    positive = base.copy(); positive[rng.random(n) < 0.1] = np.nan
    low = base.copy(); low[rng.random(n) < 0.3] = -np.inf; low[-1] = 1.0
    rows = np.stack([some, most, np.full(n, negative[0]), np.full(n, negative[2]), positive, low]).astype(np.float32)
    sd = torch.from_numpy(rows.view(np.int32)).cuda().view(torch.float32)
    ctx = runtime.make_context(synth.TINY, n, 1, 1, synth.TINY.Dff)
    for k in (1, n // 50, int(0.7 * n), n - n // 50, n - 1, n):
        for protect in (0, 1):
            out = torch.full((len(rows) * k + 4,), -7, dtype=torch.int32, device="cuda")
            ctx.spts_select_topk_batched(sd, n, k, protect, len(rows), out)
            got = out.cpu().numpy()
            assert (got[-4:] == -7).all()
            for b in range(len(rows)):
                bits = rows[b].view(np.uint32)
                bits = np.where(np.isnan(rows[b]), bits | np.uint32(0x400000), bits)   # quiet NaNs, as the sum with +0 leaves them
                key = np.where(bits >> 31, ~bits, bits | np.uint32(0x80000000)).astype(np.int64)
                if protect:
                    key[-1] = 0xFFFFFFFF
                ref = np.sort(np.argsort(-key, kind="stable")[:k])
                assert np.array_equal(got[b * k:(b + 1) * k], ref), (b, k, protect)


@pytest.mark.parametrize("n", [256, 257, 512, 513, 1024, 1025, 2048, 2049, 3072, 3073, 4096, 4097, 6144, 6145, 8192, 8193, 12288, 12289, 16384, 16385, 20480, 20481, 24576, 24577,
                               32767, 32768])
def test_register_topk_edges(torch, n):
    """The largest and smallest rows of every workgroup size of the register-resident kernel: thresholds among more than 64 neighbouring
    keys, among equal ones at the ends and in the middle of the range, and scores of both signs, the largest and minus infinity."""
    rng = np.random.default_rng(n)
    z = rng.standard_normal(n).astype(np.float32)
    near = (np.float32(0.5).view(np.int32) + rng.integers(0, max(2, n // 3), n).astype(np.int32)).view(np.float32)
    inf = z.copy(); inf[rng.random(n) < 0.3] = 3e38; inf[rng.random(n) < 0.3] = -np.inf
    rows = np.stack([z, near, inf, np.where(z > 0, 1.0, -1.0), np.where(np.arange(n) == n // 2, 3.0, 0.0), np.exp(15 * z), np.sort(z)]).astype(np.float32)
    sd = torch.from_numpy(rows).cuda()
    ctx = runtime.make_context(synth.TINY, n, 1, 1, synth.TINY.Dff)
    for k in sorted({1, 2, n // 7, n // 2, n - 1, n}):
        for protect in (0, 1):
            out = torch.full((len(rows) * k + 1,), -7, dtype=torch.int32, device="cuda")
            ctx.spts_select_topk_batched(sd, n, k, protect, len(rows), out)
            got = out.cpu().numpy()
            assert got[-1] == -7
            for b in range(len(rows)):
                assert np.array_equal(got[b * k:(b + 1) * k], orc.topk_select(rows[b], k, protect)), (b, k, protect)


@pytest.mark.parametrize("n", [2, 64, 300, 512, 1000, 2049, 6144, 20001, 32768])
def test_register_topk_orders_the_smallest_keys(torch, n):
    """NaNs with the sign bit and all or nearly all other bits set have the keys 0, 1 and 2, the same as empty slots or next to them: they are
    told apart, and an empty slot is never selected.  Whole rows of them, a few and many among scores, equal rows and segments of all lengths."""
    rng = np.random.default_rng(n)
    nans = np.array([0xFFFFFFFF, 0xFFFFFFFE, 0xFFFFFFFD], dtype=np.uint32)
    z = rng.standard_normal(n).astype(np.float32).view(np.uint32)
    low = np.where(rng.random(n) < 0.5, nans[0], nans[1])
    few = z.copy(); few[rng.permutation(n)[:min(n, 40)]] = rng.choice(nans, min(n, 40))
    rows = np.stack([low, low[::-1], np.full(n, nans[0]), rng.choice(nans, n), few, np.where(rng.random(n) < 0.7, rng.choice(nans, n), z),
                     np.where(np.arange(n) % 7 == 3, nans[1], nans[0])]).astype(np.uint32)
    keys = np.where(rows >> 31, ~rows, rows | np.uint32(0x80000000)).astype(np.int64)

    def expected(key, k, protect):
        key = key.copy()
        if protect:
            key[-1] = 0xFFFFFFFF
        return np.sort(np.argsort(-key, kind="stable")[:k])

    sd = torch.from_numpy(rows.view(np.int32)).cuda().view(torch.float32)
    ctx = runtime.make_context(synth.TINY, len(rows) * n, 1, 1, synth.TINY.Dff)
    for k in sorted({1, 2, max(1, n // 3), n - n // 5, n - 1, n} & set(range(1, n + 1))):
        for protect in (0, 1):
            out = torch.full((len(rows) * k + 4,), -7, dtype=torch.int32, device="cuda")
            ctx.spts_select_topk_batched(sd, n, k, protect, len(rows), out)
            got = out.cpu().numpy()
            assert (got[-4:] == -7).all()
            for b in range(len(rows)):
                assert np.array_equal(got[b * k:(b + 1) * k], expected(keys[b], k, protect)), (b, k, protect)
    lens = [n, 1, n - n // 3, n // 2 + 1, min(n, 65), min(n, 3), n - 1 or 1]   # segment b: a beginning of row b
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    flat = np.concatenate([rows[b, :m] for b, m in enumerate(lens)])
    for part in (0.3, 1.0):
        ks = np.array([max(1, int(part * m)) for m in lens], dtype=np.int64)
        to = np.concatenate([[0], np.cumsum(ks)]).astype(np.int64)
        out = torch.full((int(to[-1]) + 4,), -7, dtype=torch.int32, device="cuda")
        dev = [torch.from_numpy(a).cuda() for a in (offs, ks, to)]
        ctx.spts_select_topk_segmented(torch.from_numpy(flat.view(np.int32)).cuda().view(torch.float32), dev[0], dev[1], dev[2], len(lens), n, 1, out)
        got = out.cpu().numpy()
        assert (got[-4:] == -7).all()
        for b, m in enumerate(lens):
            assert np.array_equal(got[to[b]:to[b + 1]], expected(keys[b, :m], int(ks[b]), 1)), (part, b)


def _best_us(torch, call, repeats=7, per=5):
    """Shortest time of a call among `repeats` runs of `per` calls each."""
    call()
    best = float("inf")
    for _ in range(repeats):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(per):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / per * 1e3)
    return best


@pytest.mark.parametrize("share", [0.05, 0.4, 0.95])
def test_long_row_topk_time_does_not_depend_on_the_spread(torch, share):
    """Scores that spread over many octaves, and signed ones, cost what scores within an octave do: one sweep.  (A row that is sampled,
    swept and then swept three more times takes 1.6 to 2.3 times as long; the bound lies between.)"""
    rows, n = 512, 131072
    k = int(share * n)
    z = torch.randn((rows, n), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    ctx = runtime.make_context(synth.TINY, n, 1, 1, synth.TINY.Dff)
    out = torch.zeros((rows, k), dtype=torch.int32, device="cuda")
    us = {}
    for name, s in (("narrow", torch.softmax(0.5 * z, 1)), ("1.5", torch.softmax(1.5 * z, 1)), ("3", torch.softmax(3.0 * z, 1)), ("signed", z)):
        us[name] = _best_us(torch, lambda: ctx.spts_select_topk_batched(s, n, k, 1, rows, out))
    assert max(us.values()) <= 1.35 * us["narrow"], us


@pytest.mark.parametrize("n", [32772, 70000, 131072])
def test_long_row_topk_threshold_among_neighbouring_values(torch, n):
    """Signed scores whose bracket spans zero (its keys do not fit the 21 bits that are kept of them) with a threshold among values that
    are a few units in the last place apart, single and repeated."""
    rng = np.random.default_rng(n)
    s = rng.standard_normal((4, n)).astype(np.float32)
    for b, (centre, steps) in enumerate(((0.01, 4000), (-0.01, 4000), (0.003, 7), (-1e-30, 300))):
        at = rng.choice(n, n // 70, replace=False)
        s[b, at] = (np.float32(centre).view(np.int32) + rng.integers(0, steps, at.size).astype(np.int32)).view(np.float32)
    sd = torch.from_numpy(s).cuda()
    ctx = runtime.make_context(synth.TINY, n, 1, 1, synth.TINY.Dff)
    for b in range(4):
        cluster = np.abs(s[b] - np.float32((0.01, -0.01, 0.003, -1e-30)[b])) < 1e-4 * abs((0.01, -0.01, 0.003, -1e-30)[b])
        above = int((s[b] > s[b][cluster].max()).sum())
        for inside in (1, n // 300, n // 140, int(cluster.sum())):
            k = above + inside
            out = torch.full((4, k), -7, dtype=torch.int32, device="cuda")
            ctx.spts_select_topk_batched(sd, n, k, 0, 4, out)
            got = out.cpu().numpy()
            for row in range(4):
                assert np.array_equal(got[row], orc.topk_select(s[row], k, 0)), (b, k, row)


@pytest.mark.parametrize("share", [0.05, 0.4, 0.95])
def test_long_row_topk_time_does_not_depend_on_ties(torch, share):
    """Scores of fifty values, 2 % of the row each (the selection ends between equal ones), cost what distinct scores do (equal keys ranked
    one by one took 3 to 7 times as long); and the lowest indices of the last value are the ones taken."""
    rows, n = 512, 131072
    k = int(share * n)
    u = torch.rand((rows, n), generator=torch.Generator(device="cuda").manual_seed(4), device="cuda")
    ctx = runtime.make_context(synth.TINY, n, 1, 1, synth.TINY.Dff)
    out = torch.zeros((rows, k), dtype=torch.int32, device="cuda")
    distinct = _best_us(torch, lambda: ctx.spts_select_topk_batched(u, n, k, 1, rows, out))
    s = torch.floor(50.0 * u)
    tied = _best_us(torch, lambda: ctx.spts_select_topk_batched(s, n, k, 1, rows, out))
    for row in (0, 7, rows - 1):
        assert np.array_equal(out[row].cpu().numpy(), orc.topk_select(s[row].cpu().numpy(), k, 1)), row
    assert tied <= 1.6 * distinct, (tied, distinct)


@pytest.mark.parametrize("n", [32772, 65536, 131072])
def test_long_row_topk_of_rows_whose_sample_is_one_value(torch, n):
    """Rows that look like a single value at the sample's places (two of every few quads): all equal, and with every other score larger,
    smaller or on both sides, so that the threshold is that value or far from it."""
    rng = np.random.default_rng(n)
    quads = n // 4
    seen = np.zeros(quads, bool)
    seen[(np.arange(2048, dtype=np.int64) * quads) // 2048] = True
    seen = np.repeat(seen, 4)[:n]
    z = rng.standard_normal(n).astype(np.float32)
    rows = np.stack([np.full(n, 0.25), np.where(seen, 0.25, 1.0 + np.abs(z)), np.where(seen, 0.25, -np.abs(z)), np.where(seen, 0.25, z),
                     np.where(seen, -0.0, np.where(rng.random(n) < 0.5, 0.0, z))]).astype(np.float32)
    sd = torch.from_numpy(rows).cuda()
    ctx = runtime.make_context(synth.TINY, n, 1, 1, synth.TINY.Dff)
    for k in (n // 60, int(0.1 * n), int(0.4 * n), int(0.75 * n), n - n // 60):
        for protect in (0, 1):
            out = torch.full((len(rows), k), -7, dtype=torch.int32, device="cuda")
            ctx.spts_select_topk_batched(sd, n, k, protect, len(rows), out)
            got = out.cpu().numpy()
            for b in range(len(rows)):
                assert np.array_equal(got[b], orc.topk_select(rows[b], k, protect)), (b, k, protect)


@pytest.mark.parametrize("rows", [16, 512])
def test_long_row_topk_of_equal_scores_is_cheap(torch, rows):
    """Rows of equal scores leave the one-sweep route by their sample and need three sweeps (1.7 to 2.0 times the time of distinct scores), not
    the seven of a row about which nothing is known (3.3 to 4.3 times)."""
    n, k = 131072, 52428
    s = torch.full((rows, n), 0.25, device="cuda")
    u = torch.rand((rows, n), generator=torch.Generator(device="cuda").manual_seed(4), device="cuda")
    ctx = runtime.make_context(synth.TINY, n, 1, 1, synth.TINY.Dff)
    out = torch.zeros((rows, k), dtype=torch.int32, device="cuda")
    distinct = _best_us(torch, lambda: ctx.spts_select_topk_batched(u, n, k, 1, rows, out))
    equal = _best_us(torch, lambda: ctx.spts_select_topk_batched(s, n, k, 1, rows, out))
    assert equal <= 2.5 * distinct, (equal, distinct)


def test_long_row_topk_of_sorted_scores_fits_its_regions(torch):
    """Sorted normal scores: the threshold's 13-bit bin, about 790 scores, lies in one or two wavefronts' slices and has to fit their regions
    (1.8 to 2 times the time of the same scores shuffled; 3.5 times by 8-bit passes over the whole row)."""
    n, k = 131072, 52428
    z = torch.randn((1, n), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda")
    ctx = runtime.make_context(synth.TINY, n, 1, 1, synth.TINY.Dff)
    out = torch.zeros((1, k), dtype=torch.int32, device="cuda")
    shuffled = _best_us(torch, lambda: ctx.spts_select_topk_batched(z, n, k, 1, 1, out))
    for s in (torch.sort(z, 1)[0].contiguous(), torch.sort(z, 1, descending=True)[0].contiguous()):
        us = _best_us(torch, lambda: ctx.spts_select_topk_batched(s, n, k, 1, 1, out))
        assert np.array_equal(out[0].cpu().numpy(), orc.topk_select(s[0].cpu().numpy(), k, 1))
        assert us <= 2.6 * shuffled, (us, shuffled)
