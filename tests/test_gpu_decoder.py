"""Full decoder layers on the GPU against the fp64 oracle (oracle/decoder.py):
the elementwise kernels (RMSNorm, rotary embedding at absolute positions,
SwiGLU gate) to one bf16 rounding, and replay through two full layers at a
G = 2 and a G = 7 geometry against the oracle and bitwise against the full
reset (Theorem 1)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import bf16_round
from oracle import decoder as DEC
from gpu_helpers import log

from paper_2609_04875_amd import DecoderReplay, gemm_bf16, rmsnorm, rope_, silu_mul
from paper_2609_04875_amd.decoder import rope_qk_
from paper_2609_04875_amd.pool import gemm_bf16_multi, gemm_silu_bf16

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().to(torch.bfloat16)


def _f64(t):
    return t.float().cpu().numpy().astype(np.float64)


def _within_one_rounding(got, want):
    """got is want's fp32 value rounded once to bf16: within one bf16 step of
    the exact value (2^-8 relative), plus a floor for values near 0."""
    d = np.abs(got - want)
    assert (d <= 2.0 ** -8 * np.abs(want) + 1e-6).all(), (d.max(), np.argmax(d))


def test_rmsnorm_matches_oracle():
    rng = np.random.default_rng(0)
    x = bf16_round(rng.standard_normal((37, 4096)) * 3)
    g = bf16_round(1 + 0.1 * rng.standard_normal(4096))
    got = _f64(rmsnorm(_dev(x), _dev(g), 1e-5))
    _within_one_rounding(got, DEC.rms_norm(x, g, 1e-5))


def test_rope_matches_oracle_at_large_positions():
    rng = np.random.default_rng(1)
    x = bf16_round(rng.standard_normal((50, 8, 128)))
    pos = rng.integers(0, 131072, size=50).astype(np.int32)
    t = _dev(x)
    rope_(t, torch.from_numpy(pos).cuda(), 5e5)
    _within_one_rounding(_f64(t), DEC.rope(x, pos, 5e5))


@pytest.mark.parametrize("n,hq,hkv,d", [(1, 32, 8, 128), (5, 7, 1, 64), (1025, 4, 2, 128), (3, 2, 1, 256),
                                        (6, 3, 2, 272), (9, 2, 2, 24)])
def test_rope_of_q_and_k_in_one_call(n, hq, hkv, d):
    """Both row kernels (one and four tokens a workgroup, a ragged last one),
    the widest head they take, and head sizes that take the pair kernel, as does
    a tensor off the 16-byte boundary: the same bits on every route, which
    match the oracle."""
    rng = np.random.default_rng(n + d)
    q, k = bf16_round(rng.standard_normal((n, hq, d))), bf16_round(rng.standard_normal((n, hkv, d)))
    pos = rng.integers(0, 131072, size=n).astype(np.int32)
    pd = torch.from_numpy(pos).cuda()
    tq, tk = _dev(q), _dev(k)
    off = torch.empty(q.size + 2, dtype=torch.bfloat16, device="cuda")[2:].view(n, hq, d)
    off.copy_(tq)
    single = rope_(tq.clone(), pd, 5e5)
    rope_qk_(tq, tk, pd, 5e5)
    rope_(off, pd, 5e5)
    _within_one_rounding(_f64(tq), DEC.rope(q, pos, 5e5))
    _within_one_rounding(_f64(tk), DEC.rope(k, pos, 5e5))
    assert torch.equal(tq, single) and torch.equal(tq, off)


def test_silu_mul_matches_oracle():
    rng = np.random.default_rng(2)
    gu = bf16_round(rng.standard_normal((19, 2 * 1024)) * 4)
    got = _f64(silu_mul(_dev(gu)))
    _within_one_rounding(got, DEC.silu(gu[:, :1024]) * gu[:, 1024:])


def _weights(rng, n_layers, dm, hq, hkv, d, dff):
    b = lambda *shape, s=1.0: bf16_round(rng.standard_normal(shape) * s)
    ws = []
    for _ in range(n_layers):
        ws.append({"wq": b(dm, hq * d, s=dm ** -0.5), "wk": b(dm, hkv * d, s=dm ** -0.5),
                   "wv": b(dm, hkv * d, s=dm ** -0.5), "wo": b(hq * d, dm, s=(hq * d) ** -0.5),
                   "wg": b(dm, dff, s=dm ** -0.5), "wu": b(dm, dff, s=dm ** -0.5),
                   "wd": b(dff, dm, s=dff ** -0.5),
                   "g_attn": bf16_round(1 + 0.1 * rng.standard_normal(dm)),
                   "g_mlp": bf16_round(1 + 0.1 * rng.standard_normal(dm))})
    return ws


def _dev_weights(ws):
    return [{"wq": _dev(w["wq"].T), "wk": _dev(w["wk"].T), "wv": _dev(w["wv"].T), "wo": _dev(w["wo"].T),
             "w_gate_up": _dev(np.concatenate([w["wg"].T, w["wu"].T])), "w_down": _dev(w["wd"].T),
             "g_attn": _dev(w["g_attn"]), "g_mlp": _dev(w["g_mlp"])} for w in ws]


@pytest.mark.parametrize("m,dff,k", [
    # one product per tile of the projection with the gate in its epilogue, ragged in rows or columns (a
    # last group of 8), then K = 192 and the 256 x 256 kernel's size, which run as two launches
    (1, 1000, 128), (16, 2048, 640), (17, 1024, 256), (40, 2040, 384), (100, 1496, 1024), (200, 3064, 384),
    (300, 2048, 896), (700, 2056, 256), (1400, 2040, 128), (9, 96, 192), (4096, 2048, 128),
    (1, 8200, 128), (31, 8192, 384)])
def test_projection_with_gate_equals_two_steps(m, dff, k):
    rng = np.random.default_rng(m + dff)
    x, w = _dev(rng.standard_normal((m, k)) * 2), _dev(rng.standard_normal((2 * dff, k)) * k ** -0.5)
    want = silu_mul(gemm_bf16(x, w))
    scratch, out = torch.empty(m, 2 * dff, dtype=torch.bfloat16, device="cuda"), torch.empty_like(want)
    assert torch.equal(gemm_silu_bf16(x, w, scratch, out), want)


@pytest.mark.parametrize("m,k,ns", [(1, 256, (512, 128, 128)), (40, 640, (1000, 8, 264)), (102, 384, (2048, 1024)),
                                    (300, 128, (4096, 1024, 1024)), (33, 72, (64, 16, 24)),
                                    (4096, 128, (4096, 64, 64)), (5, 128, (4104,))])
def test_projections_in_one_call_equal_separate_ones(m, k, ns):
    rng = np.random.default_rng(m + k)
    x = _dev(rng.standard_normal((m, k)))
    ws = [_dev(rng.standard_normal((n, k)) * k ** -0.5) for n in ns]
    outs = [torch.empty(m, n, dtype=torch.bfloat16, device="cuda") for n in ns]
    gemm_bf16_multi(x, ws, outs)
    for w, o in zip(ws, outs):
        assert torch.equal(o, gemm_bf16(x, w))


@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 64), (7, 1, 64)])
def test_decoder_replay_matches_oracle_and_full_reset(hq, hkv, d):
    log(f"decoder layers {hq}/{hkv}/{d}")
    rng = np.random.default_rng(hq)
    dm, dff, T, P, Tc = hq * d, 384, 300, 203, 330
    eps, theta = 1e-5, 5e5
    ws = _weights(rng, 2, dm, hq, hkv, d, dff)
    x = bf16_round(rng.standard_normal((T, dm)))
    xc = np.concatenate([x[:P], bf16_round(rng.standard_normal((Tc - P, dm)))])   # contaminated run
    dec = DecoderReplay(_dev_weights(ws), hq, hkv, d, eps, theta, n_blocks=2 * (-(-Tc // 16)) + 8,
                        max_seqs=2, max_blocks_per_seq=32)
    dec.replay(0, _dev(xc))
    assert dec.crop([0], [P]) == 0
    out = dec.replay(0, _dev(x[P:]))
    full = dec.full_reset(1, _dev(x))
    torch.cuda.synchronize()
    assert torch.equal(full[P:], out)                                 # Theorem 1, bitwise
    assert dec.pool.seq_len(0) == T and dec.pool.seq_len(1) == T
    ref, _ = DEC.decoder_layers(x, ws, hq, hkv, d, eps, theta)
    got, want = _f64(out), ref[P:]
    diff = np.abs(got - want)
    # the residual stream after two layers: two bf16 steps at the largest
    # magnitude, L1-relative 1e-2 (as for the stacked layers)
    assert diff.max() <= 2.0 ** -6 * np.abs(want).max(), (diff.max(), np.abs(want).max())
    assert diff.sum() / np.abs(want).sum() <= 1e-2


def test_captured_restore_replay_matches_eager():
    """Restore + replay through two layers recorded as one HIP graph: three
    replays, each from the restored contaminated state with eager library work
    in between, give the eager replay's bits every time."""
    log("decoder restore + replay as a HIP graph")
    hq, hkv, d = 4, 2, 64
    rng = np.random.default_rng(99)
    dm, dff, T, P, Tc = hq * d, 384, 300, 203, 330
    eps, theta = 1e-5, 5e5
    ws = _weights(rng, 2, dm, hq, hkv, d, dff)
    x = bf16_round(rng.standard_normal((T, dm)))
    xc = np.concatenate([x[:P], bf16_round(rng.standard_normal((Tc - P, dm)))])
    dec = DecoderReplay(_dev_weights(ws), hq, hkv, d, eps, theta, n_blocks=3 * (-(-Tc // 16)) + 8,
                        max_seqs=2, max_blocks_per_seq=32)
    dec.replay(0, _dev(xc))
    torch.cuda.synchronize()
    saved = dec.pool.save_meta()
    assert dec.crop([0], [P]) == 0
    want = dec.replay(0, _dev(x[P:])).clone()
    torch.cuda.synchronize()
    after = dec.pool.save_meta()

    dec.pool.load_meta(saved)
    cap = dec.capture_restore_replay(0, P, _dev(x[P:]))
    for i in range(3):
        dec.pool.load_meta(saved)
        got = cap.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want), f"graph replay {i} differs from the eager replay"
        assert all(torch.equal(a, b) for a, b in zip(dec.pool.save_meta(), after)), f"replay {i} tables"
        # eager work between replays: a full reset of another sequence
        dec.pool.refresh()
        full = dec.full_reset(1, _dev(x))
        torch.cuda.synchronize()
        assert torch.equal(full[P:], want)
        assert dec.crop([1], [0]) == 0
        torch.cuda.synchronize()


@pytest.mark.parametrize("n,hq,hkv,d", [(1, 88, 8, 128), (1, 89, 8, 128), (5, 512, 64, 64), (127, 300, 20, 64),
                                        (128, 300, 20, 64), (3, 4096, 0, 16), (64, 32, 0, 128), (65, 32, 0, 128),
                                        (4100, 1, 0, 128)])
def test_rope_of_many_heads(n, hq, hkv, d):
    """Both sides of the lines between a workgroup per token and a pair per
    thread (accesses to a token, tokens, pairs of one tensor, one head), bitwise
    equal to the latter, which takes tensors off the 16-byte boundary."""
    g = torch.Generator(device="cuda").manual_seed(hq + n)
    log(f"rope n={n} heads={hq}/{hkv} d={d}")
    q, k = (torch.randn(n, h, d, device="cuda", generator=g).to(torch.bfloat16) for h in (hq, hkv))
    pos = torch.randint(0, 131072, (n,), dtype=torch.int32, device="cuda", generator=g)

    def shifted(x):
        t = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")[1:].view(x.shape)
        return t.copy_(x)
    want_q, want_k = rope_(shifted(q), pos, 5e5), rope_(shifted(k), pos, 5e5) if hkv else k
    if hkv:
        rope_qk_(q, k, pos, 5e5)
    else:
        rope_(q, pos, 5e5)
    assert torch.equal(q, want_q) and torch.equal(k, want_k)


def test_rope_of_few_tokens_and_many_heads_is_not_a_serial_walk():
    x, pos = torch.zeros(1, 4096, 128, dtype=torch.bfloat16, device="cuda"), torch.ones(1, dtype=torch.int32, device="cuda")
    off = torch.zeros(x.numel() + 1, dtype=torch.bfloat16, device="cuda")[1:].view(x.shape)

    def us(t):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(30):
            rope_(t, pos, 5e5)
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / 30 * 1e3
    us(x), us(off)
    pairs = [(us(x), us(off)) for _ in range(5)]
    log(f"rope 1 x 4096 heads: on the boundary, off it (us) {pairs}")
    assert sorted(a / b for a, b in pairs)[2] < 3         # 16 when one workgroup took them all


def test_rope_of_more_tokens_than_one_grid_of_rows():
    """2^26 + 5 tokens: a workgroup for every four of them is 2^32 threads."""
    n, d = (1 << 26) + 5, 16
    x = torch.ones(n, 1, d, dtype=torch.bfloat16, device="cuda")
    pos = torch.arange(n, dtype=torch.int32, device="cuda")
    rope_(x, pos, 5e5)
    for s in (slice(0, 9), slice(n // 2, n // 2 + 9), slice(n - 9, n)):
        part = torch.ones(9, 1, d, dtype=torch.bfloat16, device="cuda")
        assert torch.equal(x[s], rope_(part, pos[s].contiguous(), 5e5))
