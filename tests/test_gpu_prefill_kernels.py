"""The bf16 prefill kernels for head_dim 128 (the wide kernel: one wave per SIMD,
64 rows per wave, 16-token blocks; the narrow one: 32 rows per wave, for calls
that leave CUs idle; the software-pipelined kernel: two waves per SIMD) against
the four-wave kernel and the fp64 oracle.  All kernels take every query row
through the same sequence of operations, so their outputs must agree bit for
bit; each must also meet the bf16 tolerance against the oracle.  CASES and
DEFAULT_CASES cover every group size that divides 32, block sizes 16 / 32 / 64,
crops not aligned to a block with NaN-poisoned tail slots, suffixes shorter
than one query tile, tiles that straddle the diagonal, and several sequences of
different lengths in one call, against the oracle and the full reset of every
sequence in one call (bitwise); most are small, so by default they run the narrow
kernel (16-token blocks) or the four-wave one.  TAKEN has calls past the lines
of the dispatch, for the wide and the pipelined kernel and every group, and
tells by the number of workgroups which kernel ran."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_helpers import assert_close, contaminated_then_crop, dev, log, make_pool, oracle_suffix, probed_workgroups

pytestmark = pytest.mark.gpu


def _blocks(n, B):
    return -(-n // B)


def _run(kind, geom, eps, B, scale, ran=None):
    """Contaminated prefill, poisoned crop, then one replay call over all
    episodes; returns the per-episode outputs (``ran`` gets the number of
    workgroups that wrote the clock probe)."""
    nb = sum(_blocks(e.t_contaminated, B) + _blocks(e.t_sanitized, B) for e in eps) + 4
    mbps = max(_blocks(max(e.t_contaminated, e.t_sanitized), B) for e in eps) + 2
    pool = make_pool(geom, "bf16", nb, len(eps), mbps, block_size=B)
    pool.set_prefill_kernel(kind)
    for i, e in enumerate(eps):
        contaminated_then_crop(pool, e, i, scale, poison=True)
    q, k, v = (torch.cat([dev(getattr(e, x)[e.prefix:], "bf16") for e in eps]) for x in ("q", "k", "v"))
    o = torch.empty_like(q)
    n = probed_workgroups(pool, lambda: pool.replay(0, list(range(len(eps))), [e.suffix for e in eps], q, k, v, o, scale))
    if ran is not None:
        ran.append(n)
    out, off = [], 0
    for e in eps:
        out.append(o[off:off + e.suffix])
        off += e.suffix
    return out


CASES = [
    # (Hq, Hkv, B, [(P, S), ...])
    (32, 8, 16, [(300, 77)]),
    (32, 8, 16, [(0, 130)]),
    (32, 8, 16, [(8189, 96)]),          # the 8B crop point, short suffix
    (32, 8, 16, [(64, 64)]),            # aligned prefix, one query tile
    (32, 32, 16, [(100, 200)]),         # G = 1
    (64, 2, 32, [(50, 70)]),            # G = 32
    (16, 8, 64, [(129, 64)]),           # G = 2, B = 64
    (32, 4, 32, [(1021, 3)]),           # G = 8, fewer queries than one 32-row block
    (64, 4, 16, [(700, 45)]),           # G = 16
    (32, 8, 16, [(517, 90), (0, 33), (2000, 257), (63, 1)]),   # ragged batch in one call
    # more query tiles per KV head than one XCD holds at once (the tiles of a
    # head run in several rounds on its XCD)
    (32, 8, 16, [(5, 2122), (0, 4160)]),
]


@pytest.mark.parametrize("hq,hkv,B,ps", CASES)
def test_pipelined_equals_four_wave_and_oracle(hq, hkv, B, ps):
    geom = W.AttnGeometry(hq, hkv, 128)
    log(f"prefill kernels {hq}/{hkv} B={B} episodes {ps}")
    rng = np.random.default_rng(hq * 7919 + B + sum(p for p, _ in ps))
    eps = [W.draw_episode(rng, geom, "bf16", P, S, P + S + 3) for P, S in ps]
    scale = 128 ** -0.5
    auto = _run("auto", geom, eps, B, scale)          # narrow or wide where B = 16, else mostly four-wave
    pipe = _run("pipelined", geom, eps, B, scale)
    four = _run("four_wave", geom, eps, B, scale)
    for e, a, p, f in zip(eps, auto, pipe, four):
        assert torch.equal(p, f), f"pipelined and four-wave kernels differ (P={e.prefix}, S={e.suffix})"
        assert torch.equal(a, f), f"default and four-wave kernels differ (P={e.prefix}, S={e.suffix})"
        assert_close(a.float().cpu().numpy(), oracle_suffix(e, scale), "bf16", f"P={e.prefix} S={e.suffix}")


# the default kernel on more shapes: the 8B replay at full size, one partial
# query tile, tiles that straddle the diagonal, every group size dividing 16
DEFAULT_CASES = [
    (32, 8, 16, [(8189, 2048)]),         # the 8B replay at full size
    (32, 8, 16, [(300, 31)]),            # one partial query tile
    (32, 8, 16, [(0, 64)]),              # one tile, prefix 0
    (32, 8, 16, [(77, 96)]),             # a tile and a partial one
    (32, 8, 32, [(1000, 130)]),          # B = 32
    (16, 16, 64, [(129, 300)]),          # G = 1, B = 64
    (16, 8, 16, [(50, 150)]),            # G = 2
    (64, 8, 16, [(700, 45)]),            # G = 8
    (64, 4, 16, [(65, 37)]),             # G = 16
    (32, 8, 16, [(517, 90), (0, 33), (2000, 257), (63, 1), (4000, 700)]),   # ragged batch
]


@pytest.mark.parametrize("hq,hkv,B,ps", DEFAULT_CASES)
def test_default_kernel_matches_oracle_and_full_reset(hq, hkv, B, ps):
    geom = W.AttnGeometry(hq, hkv, 128)
    log(f"default kernel {hq}/{hkv} B={B} episodes {ps}")
    rng = np.random.default_rng(hq * 131 + B + sum(p + 3 * s for p, s in ps))
    eps = [W.draw_episode(rng, geom, "bf16", P, S, P + S + 3) for P, S in ps]
    scale = 128 ** -0.5
    outs = _run("auto", geom, eps, B, scale)
    for e, o in zip(eps, outs):
        if e.suffix * hq <= 65536:
            ref, rows = oracle_suffix(e, scale), None
            got = o.float().cpu().numpy()
        else:                                # the full-size case: every 7th row
            rows = np.arange(0, e.suffix * hq, 7)
            ref = oracle_suffix(e, scale, rows=rows)
            got = o.reshape(-1, 128)[torch.from_numpy(rows).cuda()].float().cpu().numpy()
        assert_close(got, ref, "bf16", f"P={e.prefix} S={e.suffix}")
    # Theorem 1, bitwise: the full reset of each sanitized trajectory in one call
    nb = sum(_blocks(e.t_sanitized, B) for e in eps) + 4
    mbps = max(_blocks(e.t_sanitized, B) for e in eps) + 2
    pool = make_pool(geom, "bf16", nb, len(eps), mbps, block_size=B)
    fq, fk, fv = (torch.cat([dev(getattr(e, x), "bf16") for e in eps]) for x in ("q", "k", "v"))
    fo = torch.empty_like(fq)
    assert pool.full_reset(0, list(range(len(eps))), [e.t_sanitized for e in eps], fq, fk, fv, fo,
                           scale) == 0
    torch.cuda.synchronize()
    off = 0
    for e, o in zip(eps, outs):
        assert torch.equal(fo[off + e.prefix:off + e.t_sanitized], o), f"P={e.prefix} S={e.suffix}"
        off += e.t_sanitized


def test_pipelined_full_reset_equals_replay_at_8b_crop():
    """Theorem 1 on the pipelined kernel at the unaligned 8B crop (P = 8189),
    with a suffix spanning several query tiles."""
    geom = W.AttnGeometry(32, 8, 128)
    rng = np.random.default_rng(8189)
    P, S = 8189, 640
    ep = W.draw_episode(rng, geom, "bf16", P, S, P + S + 3)
    scale = 128 ** -0.5
    B = 16
    pool = make_pool(geom, "bf16", 2 * _blocks(P + S + 3, B) + 4, 2, _blocks(P + S + 3, B) + 2)
    contaminated_then_crop(pool, ep, 0, scale, poison=True)
    q, k, v = (dev(getattr(ep, x)[P:], "bf16") for x in ("q", "k", "v"))
    o = torch.empty_like(q)
    assert pool.replay(0, [0], [S], q, k, v, o, scale) == 0
    fq, fk, fv = (dev(getattr(ep, x), "bf16") for x in ("q", "k", "v"))
    fo = torch.empty_like(fq)
    assert pool.full_reset(0, [1], [P + S], fq, fk, fv, fo, scale) == 0
    torch.cuda.synchronize()
    assert torch.equal(fo[P:], o)
    rows = np.arange(0, S * 32, 37 * 32 + 5)         # flat (token, head) rows
    ref = oracle_suffix(ep, scale, rows=rows)
    got = o.reshape(S * 32, 128)[torch.from_numpy(rows).cuda()]
    assert_close(got.float().cpu().numpy(), ref, "bf16", "8B crop, sampled rows")


@pytest.mark.parametrize("P,S,tile_waves", [(130700, 100, 2), (129786, 1030, 8), (130900, 100, 0), (129890, 1030, 8)])
def test_longest_sequences_for_the_lds_block_table(P, S, tile_waves):
    """Sequences at the limit of the narrow and the wide kernel (130816 keys: a
    workgroup's copy of the block table fills its LDS share) and just past it
    (the host then runs the four-wave and the pipelined kernel): the default kernel
    bitwise against the four-wave one, and sampled rows against the oracle."""
    geom = W.AttnGeometry(32, 8, 128)
    log(f"longest sequences: P={P} S={S}")
    rng = np.random.default_rng(P)
    eps = [W.draw_episode(rng, geom, "bf16", P, S, P + S + 3)]
    scale = 128 ** -0.5
    ran = []
    auto = _run("auto", geom, eps, 16, scale, ran)[0]
    assert ran[0] == (-(-S // (8 * tile_waves)) * 8 if tile_waves else 0)
    four = _run("four_wave", geom, eps, 16, scale)[0]
    assert torch.equal(auto, four), f"default and four-wave kernels differ (P={P}, S={S})"
    rows = np.arange(0, S * geom.n_q_heads, 97 if S < 1000 else 997)
    ref = oracle_suffix(eps[0], scale, rows=rows)
    got = auto.reshape(-1, 128)[torch.from_numpy(rows).cuda()].float().cpu().numpy()
    assert_close(got, ref, "bf16", f"P={P} S={S}")


# What decides the default kernel is the number of workgroups of narrow tiles (2, then 4 waves of
# floor(32 / G) tokens, at most 256 workgroups), so: one case just inside and one just past each line, a
# ragged batch of short sequences past it, groups that do not divide 32 (padded rows), splits, both
# block-size families
@pytest.mark.parametrize("hq,hkv,B,ps,ws_tokens", [
    (32, 8, 16, [(45, 512)], 0),                       # 32 tiles of 2 waves x 8 heads = 256
    (32, 8, 16, [(45, 513)], 0),                       # 33: four waves
    (32, 8, 16, [(200, 1024)], 0),                     # 32 tiles of 4 waves x 8 heads = 256
    (32, 8, 16, [(200, 1025)], 0),                     # 33: wide
    (64, 2, 16, [(33, 601)], 0),                       # G = 32, wide
    (16, 16, 16, [(7, 1900), (70, 150)], 0),           # G = 1, wide
    (32, 8, 16, [(37 * i, 33 - i % 5) for i in range(40)], 0),
    (28, 4, 16, [(300, 77)], 0),                       # G = 7: two waves
    (28, 4, 16, [(100, 700), (3, 20)], 0),             # four waves
    (28, 4, 16, [(500, 1100)], 0),                     # wide
    (20, 4, 16, [(129, 50)], 0),                       # G = 5
    (28, 4, 32, [(129, 900)], 0),                      # four-wave (57 tiles of 4 waves x 4 heads = 228)
    (28, 4, 64, [(64, 40)], 0),                        # four-wave
    (32, 8, 16, [(900, 40)], 40),                      # split keys
    (28, 4, 16, [(2000, 130)], 130),
])
def test_default_kernel_equals_four_wave_at_its_lines(hq, hkv, B, ps, ws_tokens):
    geom = W.AttnGeometry(hq, hkv, 128)
    log(f"default kernel at its lines {hq}/{hkv} B={B} {len(ps)} episodes {ps[:3]} workspace {ws_tokens}")
    rng = np.random.default_rng(hq + B + sum(p + 3 * s for p, s in ps))
    eps = [W.draw_episode(rng, geom, "bf16", P, S, P + S + 3) for P, S in ps]
    scale = 128 ** -0.5
    outs = {}
    for kind in ("auto", "pipelined", "four_wave"):
        nb = sum(_blocks(e.t_contaminated, B) + _blocks(e.t_sanitized, B) for e in eps) + 4
        mbps = max(_blocks(max(e.t_contaminated, e.t_sanitized), B) for e in eps) + 2
        pool = make_pool(geom, "bf16", nb, len(eps), mbps, block_size=B, split_q=ws_tokens, max_splits=8)
        if ws_tokens and kind == "four_wave" and 32 % (hq // hkv) == 0:
            continue                     # cut for its own tiles: another number of splits, other bits
        pool.set_prefill_kernel(kind)
        for i, e in enumerate(eps):
            contaminated_then_crop(pool, e, i, scale, poison=True)
        q, k, v = (torch.cat([dev(getattr(e, x)[e.prefix:], "bf16") for e in eps]) for x in ("q", "k", "v"))
        o = torch.empty_like(q)
        assert pool.replay(0, list(range(len(eps))), [e.suffix for e in eps], q, k, v, o, scale) == 0
        torch.cuda.synchronize()
        outs[kind] = o
    for kind in set(outs) - {"auto"}:
        assert torch.equal(outs[kind], outs["auto"]), f"{kind} differs from the default kernel"
    off = 0
    for i, e in enumerate(eps):
        if i < 2:
            rows = np.unique(np.concatenate([np.arange(0, e.suffix * hq, 37), np.arange(e.suffix * hq - hq, e.suffix * hq)]))
            got = outs["auto"][off:off + e.suffix].reshape(-1, 128)[torch.from_numpy(rows).cuda()]
            assert_close(got.float().cpu().numpy(), oracle_suffix(e, scale, rows=rows), "bf16",
                         f"P={e.prefix} S={e.suffix}")
        off += e.suffix


@pytest.mark.parametrize("hq,hkv,P,S,split_len,auto_waves,pipe_waves", [
    (32, 8, 900, 40, 128, 2, 8),         # groups that divide 32: narrow or wide, and pipelined, one plan
    (64, 8, 700, 300, 256, 8, 8),
    (28, 4, 2000, 130, 320, 0, 0),       # others: the four-wave kernel under every choice
])
def test_split_calls_of_each_choice(hq, hkv, P, S, split_len, auto_waves, pipe_waves):
    """Which kernel a bf16 call with split keys runs under each choice, and that
    one plan gives one result."""
    geom = W.AttnGeometry(hq, hkv, 128)
    ep = W.draw_episode(np.random.default_rng(hq + P), geom, "bf16", P, S, P + S + 3)
    q, k, v = (dev(getattr(ep, x)[P:], "bf16") for x in ("q", "k", "v"))
    outs = {}
    for kind, waves in (("auto", auto_waves), ("pipelined", pipe_waves), ("four_wave", 0)):
        pool = make_pool(geom, "bf16", 2 * _blocks(P + S + 3, 16) + 4, 1, _blocks(P + S + 3, 16) + 2, split_q=S, max_splits=8)
        contaminated_then_crop(pool, ep, 0, 128 ** -0.5, poison=True)
        pool.set_prefill_kernel(kind)
        o = torch.empty_like(q)
        n = probed_workgroups(pool, lambda: pool.replay(0, [0], [S], q, k, v, o, 128 ** -0.5))
        tile = waves * (32 // (hq // hkv))
        # a workgroup whose split starts past its tile's last key leaves before the probe
        want = hkv * sum(-(-(P + min(S, t + tile)) // split_len) for t in range(0, S, tile)) if tile else 0
        assert n == want, f"{kind}: {n} workgroups, not {want}"
        outs[kind] = o
    assert torch.equal(outs["auto"], outs["pipelined"])
    if 32 % (hq // hkv):                 # else the four-wave kernel cuts for its own tiles
        assert torch.equal(outs["auto"], outs["four_wave"])


# (dtype, Hq, Hkv, B, [(P, S), ...], kernel the call runs, waves that own 32 query rows each to a workgroup)
TAKEN = [
    # tiles of eight row blocks that short or few-token sequences fill badly: the four-wave kernel
    ("fp8", 16, 16, 16, [(100, 12)] * 64, "four-wave", 0),
    ("fp8", 20, 4, 32, [(400, 116)] * 50, "four-wave", 0),
    ("bf16", 24, 8, 16, [(100, 12)] * 64, "four-wave", 0),
    ("bf16", 28, 4, 64, [(90, 45)] * 33, "four-wave", 0),
    ("bf16", 28, 4, 16, [(43, 312)] * 8, "four-wave", 0),          # 5 key tiles to a query tile
    ("bf16", 28, 4, 16, [(832, 509)] * 4, "wide", 8),              # 17
    ("bf16", 28, 4, 32, [(900, 700)] * 3, "pipelined", 8),
    ("fp8", 32, 8, 16, [(1500, 600), (900, 1000)], "pipelined", 8),
    # every group in the wide kernel, past the 256 workgroups of the narrow one; crops inside a block
    ("bf16", 64, 64, 16, [(45, 530), (3, 20)], "wide", 8),
    ("bf16", 128, 64, 16, [(77, 270)], "wide", 8),
    ("bf16", 128, 32, 16, [(300, 257), (17, 64)], "wide", 8),
    ("bf16", 64, 8, 16, [(301, 520), (0, 33)], "wide", 8),
    ("bf16", 256, 32, 16, [(129, 140)], "wide", 8),
    ("bf16", 256, 16, 16, [(65, 140)], "wide", 8),
    ("bf16", 256, 8, 16, [(129, 135), (1000, 1)], "wide", 8),
    ("bf16", 200, 40, 16, [(700, 192)], "wide", 8),
    # and in the pipelined one by default
    ("bf16", 64, 64, 32, [(45, 530), (3, 20)], "pipelined", 8),
    ("bf16", 128, 64, 64, [(77, 270)], "pipelined", 8),
    ("bf16", 128, 32, 32, [(300, 257), (17, 64)], "pipelined", 8),
    ("bf16", 256, 32, 64, [(129, 140)], "pipelined", 8),
    ("bf16", 256, 16, 32, [(65, 140)], "pipelined", 8),
    ("bf16", 256, 8, 64, [(129, 135), (1000, 1)], "pipelined", 8),
    ("bf16", 224, 32, 32, [(701, 150)], "pipelined", 8),
]


@pytest.mark.parametrize("dtype,hq,hkv,B,ps,kernel,waves", TAKEN)
def test_kernel_taken_by_default(dtype, hq, hkv, B, ps, kernel, waves):
    """Which kernel a call takes, its bits against the four-wave kernel's, and
    sampled rows of two episodes against the oracle (bf16)."""
    from paper_2609_04875_amd import BF16, FP8_E4M3, KVPool
    geom = W.AttnGeometry(hq, hkv, 128)
    log(f"kernel taken {dtype} {hq}/{hkv} B={B} {len(ps)} x {ps[0]}: {kernel}")
    rng = np.random.default_rng(hq + 7 * hkv + B + len(ps))
    eps = [W.draw_episode(rng, geom, "bf16", P, S, P + S + 3) for P, S in ps[:4]]
    eps = [eps[i % len(eps)] for i in range(len(ps))]
    scale = 128 ** -0.5
    need = [_blocks(e.t_contaminated, B) + 1 for e in eps]
    q, k, v = (torch.cat([dev(getattr(e, x)[e.prefix:], "bf16") for e in eps]) for x in ("q", "k", "v"))
    outs = []
    for kind in ("auto", "four_wave"):
        pool = KVPool(1, hq, hkv, 128, sum(need) + 4, len(eps), max(need) + 2, FP8_E4M3 if dtype == "fp8" else BF16, B)
        if dtype == "fp8":
            pool.set_kv_scales([5 / 448], [4 / 448])
        for i, e in enumerate(eps):
            contaminated_then_crop(pool, e, i, scale, poison=True)
        pool.set_prefill_kernel(kind)
        o = torch.empty_like(q)
        n = probed_workgroups(pool, lambda: pool.replay(0, list(range(len(eps))), [e.suffix for e in eps], q, k, v, o, scale))
        tile = (waves if kind == "auto" else 0) * (32 // (hq // hkv))
        assert n == (sum(-(-S // tile) for _, S in ps) * hkv if tile else 0), f"{kind}: {n} workgroups"
        outs.append(o)
    assert torch.isfinite(outs[0].float()).all() and torch.equal(outs[0], outs[1])
    off = 0
    for e in eps[:2]:
        if dtype == "bf16":
            rows = np.unique(np.concatenate([np.arange(0, e.suffix * hq, 97), np.arange(e.suffix * hq - hq, e.suffix * hq)]))
            got = outs[0][off:off + e.suffix].reshape(-1, 128)[torch.from_numpy(rows).cuda()]
            assert_close(got.float().cpu().numpy(), oracle_suffix(e, scale, rows=rows), "bf16", f"P={e.prefix} S={e.suffix}")
        off += e.suffix
