"""What a program that uses this framework has it do, as cases that can be timed.

A case is a dict of plain values.  ``prepare`` builds what the program has in
hand before the call (inputs on the GPU, the pool with its cached sequences,
weights), ``run`` is one pass through the public entry points, ``exact`` is the
same result in 64 bits from plain torch.  The kinds:

* ``replay``: restore (crop) + replay of the sanitized suffix of one or more
  episodes against their cached prefixes, one attention layer, in one call or
  in chunks (``KVPool.restore_replay`` / ``KVPool.replay``);
* ``decode``: one re-decode token for each of several cached sequences, one
  attention layer that is not the last (``KVPool.replay`` without commit);
* ``decoder``: restore + replay of a few tokens through full decoder layers
  (``DecoderReplay``);
* ``dense``: what surrounds the attention in one decoder layer, for many tokens
  (``rmsnorm``, ``gemm_bf16``, ``rope_``, ``silu_mul``);
* ``sample``: the next tokens from a batch of logits (``sample_tokens``).

Geometries are those of the workloads, the benchmark and the tests: 8B-like
(32 query / 8 KV heads of 128, d_model 4096, d_ff 14336), 70B-like (64 / 8,
d_model 8192), 7B-like with groups of seven (28 / 4, d_model 3584, d_ff 18944)
and the small fp32 one (8 / 8 heads of 64).
"""
from __future__ import annotations

import math
import random

import torch

from paper_2609_04875_amd import (BF16, F32, FP8_E4M3, DecoderReplay, KVPool, gemm_bf16, rmsnorm, rope_,
                                  sample_tokens, sample_workspace_bytes, silu_mul, workspace_bytes)

GEOMETRY = {            # query heads, KV heads, head size, d_model, d_ff
    "8b": (32, 8, 128, 4096, 14336),
    "70b": (64, 8, 128, 8192, 28672),
    "7b_g7": (28, 4, 128, 3584, 18944),
    "mha8_d64": (8, 8, 64, 512, 1408),
}
POOL_DTYPE = {"bf16": BF16, "fp8": FP8_E4M3, "f32": F32}
BLOCK = 16
KV_SCALE = 5.0 / 448    # FP8 cache: N(0, 1) values up to 5 sigma use the full range
EPS, THETA = 1e-5, 5e5


def listed():
    return [
        # the small accuracy-first episode: 640 cached tokens, target at 512, fp32; latency decides
        {"name": "replay_tiny_f32", "kind": "replay", "geometry": "mha8_d64", "dtype": "f32",
         "t_lo": 640, "t_hi": 640, "keep": 0.8, "episodes": 1, "len_seed": 0, "chunk": 0},
        # the benchmark's episode: 8189 tokens kept (inside a block), 2048 replayed
        {"name": "replay_8b", "kind": "replay", "geometry": "8b", "dtype": "bf16",
         "t_lo": 10237, "t_hi": 10237, "keep": 0.79995, "episodes": 1, "len_seed": 0, "chunk": 0},
        # many sessions forget at once: ragged lengths, targets at 10 % to 90 % of them, one launch
        {"name": "replay_ragged16_8b", "kind": "replay", "geometry": "8b", "dtype": "bf16",
         "t_lo": 4096, "t_hi": 16384, "keep": 0.0, "episodes": 16, "len_seed": 2, "chunk": 0},
        # a long-horizon agent: 32768 tokens kept, 4096 replayed in chunks of 512
        {"name": "replay_32k_chunk512_8b", "kind": "replay", "geometry": "8b", "dtype": "bf16",
         "t_lo": 36864, "t_hi": 36864, "keep": 0.888889, "episodes": 1, "len_seed": 0, "chunk": 512},
        # seven query heads to a KV head (rows that do not fill a matrix tile)
        {"name": "replay_7b_g7", "kind": "replay", "geometry": "7b_g7", "dtype": "bf16",
         "t_lo": 8190, "t_hi": 8190, "keep": 0.61, "episodes": 1, "len_seed": 0, "chunk": 0},
        # the cache kept in FP8, the benchmark's episode
        {"name": "replay_8b_fp8", "kind": "replay", "geometry": "8b", "dtype": "fp8",
         "t_lo": 10237, "t_hi": 10237, "keep": 0.79995, "episodes": 1, "len_seed": 0, "chunk": 0},
        # re-decode of 32 sessions in step, 8192 tokens cached for each
        {"name": "decode_b32_8k", "kind": "decode", "geometry": "8b", "dtype": "bf16",
         "ctx_lo": 8192, "ctx_hi": 8192, "seqs": 32, "len_seed": 0},
        # the same with an FP8 cache and sessions of different lengths
        {"name": "decode_b32_ragged_fp8", "kind": "decode", "geometry": "8b", "dtype": "fp8",
         "ctx_lo": 1024, "ctx_hi": 16384, "seqs": 32, "len_seed": 3},
        # an episode of the paper's scale, 1330 tokens with the target near the end: whole layers
        {"name": "decoder_paper_102", "kind": "decoder", "geometry": "8b", "layers": 4, "prefix": 1228,
         "tokens": 102, "workspace": False},
        # one re-decoded token of such an episode through whole layers
        {"name": "decoder_redecode_1", "kind": "decoder", "geometry": "8b", "layers": 4, "prefix": 1330,
         "tokens": 1, "workspace": True},
        # projections, norms, rotary embedding and MLP of one layer for a long replayed suffix
        {"name": "dense_8b_2048", "kind": "dense", "geometry": "8b", "tokens": 2048},
        # next tokens of 32 sessions over a 128256-entry vocabulary
        {"name": "sample_b32", "kind": "sample", "rows": 32, "vocab": 128256, "dtype": "bf16",
         "temperature": 0.7},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["replay", "replay", "replay", "chunked", "decode", "decode", "decoder", "decoder",
                       "dense", "sample"])
    if kind == "replay":
        dtype = rng.choice(["bf16", "bf16", "fp8", "f32"])
        if dtype == "f32":
            t = _log_int(rng, 100, 3000)
            return {"kind": "replay", "geometry": "mha8_d64", "dtype": "f32", "t_lo": t, "t_hi": t,
                    "keep": rng.uniform(0.1, 0.95), "episodes": 1, "len_seed": 0, "chunk": 0}
        episodes = _log_int(rng, 1, 12)
        t = _log_int(rng, 300, 12000)
        return {"kind": "replay", "geometry": rng.choice(["8b", "8b", "70b", "7b_g7"]) if episodes <= 4 else "8b",
                "dtype": dtype, "t_lo": max(200, int(t * rng.uniform(0.3, 1.0))), "t_hi": t,
                "keep": rng.choice([0.0, rng.uniform(0.1, 0.95)]), "episodes": episodes,
                "len_seed": rng.randrange(1000), "chunk": 0}
    if kind == "chunked":
        t = _log_int(rng, 3000, 36000)
        return {"kind": "replay", "geometry": rng.choice(["8b", "7b_g7"]), "dtype": "bf16", "t_lo": t, "t_hi": t,
                "keep": 1.0 - rng.uniform(0.3, 1.0) * min(0.5, 4096 / t), "episodes": 1, "len_seed": 0,
                "chunk": rng.choice([256, 500, 512, 1024])}
    if kind == "decode":
        seqs = _log_int(rng, 1, 80)
        ctx = _log_int(rng, 300, min(32000, 400000 // seqs))
        return {"kind": "decode", "geometry": rng.choice(["8b", "8b", "70b", "7b_g7"]),
                "dtype": rng.choice(["bf16", "fp8"]), "ctx_lo": max(100, int(ctx * rng.uniform(0.1, 1.0))),
                "ctx_hi": ctx, "seqs": seqs, "len_seed": rng.randrange(1000)}
    if kind == "decoder":
        return {"kind": "decoder", "geometry": rng.choice(["8b", "8b", "7b_g7"]), "layers": rng.choice([1, 2, 4]),
                "prefix": _log_int(rng, 100, 6000), "tokens": _log_int(rng, 1, 600),
                "workspace": rng.random() < 0.5}
    if kind == "dense":
        return {"kind": "dense", "geometry": rng.choice(["8b", "70b", "7b_g7"]), "tokens": _log_int(rng, 16, 3000)}
    return {"kind": "sample", "rows": _log_int(rng, 1, 100), "vocab": _log_int(rng, 2000, 152064),
            "dtype": rng.choice(["bf16", "f32"]), "temperature": rng.choice([0.0, 0.7, 1.0])}


# --------------------------------------------------------------------------- #
# inputs                                                                       #
# --------------------------------------------------------------------------- #
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)


def _randn(g, *shape, dtype=torch.bfloat16, scale=1.0):
    return (torch.randn(*shape, device="cuda", generator=g) * scale).to(dtype)


def _lengths(case):
    """Per episode (tokens kept, tokens replayed)."""
    r = random.Random(case["len_seed"])
    out = []
    for _ in range(case["episodes"]):
        t = r.randint(case["t_lo"], case["t_hi"])
        keep = case["keep"] or r.uniform(0.1, 0.9)
        p = min(t - 1, int(keep * t))
        out.append((p, t - p))
    return out


def _contexts(case):
    r = random.Random(case["len_seed"])
    return [r.randint(case["ctx_lo"], case["ctx_hi"]) for _ in range(case["seqs"])]


def _element(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _episode(case, seed, i, p, s):
    """Episode i: K, V of the kept prefix, q, k, v of the sanitized suffix and K, V of the contaminated one."""
    hq, hkv, d = GEOMETRY[case["geometry"]][:3]
    g, dt = _generator(seed * 64 + i), _element(case)
    new = lambda n, h: _randn(g, n, h, d, dtype=dt)  # noqa: E731
    return {"kp": new(p, hkv), "vp": new(p, hkv), "q": new(s, hq), "k": new(s, hkv), "v": new(s, hkv),
            "kc": new(s + 3, hkv), "vc": new(s + 3, hkv)}


def _decode_sequence(case, seed, i, ctx):
    hkv, d = GEOMETRY[case["geometry"]][1:3]
    g = _generator(seed * 64 + i)
    return _randn(g, ctx, hkv, d), _randn(g, ctx, hkv, d)


def _decode_step(case, seed):
    hq, hkv, d = GEOMETRY[case["geometry"]][:3]
    g, n = _generator(seed + 500009), case["seqs"]
    return _randn(g, n, hq, d), _randn(g, n, hkv, d), _randn(g, n, hkv, d)


def _layer_weights(geometry, g):
    hq, hkv, d, dm, dff = GEOMETRY[geometry]
    gain = lambda: (1 + 0.1 * torch.randn(dm, device="cuda", generator=g)).to(torch.bfloat16)  # noqa: E731
    return {"wq": _randn(g, hq * d, dm, scale=dm ** -0.5), "wk": _randn(g, hkv * d, dm, scale=dm ** -0.5),
            "wv": _randn(g, hkv * d, dm, scale=dm ** -0.5), "wo": _randn(g, dm, hq * d, scale=(hq * d) ** -0.5),
            "w_gate_up": _randn(g, 2 * dff, dm, scale=dm ** -0.5), "w_down": _randn(g, dm, dff, scale=dff ** -0.5),
            "g_attn": gain(), "g_mlp": gain()}


def _decoder_inputs(case, seed):
    """Weights, states of the kept tokens, of the contaminated suffix and of the sanitized one."""
    g, dm = _generator(seed), GEOMETRY[case["geometry"]][3]
    weights = [_layer_weights(case["geometry"], g) for _ in range(case["layers"])]
    return (weights, _randn(g, case["prefix"], dm), _randn(g, case["tokens"] + 3, dm),
            _randn(g, case["tokens"], dm))


def _dense_inputs(case, seed):
    g = _generator(seed)
    hq, _, d, dm, _ = GEOMETRY[case["geometry"]]
    n = case["tokens"]
    return (_layer_weights(case["geometry"], g), _randn(g, n, dm), _randn(g, n, hq * d, scale=0.05),
            torch.arange(1000, 1000 + n, dtype=torch.int32, device="cuda"))


# --------------------------------------------------------------------------- #
# prepare                                                                      #
# --------------------------------------------------------------------------- #
def _pool(case, lengths, n_seqs, workspace):
    hq, hkv, d = GEOMETRY[case["geometry"]][:3]
    blocks = [-(-n // BLOCK) + 1 for n in lengths]
    pool = KVPool(1, hq, hkv, d, sum(blocks) + 8, n_seqs, max(blocks) + 2, POOL_DTYPE[case["dtype"]], BLOCK,
                  workspace_bytes=workspace)
    if case["dtype"] == "fp8":
        pool.set_kv_scales([KV_SCALE], [KV_SCALE])
    return pool


def _fill(pool, seq, k, v, scale):
    """The run that filled the cache; what it attended to is over."""
    q = torch.zeros(k.shape[0], pool.hq, pool.d, dtype=k.dtype, device="cuda")
    if pool.replay(0, [seq], [k.shape[0]], q, k.contiguous(), v.contiguous(), torch.empty_like(q), scale):
        raise RuntimeError("prefill failed")


def prepare(case, seed):
    kind = case["kind"]
    if kind == "replay":
        hq, hkv, d = GEOMETRY[case["geometry"]][:3]
        lens = _lengths(case)
        total = sum(s for _, s in lens)
        # a program gives the pool a workspace where its calls are small
        small = case["chunk"] or (total if total * hq < 1 << 15 else 0)
        pool = _pool(case, [p + s + 3 for p, s in lens], len(lens), workspace_bytes(hq, d, small) if small else 0)
        q, k, v = [], [], []
        for i, (p, s) in enumerate(lens):
            e = _episode(case, seed, i, p, s)
            _fill(pool, i, torch.cat([e["kp"], e["kc"]]), torch.cat([e["vp"], e["vc"]]), d ** -0.5)
            q.append(e["q"])
            k.append(e["k"])
            v.append(e["v"])
        q, k, v = torch.cat(q), torch.cat(k), torch.cat(v)
        return {"case": case, "pool": pool, "q": q, "k": k, "v": v, "o": torch.empty_like(q),
                "keep": [p for p, _ in lens], "new": [s for _, s in lens], "scale": d ** -0.5}
    if kind == "decode":
        hq, hkv, d = GEOMETRY[case["geometry"]][:3]
        ctx = _contexts(case)
        pool = _pool(case, [c + 1 for c in ctx], len(ctx), workspace_bytes(hq, d, len(ctx), 32))
        for i, c in enumerate(ctx):
            _fill(pool, i, *_decode_sequence(case, seed, i, c), d ** -0.5)
        q, k, v = _decode_step(case, seed)
        return {"case": case, "pool": pool, "q": q, "k": k, "v": v, "o": torch.empty_like(q),
                "seqs": list(range(len(ctx))), "new": [1] * len(ctx), "scale": d ** -0.5}
    if kind == "decoder":
        hq, hkv, d = GEOMETRY[case["geometry"]][:3]
        weights, xp, xc, xs = _decoder_inputs(case, seed)
        blocks = -(-(case["prefix"] + case["tokens"] + 3) // BLOCK)
        dec = DecoderReplay(weights, hq, hkv, d, EPS, THETA, blocks + 8, 1, blocks + 4, BLOCK,
                            workspace_bytes=workspace_bytes(hq, d, case["tokens"], 32) if case["workspace"] else 0)
        dec.replay(0, torch.cat([xp, xc]))
        return {"case": case, "decoder": dec, "x": xs}
    if kind == "dense":
        w, x, attended, positions = _dense_inputs(case, seed)
        return {"case": case, "w": w, "x": x, "attended": attended, "positions": positions}
    g, rows, vocab = _generator(seed), case["rows"], case["vocab"]
    # a language model's logits: a wide body and some tens of likely tokens
    logits = 2.0 * torch.randn(rows, vocab, device="cuda", generator=g)
    likely = torch.randint(vocab, (rows, 32), device="cuda", generator=g)
    logits.scatter_add_(1, likely, 12.0 * torch.rand(rows, 32, device="cuda", generator=g))
    return {"case": case, "logits": logits.to(torch.float32 if case["dtype"] == "f32" else torch.bfloat16),
            "streams": list(range(rows)), "positions": [1000 + 7 * i for i in range(rows)], "seed": int(seed),
            "tokens": torch.empty(rows, dtype=torch.int32, device="cuda"),
            "workspace": torch.empty(max(sample_workspace_bytes(rows, vocab), 1), dtype=torch.uint8, device="cuda")}


# --------------------------------------------------------------------------- #
# run                                                                          #
# --------------------------------------------------------------------------- #
def _state_of(pool):
    return {"k_cache": pool.k_cache, "v_cache": pool.v_cache, "tables": pool.block_tables, "lens": pool.seq_lens,
            "free_top": pool.free_top}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "replay":
        pool, q, k, v, o = (state[n] for n in ("pool", "q", "k", "v", "o"))
        if case["chunk"]:
            total = state["new"][0]
            for c in range(0, total, case["chunk"]):
                n = min(case["chunk"], total - c)
                part = slice(c, c + n)
                if c == 0:
                    rc = pool.restore_replay(0, [0], state["keep"], [n], q[part], k[part], v[part], o[part],
                                             state["scale"])
                else:
                    rc = pool.replay(0, [0], [n], q[part], k[part], v[part], o[part], state["scale"])
                if rc:
                    raise RuntimeError("replay failed")
        elif pool.restore_replay(0, list(range(len(state["keep"]))), state["keep"], state["new"], q, k, v, o,
                                 state["scale"]):
            raise RuntimeError("restore + replay failed")
        return {"o": o, **_state_of(pool)}
    if kind == "decode":
        pool = state["pool"]
        if pool.replay(0, state["seqs"], state["new"], state["q"], state["k"], state["v"], state["o"],
                       state["scale"], commit=False):
            raise RuntimeError("decode step failed")
        return {"o": state["o"], **_state_of(pool)}
    if kind == "decoder":
        dec = state["decoder"]
        if dec.crop([0], [case["prefix"]]):
            raise RuntimeError("crop failed")
        return {"x": dec.replay(0, state["x"]), **_state_of(dec.pool)}
    if kind == "dense":
        w, x = state["w"], state["x"]
        hq, hkv, d = GEOMETRY[case["geometry"]][:3]
        n = x.shape[0]
        h = rmsnorm(x, w["g_attn"], EPS)
        q = rope_(gemm_bf16(h, w["wq"]).view(n, hq, d), state["positions"], THETA)
        k = rope_(gemm_bf16(h, w["wk"]).view(n, hkv, d), state["positions"], THETA)
        v = gemm_bf16(h, w["wv"])
        x1 = gemm_bf16(state["attended"], w["wo"], r=x)
        a = silu_mul(gemm_bf16(rmsnorm(x1, w["g_mlp"], EPS), w["w_gate_up"]))
        return {"q": q, "k": k, "v": v, "x1": x1, "a": a, "x2": gemm_bf16(a, w["w_down"], r=x1)}
    return {"tokens": sample_tokens(state["logits"], case["temperature"], state["seed"], state["streams"],
                                    state["positions"], out=state["tokens"], workspace=state["workspace"])}


# --------------------------------------------------------------------------- #
# work, tolerance                                                              #
# --------------------------------------------------------------------------- #
def _layer_parameters(geometry):
    hq, hkv, d, dm, dff = GEOMETRY[geometry]
    return dm * (hq + 2 * hkv) * d + hq * d * dm + 3 * dm * dff


def work(case):
    kind = case["kind"]
    if kind == "sample":
        n = case["rows"] * case["vocab"]
        return {"bytes": n * (4 if case["dtype"] == "f32" else 2), "flops": 2 * n}
    hq, hkv, d, dm, dff = GEOMETRY[case["geometry"]]
    if kind == "replay":
        eb = 4 if case["dtype"] == "f32" else 2
        cb = {"f32": 4, "bf16": 2, "fp8": 1}[case["dtype"]]
        b = f = 0.0
        for p, s in _lengths(case):
            f += 4.0 * hq * d * (s * p + s * (s + 1) / 2)
            # q and o, the prefix's K and V (once for each chunk), the suffix's K and V read and stored
            starts = range(0, s, case["chunk"]) if case["chunk"] else [0]
            b += 2 * s * hq * d * eb + sum(2 * (p + c) * hkv * d * cb for c in starts) + 2 * s * hkv * d * (eb + cb)
        return {"bytes": b, "flops": f}
    if kind == "decode":
        cb, n, keys = (1 if case["dtype"] == "fp8" else 2), case["seqs"], sum(_contexts(case))
        return {"bytes": 2 * keys * hkv * d * cb + n * (2 * hq * d * 2 + 2 * hkv * d * (2 + cb)),
                "flops": 4.0 * hq * d * (keys + n)}
    n, params = case["tokens"], _layer_parameters(case["geometry"])
    if kind == "dense":
        out = n * ((hq + 2 * hkv) * d + 2 * dm + dff)
        return {"bytes": 2 * (params + 2 * dm + n * (dm + hq * d) + out), "flops": 2.0 * n * params}
    p = case["prefix"]
    return {"bytes": case["layers"] * 2 * (params + 2 * dm + 2 * (p + n) * hkv * d) + 2 * 2 * n * dm,
            "flops": case["layers"] * (2.0 * n * params + 4.0 * hq * d * (n * p + n * (n + 1) / 2))}


def tolerance(case):
    kind = case["kind"]
    if kind == "sample":
        return "exact"
    if kind == "replay" and case["dtype"] == "f32":     # measured 2.3e-7 from 64 bits
        return {"rel": 2e-6, "max": 2e-5}
    if kind == "decoder":                               # measured 7e-3: each layer rounds what the next one reads
        return {"rel": 2.5e-2, "max": 0.5}
    # bf16 storage (the result, each softmax weight, each stored value of a block): measured 2.3e-3 to 4.6e-3
    return {"rel": 1.2e-2, "max": 0.25}


# --------------------------------------------------------------------------- #
# exact                                                                        #
# --------------------------------------------------------------------------- #
def _attention64(q, k, v, prefix, scale):
    """q [s, hq, d] at positions prefix + i against k, v [prefix + s, hkv, d], in 64 bits."""
    s, hq, d = q.shape
    hkv = k.shape[1]
    group = hq // hkv
    out = torch.empty(s, hq, d, dtype=torch.float64, device=q.device)
    step = max(1, (1 << 27) // (group * k.shape[0]))
    for h in range(hkv):
        kh, vh = k[:, h].double().contiguous(), v[:, h].double().contiguous()
        for a in range(0, s, step):
            b = min(s, a + step)
            end = prefix + b
            rows = q[a:b, h * group:(h + 1) * group].double().reshape(-1, d)
            score = torch.matmul(rows, kh[:end].t().contiguous()).mul_(scale).view(b - a, group, end)
            pos = prefix + torch.arange(a, b, device=q.device)
            score.masked_fill_((torch.arange(end, device=q.device)[None, :] > pos[:, None])[:, None, :], -math.inf)
            weight = torch.softmax(score.view(-1, end), dim=-1)
            out[a:b, h * group:(h + 1) * group] = torch.matmul(weight, vh[:end]).view(b - a, group, d)
    return out


def _stored(case, x):
    """What the cache gives back for x."""
    if case["dtype"] != "fp8":
        return x
    scale = torch.tensor(KV_SCALE, dtype=torch.float32, device=x.device)
    # magnitudes past the largest code saturate
    return (x.float() / scale).clamp(-448, 448).to(torch.float8_e4m3fn).double() * scale.double()


def _norm64(x, gain):
    return x / torch.sqrt(x.square().mean(dim=-1, keepdim=True) + EPS) * gain.double()


def _rope64(x, positions):
    d = x.shape[-1]
    half = d // 2
    rate = THETA ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / d)
    angle = positions.double()[:, None, None] * rate
    a, b, c, s = x[..., :half], x[..., half:], torch.cos(angle), torch.sin(angle)
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _mlp64(x, w):
    gate, up = torch.matmul(_norm64(x, w["g_mlp"]), w["w_gate_up"].double().t()).chunk(2, dim=-1)
    a = gate / (1 + torch.exp(-gate)) * up
    return a, x + torch.matmul(a, w["w_down"].double().t())


def exact(case, seed):
    kind = case["kind"]
    if kind == "sample":
        return None
    hq, hkv, d = GEOMETRY[case["geometry"]][:3]
    state = {"k_cache": None, "v_cache": None, "tables": None, "lens": None, "free_top": None}
    if kind == "replay":
        outs = []
        for i, (p, s) in enumerate(_lengths(case)):
            e = _episode(case, seed, i, p, s)
            outs.append(_attention64(e["q"], _stored(case, torch.cat([e["kp"], e["k"]])),
                                     _stored(case, torch.cat([e["vp"], e["v"]])), p, d ** -0.5))
        return {"o": torch.cat(outs), **state}
    if kind == "decode":
        q, k, v = _decode_step(case, seed)
        outs = []
        for i, c in enumerate(_contexts(case)):
            kc, vc = _decode_sequence(case, seed, i, c)
            outs.append(_attention64(q[i:i + 1], _stored(case, torch.cat([kc, k[i:i + 1]])),
                                     _stored(case, torch.cat([vc, v[i:i + 1]])), c, d ** -0.5))
        return {"o": torch.cat(outs), **state}
    if kind == "dense":
        w, x, attended, positions = _dense_inputs(case, seed)
        n = x.shape[0]
        x64 = x.double()
        h = _norm64(x64, w["g_attn"])
        q, k, v = (torch.matmul(h, w[m].double().t()) for m in ("wq", "wk", "wv"))
        x1 = x64 + torch.matmul(attended.double(), w["wo"].double().t())
        a, x2 = _mlp64(x1, w)
        return {"q": _rope64(q.view(n, hq, d), positions), "k": _rope64(k.view(n, hkv, d), positions), "v": v,
                "x1": x1, "a": a, "x2": x2}
    weights, xp, _, xs = _decoder_inputs(case, seed)
    x = torch.cat([xp, xs]).double()
    n = x.shape[0]
    positions = torch.arange(n, device="cuda")
    for w in weights:
        h = _norm64(x, w["g_attn"])
        q, k, v = (torch.matmul(h, w[m].double().t()) for m in ("wq", "wk", "wv"))
        o = _attention64(_rope64(q.view(n, hq, d), positions), _rope64(k.view(n, hkv, d), positions),
                         v.view(n, hkv, d), 0, d ** -0.5)
        x = x + torch.matmul(o.view(n, hq * d), w["wo"].double().t())
        x = _mlp64(x, w)[1]
    return {"x": x[case["prefix"]:], **state}
