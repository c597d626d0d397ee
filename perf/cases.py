"""The framework's performance cases: what a program asks of it, over the real range of sizes.

A case is one pass through public entry points: a whole call (reuse prefill, caching of a
memory unit, decode step) or the step entries of one layer that a serving loop of its own
would call (projections, attention, check layer, correction, quantiser, LM head). The model
widths are those of the benchmark's workloads; depth is cut where one layer is like the next.

prepare() makes a case's inputs on the GPU from its seed, run() is the timed pass, exact()
the same outputs in plain torch in 64 bits.
"""
import math
from dataclasses import dataclass

import numpy as np
import torch

from paper_2607_21604_amd import akvs, runtime

DEV = "cuda"


@dataclass(frozen=True)
class Shape:
    n_layers: int
    d_model: int
    n_q_heads: int
    n_kv_heads: int
    head_dim: int
    ffn_dim: int
    vocab: int
    rope_theta: float
    rms_eps: float = 1e-6
    dtype: str = "bf16"

    @property
    def hqw(self):
        return self.n_q_heads * self.head_dim

    @property
    def kvw(self):
        return self.n_kv_heads * self.head_dim


# decoder widths of the benchmark's workloads
SHAPES = {
    "tiny": dict(d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, ffn_dim=688, vocab=1024,
                 rope_theta=1.0e4, dtype="f32"),
    "3b": dict(d_model=3072, n_q_heads=24, n_kv_heads=8, head_dim=128, ffn_dim=8192,
               vocab=128256, rope_theta=1.0e6),
    "7b": dict(d_model=3584, n_q_heads=28, n_kv_heads=4, head_dim=128, ffn_dim=18944,
               vocab=152064, rope_theta=1.0e6),
    "32b": dict(d_model=5120, n_q_heads=40, n_kv_heads=8, head_dim=128, ffn_dim=27648,
                vocab=152064, rope_theta=1.0e6),
}
CODE = {16: akvs.AKVS_BF16, 4: akvs.AKVS_U4G64, 2: akvs.AKVS_U2G64, 8: akvs.AKVS_E4M3G64}


def _shape(case):
    return Shape(n_layers=case.get("layers", 1), **SHAPES[case["model"]])


def listed():
    return [
        # the smallest whole call: a two-layer fp32 decoder, 288 tokens; launches count
        dict(name="reuse-tiny-f32", kind="reuse", model="tiny", layers=2, units=4, unit_len=64,
             ragged=False, q=32, num=1, den=5, bits=32),
        # the product's headline call on the 3B workload at its default refresh ratio, at half
        # its depth (in bf16 a changed rounding grows with each layer that follows)
        dict(name="reuse-3b", kind="reuse", model="3b", layers=14, units=20, unit_len=223,
             ragged=True, q=64, num=1, den=5, bits=16),
        # caching one memory unit (each unit is prefilled alone, once, when it is written)
        dict(name="unit-3b", kind="unit", model="3b", layers=4, n=203, pos0=0),
        # a generated token after the reuse prefill: every weight is read for one row
        dict(name="decode-3b", kind="decode", model="3b", layers=14, past=4517),
        # one probe layer's projections at a 1 % refresh: few rows, the weights stream
        dict(name="proj-3b-few", kind="proj", model="3b", rows=173),
        # the same at the largest workload's 20 % refresh: the matrix cores' case
        dict(name="proj-32b", kind="proj", model="32b", rows=5534),
        # a probe layer's attention over the whole context, 3B and the largest workload
        dict(name="attn-3b", kind="attn", model="3b", rows=1413, q=64, keys=4516),
        dict(name="attn-32b", kind="attn", model="32b", rows=5534, q=128, keys=16128),
        # the check layer's divergences and the probe selection over 80 units
        dict(name="check-32b", kind="check", model="32b", units=80, unit_len=200, ragged=False,
             q=128, num=1, den=5, bits=16),
        # one layer's offsets and corrected caches from a 4-bit unit cache
        dict(name="correct-7b-4bit", kind="correct", model="7b", units=40, unit_len=200,
             ragged=False, q=128, num=1, den=5, bits=4),
        # quantising the unit caches of a whole 7B model (keys or values) to 4 bits
        dict(name="quantize-7b", kind="quantize", model="7b", tokens=28 * 8000, bits=4),
        # first tokens of a batch of 16 requests
        dict(name="lm-head-3b", kind="head", model="3b", rows=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["reuse", "reuse", "tiny", "unit", "decode", "proj", "proj", "attn", "attn",
                       "check", "correct", "quantize", "head"])
    model = rng.choice(["3b", "7b", "32b"])
    num, den = rng.choice([(1, 100), (1, 20), (1, 10), (1, 5), (3, 10), (1, 2)])
    units = dict(units=_log(rng, 3, 80), unit_len=rng.randint(100, 256),
                 ragged=rng.random() < 0.7, q=_log(rng, 9, 128), num=num, den=den)
    if kind == "tiny":
        return dict(kind="reuse", model="tiny", layers=2, units=rng.randint(2, 8),
                    unit_len=rng.randint(40, 128), ragged=True, q=_log(rng, 9, 64), num=num,
                    den=den, bits=32)
    if kind == "reuse":
        units["units"] = _log(rng, 3, 30)
        return dict(kind=kind, model=rng.choice(["3b", "7b"]), layers=4,
                    bits=rng.choice([16, 16, 8, 4, 2]), **units)
    if kind == "unit":
        return dict(kind=kind, model=rng.choice(["3b", "7b"]), layers=4, n=_log(rng, 17, 520),
                    pos0=rng.choice([0, 0, 411]))
    if kind == "decode":
        return dict(kind=kind, model=model, layers=4, past=_log(rng, 60, 16500))
    if kind == "proj":
        return dict(kind=kind, model=model, rows=_log(rng, 33, 5534))
    if kind == "attn":
        keys = _log(rng, 500, 16128)
        rows = min(keys, max(9, _log(rng, max(9, keys // 100), max(10, keys // 3))))
        return dict(kind=kind, model=model, rows=rows, q=min(rows, _log(rng, 9, 128)), keys=keys)
    if kind == "check":
        return dict(kind=kind, model=model, bits=rng.choice([16, 16, 8, 4, 2]), **units)
    if kind == "correct":
        return dict(kind=kind, model=model, bits=rng.choice([16, 16, 8, 4, 2]), **units)
    if kind == "quantize":
        return dict(kind=kind, model=model, tokens=_log(rng, 200, 28 * 4000),
                    bits=rng.choice([2, 4, 8]))
    return dict(kind=kind, model=model, rows=_log(rng, 1, 64))


# ---- inputs --------------------------------------------------------------------------------


def _lens(case):
    n, base = case["units"], case["unit_len"]
    return [base + ((37 * i) % 65 - 32 if case["ragged"] else 0) for i in range(n)]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std, dtype):
    """N(0, std^2) values; tensors of over 2^29 elements are drawn in slices."""
    t = torch.empty(shape, dtype=dtype, device=DEV)
    f = t.view(-1)
    for a in range(0, f.numel(), 1 << 29):
        b = min(f.numel(), a + (1 << 29))
        f[a:b].copy_(torch.empty(b - a, device=DEV).normal_(0.0, std, generator=g))
    return t


def _layer(sh, g):
    dt = torch.float32 if sh.dtype == "f32" else torch.bfloat16
    D, F = sh.d_model, sh.ffn_dim
    gain = lambda: (1.0 + 0.1 * torch.randn(D, generator=g, device=DEV)).to(dt)  # noqa: E731
    return {"attn_norm": gain(), "w_qkv": _normal(g, (sh.hqw + 2 * sh.kvw, D), 0.02, dt),
            "w_o": _normal(g, (D, sh.hqw), 0.02, dt), "mlp_norm": gain(),
            "w_gate_up": _normal(g, (2 * F, D), 0.02, dt),
            "w_down": _normal(g, (D, F), 0.02, dt)}


def _engine(sh, g):
    dt = torch.float32 if sh.dtype == "f32" else torch.bfloat16
    w = {"embed": _normal(g, (sh.vocab, sh.d_model), 0.02, dt),
         "final_norm": (1.0 + 0.1 * torch.randn(sh.d_model, generator=g, device=DEV)).to(dt),
         "layers": [_layer(sh, g) for _ in range(sh.n_layers)]}
    return runtime.Engine(sh, w, DEV)


def _cache(sh, g, lead, bits):
    """A unit cache side [*lead][Hkv][hd]: the values (or codes) and the groups' metadata.
    Keys and values of these decoders have a standard deviation near one."""
    hd, hkv = sh.head_dim, sh.n_kv_heads
    if bits in (16, 32):
        dt = torch.float32 if bits == 32 else torch.bfloat16
        return _normal(g, (*lead, hkv, hd), 1.0, dt), None
    codes = torch.randint(0, 256, (*lead, hkv, hd * bits // 8), generator=g, device=DEV,
                          dtype=torch.uint8)
    scale = 0.9 + 0.2 * torch.rand((*lead, hkv, hd // 64, 1), generator=g, device=DEV)
    if bits == 8:  # E4M3 magnitudes up to 448 stand for the group's largest value (about 2.5)
        codes = torch.where((codes & 0x7F) == 0x7F, codes & 0x80, codes)
        scale, zero = scale * (2.5 / 448), torch.zeros_like(scale)
    else:
        scale = scale * (5.0 / (2 ** bits - 1))
        zero = -2.5 + 0.1 * torch.randn(scale.shape, generator=g, device=DEV)
    return codes, torch.cat([scale, zero], dim=-1).to(torch.float16).contiguous()


def _probes(case, rng, lens):
    """Random probe sets of both sides, ascending, units back to back."""
    pk, pv, s = [], [], 0
    for n in lens:
        b = -(-case["num"] * n // case["den"])
        for out in (pk, pv):
            out.append(s + np.sort(rng.permutation(n)[:b]))
        s += n
    cat = lambda v: np.concatenate(v).astype(np.int32)  # noqa: E731
    return cat(pk), cat(pv)


def _int(a):
    return torch.tensor(np.asarray(a), dtype=torch.int32, device=DEV)


def _rope(sh, n):
    t = torch.empty((n, sh.head_dim // 2, 2), dtype=torch.float32, device=DEV)
    akvs.akvs_rope_table(n, sh.head_dim, sh.rope_theta, t)
    return t


def prepare(case, seed):
    sh, g, rng = _shape(case), _gen(seed), np.random.default_rng(int(seed))
    m = akvs.model_cfg(sh)
    s = {"kind": case["kind"], "case": dict(case), "sh": sh, "m": m}
    kind, D, hd, hkv = case["kind"], sh.d_model, sh.head_dim, sh.n_kv_heads
    dt = torch.float32 if sh.dtype == "f32" else torch.bfloat16
    empty = lambda *shape, d=dt: torch.empty(shape, dtype=d, device=DEV)  # noqa: E731
    if kind in ("reuse", "check", "correct"):
        s["lens"] = lens = _lens(case)
        tc = sum(lens)
        T = tc + case["q"]
    if kind in ("reuse", "unit", "decode"):
        s["eng"] = _engine(sh, g)
    if kind == "reuse":
        s["tokens"] = torch.randint(0, sh.vocab, (T,), generator=g, device=DEV, dtype=torch.int32)
        s["k"], s["k_meta"] = _cache(sh, g, (sh.n_layers, tc), case["bits"])
        s["v"], s["v_meta"] = _cache(sh, g, (sh.n_layers, tc), case["bits"])
        # the probe sets are given, as when a request is repeated: what follows from the
        # sets is then comparable (near ties of computed divergences may fall either way)
        pk, pv = _probes(case, rng, lens)
        s["out"] = {"h_query": empty(case["q"], D, d=torch.float32),
                    "k_corr": empty(sh.n_layers, T, hkv, hd),
                    "v_corr": empty(sh.n_layers, T, hkv, hd), "probe_k": _int(pk),
                    "probe_v": _int(pv), "d_k": empty(tc, d=torch.float32),
                    "d_v": empty(tc, d=torch.float32), "rows": empty(T, d=torch.int32),
                    "n_rows": empty(1, d=torch.int32)}
    elif kind == "unit":
        s["tokens"] = torch.randint(0, sh.vocab, (case["n"],), generator=g, device=DEV,
                                    dtype=torch.int32)
    elif kind == "decode":
        rows = case["past"] + 16  # room for the tokens to come
        s["token"] = torch.randint(0, sh.vocab, (1,), generator=g, device=DEV, dtype=torch.int32)
        s["k"] = _normal(g, (sh.n_layers, rows, hkv, hd), 1.0, dt)
        s["v"] = _normal(g, (sh.n_layers, rows, hkv, hd), 1.0, dt)
        s["logits"] = empty(sh.vocab, d=torch.float32)
        s["next"] = empty(1, d=torch.int32)
    elif kind == "proj":
        r = case["rows"]
        s["layer"] = lw = _layer(sh, g)
        s["lw"] = akvs.layer_array({"layers": [lw]})[0]
        s["h"] = _normal(g, (r, D), 1.0, torch.float32)
        s["att"] = _normal(g, (r, sh.hqw), 0.1, dt)
        n_pos = 4 * r  # recomputed rows: about a quarter of the context
        s["positions"] = _int(np.sort(rng.permutation(n_pos)[:r]))
        s["rope"] = _rope(sh, n_pos)
        s["q"], s["kf"], s["vf"] = empty(r, sh.hqw), empty(r, sh.kvw), empty(r, sh.kvw)
        s["ws"] = empty(akvs.akvs_step_workspace_size(m, r), d=torch.uint8)
    elif kind == "attn":
        r, q, n = case["rows"], case["q"], case["keys"]
        ctx = np.sort(rng.permutation(n - q)[:r - q])
        s["positions"] = _int(np.concatenate([ctx, np.arange(n - q, n)]))
        s["q"] = _normal(g, (r, sh.n_q_heads, hd), 1.0, dt)
        s["k"], s["v"] = (_normal(g, (n, hkv, hd), 1.0, dt) for _ in range(2))
        s["out"] = empty(r, sh.hqw)
        size = akvs.akvs_attention_workspace_size(m, r, n)
        s["ws"] = empty(size, d=torch.uint8) if size else None
    elif kind == "check":
        s["cfg"] = akvs.reuse_cfg(lens, case["q"], (case["num"], case["den"]))
        meta, (_, sb, cap, _, sbv) = akvs.akvs_chunk_meta(s["cfg"])
        s["meta"] = meta.to(DEV)
        s["k"], s["k_meta"] = _cache(sh, g, (tc,), case["bits"])
        s["v"], s["v_meta"] = _cache(sh, g, (tc,), case["bits"])
        starts = np.repeat(np.cumsum([0] + lens[:-1]), lens)
        s["delta"], s["rope"] = _int(starts), _rope(sh, T)
        # fresh states near the re-rotated cached ones: residuals of a third of their size
        kd, vd = (_dequant(sh, s[x], s[x + "_meta"], case["bits"]) for x in ("k", "v"))
        kd = _rotate(kd, _angles(sh, s["delta"]))
        s["kf"], s["vf"] = ((x + 0.3 * torch.randn(x.shape, generator=g, device=DEV)).to(dt)
                            for x in (kd, vd))
        f, i = torch.float32, torch.int32
        s["out"] = {"d_k": empty(tc, d=f), "d_v": empty(tc, d=f), "probe_k": empty(sb, d=i),
                    "probe_v": empty(sbv, d=i), "w_k": empty(tc, d=f), "w_v": empty(tc, d=f),
                    "flags": empty(tc, d=torch.uint8), "chunk_rows": empty(len(lens), d=i),
                    "rows": torch.zeros(cap, dtype=i, device=DEV), "n_rows": empty(1, d=i),
                    "fresh_row": empty(T, d=i)}
    elif kind == "correct":
        s["cfg"] = akvs.reuse_cfg(lens, case["q"], (case["num"], case["den"]))
        s["meta"] = akvs.akvs_chunk_meta(s["cfg"])[0].to(DEV)
        s["k"], s["k_meta"] = _cache(sh, g, (tc,), case["bits"])
        s["v"], s["v_meta"] = _cache(sh, g, (tc,), case["bits"])
        s["rope"] = _rope(sh, T)
        pk, pv = _probes(case, rng, lens)
        flags = np.zeros(tc, np.uint8)
        flags[pk] |= 1
        flags[pv] |= 2
        rows = np.concatenate([np.nonzero(flags)[0], np.arange(tc, T)])
        fresh = np.full(T, -1, np.int64)
        fresh[rows] = np.arange(len(rows))
        s["pk"], s["pv"], s["fresh_row"] = _int(pk), _int(pv), _int(fresh)
        s["flags"] = torch.tensor(flags, device=DEV)
        s["kf"], s["vf"] = (_normal(g, (len(rows), hkv, hd), 1.0, dt) for _ in range(2))
        s["wk"], s["wv"] = (torch.clamp(2 * torch.rand(tc, generator=g, device=DEV), max=1.0)
                            for _ in range(2))
        s["mu_k"], s["mu_v"] = (empty(len(lens), hkv, hd, d=torch.float32) for _ in range(2))
        s["k_corr"], s["v_corr"] = empty(T, hkv, hd), empty(T, hkv, hd)
    elif kind == "quantize":
        s["x"] = _normal(g, (case["tokens"], hkv, hd), 1.0, dt)
    elif kind == "head":
        s["h"] = _normal(g, (case["rows"], D), 1.0, torch.float32)
        s["w"] = _normal(g, (sh.vocab, D), 0.02, dt)
        s["logits"] = empty(case["rows"], sh.vocab, d=torch.float32)
        s["next"] = empty(case["rows"], d=torch.int32)
        s["ws"] = empty(akvs.akvs_decode_workspace_size(m, 0), d=torch.uint8)
    return s


# ---- the timed pass ------------------------------------------------------------------------


def run(s):
    kind, case, sh, m = s["kind"], s["case"], s["sh"], s["m"]
    hkv, hd = sh.n_kv_heads, sh.head_dim
    if kind == "reuse":
        out = s["eng"].reuse_prefill(
            s["tokens"], s["lens"], case["q"], s["k"], s["v"], refresh=(case["num"], case["den"]),
            flags=akvs.AKVS_F_GIVEN_PROBES, k_meta=s["k_meta"], v_meta=s["v_meta"],
            cache_dtype=CODE.get(case["bits"]), outputs=s["out"])
        return [out[x] for x in ("h_query", "k_corr", "v_corr", "d_k", "d_v", "n_rows")]
    if kind == "unit":
        return list(s["eng"].full_prefill(s["tokens"], case["pos0"]))
    if kind == "decode":  # (the greedy token of near-equal bf16 logits is not compared)
        s["eng"].decode_step(s["token"], case["past"], s["k"], s["v"], logits=s["logits"],
                             next_token=s["next"])
        n = case["past"] + 1
        return [s["logits"], s["k"][:, :n], s["v"][:, :n]]
    if kind == "proj":
        r = case["rows"]
        akvs.akvs_probe_qkv(s["h"], r, s["positions"], m, s["lw"], s["rope"], 4 * r, s["q"],
                            s["kf"], s["vf"], s["ws"])
        akvs.akvs_probe_out_mlp(s["h"], r, s["att"], m, s["lw"], s["ws"])
        return [s["q"], s["kf"], s["vf"], s["h"]]
    if kind == "attn":
        akvs.akvs_sparse_query_attention(s["q"], s["positions"], case["rows"], s["k"], s["v"],
                                         case["keys"], m, s["out"], s["ws"])
        return [s["out"]]
    if kind == "check":
        cache = akvs.cache_struct(s["k"], s["v"], s["k_meta"], s["v_meta"], CODE[case["bits"]])
        o = s["out"]
        akvs.akvs_check_divergence(s["kf"], s["vf"], akvs.AKVS_BF16, cache, int(s["k"].shape[0]),
                                   hkv, hd, s["delta"], s["rope"], int(s["rope"].shape[0]),
                                   o["d_k"], o["d_v"])
        akvs.akvs_select_probes(o["d_k"], o["d_v"], s["cfg"], s["meta"], o["probe_k"],
                                o["probe_v"], o["w_k"], o["w_v"], o["flags"], o["chunk_rows"],
                                o["rows"], o["n_rows"], o["fresh_row"])
        return [o["d_k"], o["d_v"], o["w_k"], o["w_v"], o["probe_k"], o["probe_v"], o["flags"],
                o["chunk_rows"], o["rows"], o["n_rows"], o["fresh_row"]]
    if kind == "correct":
        cache = akvs.cache_struct(s["k"], s["v"], s["k_meta"], s["v_meta"], CODE[case["bits"]])
        n_pos = int(s["rope"].shape[0])
        akvs.akvs_chunk_offset(s["kf"], s["vf"], s["fresh_row"], cache, s["cfg"], s["meta"],
                               s["pk"], s["pv"], m, s["rope"], n_pos, s["mu_k"], s["mu_v"])
        akvs.akvs_apply_correction(cache, s["mu_k"], s["mu_v"], s["wk"], s["wv"], s["flags"],
                                   s["kf"], s["vf"], s["fresh_row"], s["cfg"], s["meta"], m,
                                   s["rope"], n_pos, s["k_corr"], s["v_corr"])
        return [s["mu_k"], s["mu_v"], s["k_corr"], s["v_corr"]]
    if kind == "quantize":
        return list(runtime.quantize_cache(s["x"], case["bits"]))
    akvs.akvs_lm_head(s["h"], case["rows"], s["w"], m, s["logits"], s["next"], s["ws"])
    return [s["logits"], s["next"]]


# ---- what a pass cannot do without ---------------------------------------------------------


def _row_flops(sh):
    return 2 * (sh.d_model * (sh.hqw + 2 * sh.kvw) + sh.hqw * sh.d_model +
                3 * sh.ffn_dim * sh.d_model)


def _layer_weights(sh):
    return _row_flops(sh) // 2 * (4 if sh.dtype == "f32" else 2)


def _side_bytes(sh, tokens, bits):
    extra = sh.n_kv_heads * (sh.head_dim // 64) * 4 if bits < 16 else 0
    return tokens * (sh.kvw * bits // 8 + extra)


def work(case):
    sh, kind = _shape(case), case["kind"]
    es = 4 if sh.dtype == "f32" else 2
    L, D, F = sh.n_layers, sh.d_model, sh.ffn_dim
    if kind in ("reuse", "check", "correct"):
        lens = _lens(case)
        tc, q = sum(lens), case["q"]
        T = tc + q
        b = [-(-case["num"] * n // case["den"]) for n in lens]
        # distinct rows of two independent probe sets of each unit
        M = int(sum(n - (n - x) ** 2 / n for n, x in zip(lens, b))) + q
    if kind == "reuse":
        per_key = 4 * sh.hqw
        flops = T * _row_flops(sh) + per_key * T * (T + 1) / 2 + 4 * tc * D * sh.kvw
        flops += (L - 2) * (M * _row_flops(sh) + per_key * M * T / 2)
        flops += 2 * M * D * (sh.hqw + 2 * sh.kvw) + q * _row_flops(sh) + per_key * q * T
        byts = (L * (_layer_weights(sh) + 2 * T * sh.kvw * es) + q * D * 4 + T * D * es +
                2 * L * _side_bytes(sh, tc, case["bits"]))
    elif kind == "unit":
        n = case["n"]
        flops = L * (n * _row_flops(sh) + 2 * sh.hqw * n * (n + 1))
        byts = L * (_layer_weights(sh) + 2 * n * sh.kvw * es) + n * D * (4 + es)
    elif kind == "decode":
        n = case["past"] + 1
        flops = L * (_row_flops(sh) + 4 * sh.hqw * n) + 2 * sh.vocab * D
        byts = L * (_layer_weights(sh) + 2 * n * sh.kvw * es) + sh.vocab * (D * es + 4)
    elif kind == "proj":
        r = case["rows"]
        flops = r * _row_flops(sh)
        byts = _layer_weights(sh) + r * (8 * D + (2 * sh.hqw + 2 * sh.kvw) * es)
    elif kind == "attn":
        r, q, n = case["rows"], case["q"], case["keys"]
        flops = 4 * sh.hqw * ((r - q) * (n - q) / 2 + q * n)
        byts = (2 * r * sh.hqw + 2 * n * sh.kvw) * es
    elif kind == "check":
        flops = 10 * tc * sh.kvw
        byts = 2 * tc * sh.kvw * es + 2 * _side_bytes(sh, tc, case["bits"]) + 30 * tc
    elif kind == "correct":
        flops = 10 * tc * sh.kvw
        # offsets read the probes' cached rows, the correction the reused ones
        byts = 2 * _side_bytes(sh, tc, case["bits"]) + 2 * (T + M) * sh.kvw * es + 13 * T
    elif kind == "quantize":
        flops = 6 * case["tokens"] * sh.kvw
        byts = case["tokens"] * sh.kvw * es + _side_bytes(sh, case["tokens"], case["bits"])
    else:
        flops = 2 * case["rows"] * sh.vocab * D
        byts = sh.vocab * D * es + case["rows"] * (4 * D + 4 * sh.vocab)
    return {"bytes": int(byts), "flops": int(flops)}


def tolerance(case):
    kind = case["kind"]
    if kind == "quantize":
        return "exact"  # codes and fp16 metadata
    # about four times what was measured against exact(): 6e-7 for the fp32 decoder, 1.4e-7
    # for the fp32 logits, 4e-8 for the divergences; in bf16 2e-3 for one layer's outputs and
    # 1e-2 to 2e-2 at the end of 4 to 14 layers
    if case["model"] == "tiny":
        return {"rel": 4e-6, "max": 1e-3}
    return {"reuse": {"rel": 3e-2}, "unit": {"rel": 3e-2}, "decode": {"rel": 3e-2},
            "proj": {"rel": 1e-2}, "attn": {"rel": 1e-2},
            "check": {"rel": 1e-6, "differ": 1e-3}, "correct": {"rel": 6e-3},
            "head": {"rel": 2e-6}}[kind]


# ---- the same in 64 bits -------------------------------------------------------------------


def _dequant(sh, x, meta, bits):
    """A cache side in 64 bits, [..][Hkv][hd]."""
    if bits in (16, 32):
        return x.double()
    if bits == 8:
        v = x.view(torch.float8_e4m3fn).to(torch.float64)
    else:
        per = 8 // bits
        sh_ = torch.arange(per, device=DEV, dtype=torch.int32) * bits
        v = ((x.to(torch.int32).unsqueeze(-1) >> sh_) & (2 ** bits - 1)).flatten(-2).double()
    mt = meta.double().repeat_interleave(64, dim=-2)
    return v * mt[..., 0] + mt[..., 1]


def _angles(sh, pos):
    half = sh.head_dim // 2
    inv = sh.rope_theta ** (-torch.arange(half, device=DEV, dtype=torch.float64) / half)
    a = pos.double()[:, None] * inv
    return torch.cos(a)[:, None, :], torch.sin(a)[:, None, :]


def _rotate(x, cs):
    lo, hi = x.chunk(2, dim=-1)
    return torch.cat([lo * cs[0] - hi * cs[1], hi * cs[0] + lo * cs[1]], dim=-1)


def _norm(h, gain, eps):
    return h * torch.rsqrt(h.square().mean(-1, keepdim=True) + eps) * gain.double()


def _qkv(sh, h, lw, pos):
    x = _norm(h, lw["attn_norm"], sh.rms_eps) @ lw["w_qkv"].double().T
    q, k, v = x.split([sh.hqw, sh.kvw, sh.kvw], dim=-1)
    cs = _angles(sh, pos)
    heads = lambda t: t.view(len(t), -1, sh.head_dim)  # noqa: E731
    return _rotate(heads(q), cs), _rotate(heads(k), cs), heads(v)


def _attend(sh, q, pos, k, v):
    out = torch.empty_like(q)
    G = sh.n_q_heads // sh.n_kv_heads
    hidden = torch.arange(len(k), device=DEV)[None, :] > pos[:, None]
    for h in range(sh.n_q_heads):
        s = q[:, h] @ k[:, h // G].T / math.sqrt(sh.head_dim)
        out[:, h] = torch.softmax(s.masked_fill_(hidden, -math.inf), dim=-1) @ v[:, h // G]
    return out.flatten(1)


def _out_mlp(sh, h, att, lw):
    h = h + att @ lw["w_o"].double().T
    g, u = (_norm(h, lw["mlp_norm"], sh.rms_eps) @ lw["w_gate_up"].double().T).chunk(2, dim=-1)
    return h + (torch.nn.functional.silu(g) * u) @ lw["w_down"].double().T


def _offset(fresh, fresh_row, cached, probes, lens, num_den):
    """Mean of fresh minus (re-rotated) cached over each unit's probes."""
    num, den = num_den
    out, at = [], 0
    for n in lens:
        b = -(-num * n // den)
        p = probes[at:at + b].long()
        out.append((fresh[fresh_row[p].long()] - cached[p]).mean(0))
        at += b
    return torch.stack(out)


def _correct(s, kd, vd, kf, vf, fresh_row, pk, pv, wk, wv):
    """(offsets, corrected keys and values) from dequantised caches and fresh rows."""
    case, lens = s["case"], s["lens"]
    tc, nd = sum(lens), (case["num"], case["den"])
    unit = torch.tensor(np.repeat(np.arange(len(lens)), lens), device=DEV)
    starts = torch.tensor(np.cumsum([0] + lens[:-1]), device=DEV)
    kd = _rotate(kd, _angles(s["sh"], starts[unit]))
    res = []
    for cached, fresh, p, w in ((kd, kf, pk, wk), (vd, vf, pv, wv)):
        mu = _offset(fresh, fresh_row, cached, p, lens, nd)
        c = cached + w.double()[:, None, None] * mu[unit]
        c[p.long()] = fresh[fresh_row[p.long()].long()]
        res.append((mu, torch.cat([c, fresh[fresh_row[tc:].long()]])))
    return res[0][0], res[1][0], res[0][1], res[1][1]


def exact(case, seed):
    s = prepare(case, seed)
    kind, sh = s["kind"], s["sh"]
    if kind == "quantize":
        return None
    if kind == "reuse":
        return _exact_reuse(s)
    if kind == "unit":
        w, n = s["eng"].weights, case["n"]
        pos = torch.arange(case["pos0"], case["pos0"] + n, device=DEV)
        h, ks, vs = w["embed"][s["tokens"].long()].double(), [], []
        for lw in w["layers"]:
            q, k, v = _qkv(sh, h, lw, pos)
            h = _out_mlp(sh, h, _attend(sh, q, pos - case["pos0"], k, v), lw)
            ks.append(k)
            vs.append(v)
        return [_norm(h, w["final_norm"], sh.rms_eps), torch.stack(ks), torch.stack(vs)]
    if kind == "decode":
        w, n = s["eng"].weights, case["past"] + 1
        pos = torch.tensor([case["past"]], device=DEV)
        h = w["embed"][s["token"].long()].double()
        kc, vc = s["k"][:, :n].double(), s["v"][:, :n].double()
        for l, lw in enumerate(w["layers"]):
            q, k, v = _qkv(sh, h, lw, pos)
            kc[l, -1], vc[l, -1] = k[0], v[0]
            h = _out_mlp(sh, h, _attend(sh, q, pos, kc[l], vc[l]), lw)
        logits = _norm(h, w["final_norm"], sh.rms_eps) @ w["embed"].double().T
        return [logits[0], kc, vc]
    if kind == "proj":
        h = s["h"].double()
        q, k, v = _qkv(sh, h, s["layer"], s["positions"])
        return [q.flatten(1), k.flatten(1), v.flatten(1),
                _out_mlp(sh, h, s["att"].double(), s["layer"])]
    if kind == "attn":
        return [_attend(sh, s["q"].double(), s["positions"], s["k"].double(), s["v"].double())]
    if kind in ("check", "correct"):
        kd, vd = (_dequant(sh, s[x], s[x + "_meta"], case["bits"]) for x in ("k", "v"))
    if kind == "check":
        d_k = (s["kf"].double() - _rotate(kd, _angles(sh, s["delta"]))).flatten(1).norm(dim=1)
        d_v = (s["vf"].double() - vd).flatten(1).norm(dim=1)
        return [d_k, d_v, d_k.clamp(max=1.0), d_v.clamp(max=1.0)] + [None] * 7
    if kind == "correct":
        return list(_correct(s, kd, vd, s["kf"].double(), s["vf"].double(), s["fresh_row"],
                             s["pk"], s["pv"], s["wk"], s["wv"]))
    return [s["h"].double() @ s["w"].double().T, None]


def _exact_reuse(s):
    case, sh, w, lens = s["case"], s["sh"], s["eng"].weights, s["lens"]
    tc, q = sum(lens), case["q"]
    T = tc + q
    pk, pv = s["out"]["probe_k"], s["out"]["probe_v"]
    every = torch.arange(T, device=DEV)
    starts = torch.tensor(np.repeat(np.cumsum([0] + lens[:-1]), lens), device=DEV)
    side = lambda x, l: _dequant(sh, s[x][l], None if s[x + "_meta"] is None  # noqa: E731
                                 else s[x + "_meta"][l], case["bits"])
    # the first layer over every token, the second one's fresh states for the divergences
    h = w["embed"][s["tokens"].long()].double()
    qq, k, v = _qkv(sh, h, w["layers"][0], every)
    ks, vs = [k], [v]
    h = _out_mlp(sh, h, _attend(sh, qq, every, k, v), w["layers"][0])
    _, k, v = _qkv(sh, h[:tc], w["layers"][1], every[:tc])
    d_k = (k - _rotate(side("k", 1), _angles(sh, starts))).flatten(1).norm(dim=1)
    d_v = (v - side("v", 1)).flatten(1).norm(dim=1)
    recomputed = torch.zeros(T, dtype=torch.bool, device=DEV)
    recomputed[pk.long()] = recomputed[pv.long()] = recomputed[tc:] = True
    rows = recomputed.nonzero()[:, 0]
    fresh_row = torch.full((T,), -1, device=DEV)
    fresh_row[rows] = torch.arange(len(rows), device=DEV)
    h = h[rows]
    for l in range(1, sh.n_layers):
        lw = w["layers"][l]
        qq, kf, vf = _qkv(sh, h, lw, rows)
        _, _, kc, vc = _correct(s, side("k", l), side("v", l), kf, vf, fresh_row, pk, pv,
                                d_k.clamp(max=1.0), d_v.clamp(max=1.0))
        ks.append(kc)
        vs.append(vc)
        h = _out_mlp(sh, h, _attend(sh, qq, rows, kc, vc), lw)
    return [_norm(h[-q:], w["final_norm"], sh.rms_eps), torch.stack(ks), torch.stack(vs), d_k,
            d_v, None]
