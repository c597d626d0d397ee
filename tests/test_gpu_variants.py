"""Parity of the size- and alignment-dependent kernel variants at the edges of their ranges:
the wide quantiser against the oracle at ties, the LM head over several rows, the fp32 tiles,
the few-row projections, the attention over packed head lists and short contexts, the
correction's unit search."""
import numpy as np
import pytest
import torch

import oracle
import synthetic
from paper_2607_21604_amd import akvs
from paper_2607_21604_amd.runtime import Engine, _reuse_outputs
from tests.test_gpu_steps import (gpu_offset_and_correction, make_offset_case,
                                  oracle_offset_and_correction, run_select)
from tests.gpu_util import DEV, dev_weights, f64, max_rel, storage_round, to_dev

pytestmark = pytest.mark.gpu


def _near_ties(rows, hd, bits, seed):
    """fp32 values on and beside the quantiser's rounding boundaries of their group."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((rows, hd)).astype(np.float32)
    if bits == 8:
        scale = np.float32(0.25)
        pos = oracle.e4m3_value(np.arange(0x7F))
        mid = ((pos[:-1] + pos[1:]) / 2).astype(np.float32)
        v = scale * rng.choice(mid, size=(rows, hd)) * rng.choice([-1, 1], size=(rows, hd))
        v[:, ::64] = 448 * scale
    else:
        top = 2 ** bits - 1
        scale, zero = np.float32(0.3125), np.float32(-1.5)
        v = zero + scale * (rng.integers(0, top, size=(rows, hd)) + np.float32(0.5))
        v[:, ::64], v[:, 1::64] = zero, zero + top * scale
    v = v.astype(np.float32)
    step = rng.integers(-1, 2, size=v.shape)
    step[:, ::64] = step[:, 1::64] = 0
    v = np.where(step == 0, v, np.nextafter(v, np.where(step > 0, np.inf, -np.inf),
                                            dtype=np.float32))
    x[::2] = v[::2]
    return x


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("rows,hd", [(1, 64), (33, 192), (127, 128), (257, 64), (4097, 64),
                                     (8193, 128), (5462, 192)])
def test_quantise_codes_at_ties(bits, rows, hd):
    """Bit-exact codes and metadata at the rounding boundaries, for block remainders, fp32 and
    bf16 inputs, operands that miss the wide kernel's alignment, and group counts on both sides
    of those from which it is taken (4096, or 16384 at 8 bits)."""
    x32 = torch.from_numpy(_near_ties(rows, hd, bits, 7 * rows + bits))
    for x in (x32, x32.to(torch.bfloat16)):
        if bits == 8:
            codes, meta = oracle.quantize_e4m3_g64(f64(x))
        else:
            codes, meta = oracle.quantize_g64(f64(x), bits)
            codes = oracle.pack_codes(codes, bits)
        for shift in (0, 1):  # one element off: not 16-byte aligned
            buf = torch.zeros(rows * hd + shift, dtype=x.dtype, device=DEV)
            xd = buf[shift:].view(rows, hd)
            xd.copy_(x)
            c = torch.full((rows, hd * bits // 8), 0xA5, dtype=torch.uint8, device=DEV)
            mt = torch.empty((rows, hd // 64, 2), dtype=torch.float16, device=DEV)
            akvs.akvs_quantize_cache(xd, rows, hd, bits, c, mt)
            np.testing.assert_array_equal(c.cpu().numpy(), codes)
            np.testing.assert_array_equal(mt.cpu().numpy().view(np.uint16), meta.view(np.uint16))


@pytest.mark.parametrize("rows", [1, 2, 16, 17, 33])
@pytest.mark.parametrize("vocab,d", [(1021, 192), (160, 64), (1000, 320)])
def test_lm_head_rows(rows, vocab, d):
    """Several rows in one call: fp32 logits (error bound of a K-term fp32 sum in any order,
    K 2^-24 sum |h w|), picks of the lowest index on ties, with and without logits."""
    sh = synthetic.ModelShape("head", 1, d, 2, 2, 64, 128, vocab, 1e4)
    m = akvs.model_cfg(sh)
    h = torch.from_numpy(synthetic.random_array((rows, d), 3 + rows)).float()
    w = torch.from_numpy(synthetic.random_array((vocab, d), 5 + vocab) * 0.02).to(torch.bfloat16)
    ref = f64(h) @ f64(w).T
    bound = d * 2.0 ** -24 * (np.abs(f64(h)) @ np.abs(f64(w)).T)
    w[vocab - 1] = w[int(ref[0].argmax())]  # row 0's best logit twice: the lower index wins
    ref = f64(h) @ f64(w).T
    hd, wd = to_dev(h), to_dev(w)
    ws = torch.empty(akvs.akvs_decode_workspace_size(m, 0), dtype=torch.uint8, device=DEV)
    logits = torch.full((rows, vocab), float("nan"), device=DEV)
    toks = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    akvs.akvs_lm_head(hd, rows, wd, m, logits, toks, ws)
    got = f64(logits)
    assert np.all(np.abs(got[:, :vocab - 1] - ref[:, :vocab - 1]) <= bound[:, :vocab - 1])
    np.testing.assert_array_equal(toks.cpu().numpy(), got.argmax(axis=1))
    only = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    akvs.akvs_lm_head(hd, rows, wd, m, None, only, ws)
    assert torch.equal(only, toks)


@pytest.mark.parametrize("rows", [2, 17, 32])
@pytest.mark.parametrize("vocab", [152064, 131075])
def test_lm_head_rows_of_large_vocabularies(vocab, rows):
    """Vocabularies past 131072 rows, which take 80 of them per wave: the last blocks' remainders
    of 320, rows past the vocabulary, picks there, with and without logits."""
    d = 192
    sh = synthetic.ModelShape("head", 1, d, 2, 2, 64, 128, vocab, 1e4)
    m = akvs.model_cfg(sh)
    h = torch.from_numpy(synthetic.random_array((rows, d), 13 + rows)).float()
    w = torch.from_numpy(synthetic.random_array((vocab, d), 17) * 0.02).to(torch.bfloat16)
    w[vocab - 1] = (h[0] / h[0].norm()).to(torch.bfloat16)  # row 0 picks the last
    w[vocab - 3] = (h[1] / h[1].norm()).to(torch.bfloat16)
    ref = f64(h) @ f64(w).T
    bound = d * 2.0 ** -24 * (np.abs(f64(h)) @ np.abs(f64(w)).T)
    hd, wd = to_dev(h), to_dev(w)
    ws = torch.empty(akvs.akvs_decode_workspace_size(m, 0), dtype=torch.uint8, device=DEV)
    logits = torch.full((rows, vocab), float("nan"), device=DEV)
    toks = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    akvs.akvs_lm_head(hd, rows, wd, m, logits, toks, ws)
    got = f64(logits)
    assert np.all(np.abs(got - ref) <= bound)
    np.testing.assert_array_equal(toks.cpu().numpy(), got.argmax(axis=1))
    assert toks[0].item() == vocab - 1 and toks[1].item() == vocab - 3
    only = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    akvs.akvs_lm_head(hd, rows, wd, m, None, only, ws)
    assert torch.equal(only, toks)


def test_lm_head_rows_infinities_and_nan():
    """Infinite weights and rows holding an infinity or a NaN: the values of the plain sums;
    NaN never wins the pick, a row of NaN picks nothing."""
    sh = synthetic.ModelShape("head", 1, 64, 2, 2, 64, 128, 300, 1e4)
    m = akvs.model_cfg(sh)
    h = torch.from_numpy(synthetic.random_array((4, 64), 9)).float()
    w = torch.from_numpy(synthetic.random_array((300, 64), 10)).to(torch.bfloat16)
    h[0, 5] = 1.0  # exactly one bf16 value: the split's other terms are 0
    w[17, 5] = float("inf")
    h[1, 3], h[2, 3] = float("inf"), float("nan")
    ref = (h.double() @ w.double().T).numpy()
    ws = torch.empty(akvs.akvs_decode_workspace_size(m, 0), dtype=torch.uint8, device=DEV)
    logits = torch.empty((4, 300), device=DEV)
    toks = torch.empty(4, dtype=torch.int32, device=DEV)
    akvs.akvs_lm_head(to_dev(h), 4, to_dev(w), m, logits, toks, ws)
    got = f64(logits)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    fin = np.isfinite(ref)
    np.testing.assert_allclose(got[fin], ref[fin], rtol=0, atol=1e-4)
    np.testing.assert_array_equal(got[~fin & ~np.isnan(ref)], ref[~fin & ~np.isnan(ref)])
    assert toks[0].item() == 17 and toks[2].item() == -1


def _gpu_us(f, reps=5):
    """Best of a few timings of one call, in us."""
    f()
    best = float("inf")
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.parametrize("fill", [float("nan"), float("inf")])
def test_lm_head_nonfinite_row_costs_no_other_row(fill):
    """One row of h that is not finite leaves the call's time of the order of the finite one's
    (at 3B width a single row's own sums are one read of the vocabulary, as the whole call is),
    and the other rows' logits as they were."""
    vocab, d, rows = 128256, 3072, 16
    sh = synthetic.ModelShape("head", 1, d, 2, 2, 64, 128, vocab, 1e4)
    m = akvs.model_cfg(sh)
    g = torch.Generator(device=DEV).manual_seed(3)
    w = (torch.randn((vocab, d), device=DEV, generator=g) * 0.02).to(torch.bfloat16)
    h = torch.randn((rows, d), device=DEV, generator=g)
    bad = h.clone()
    bad[5, 7] = fill
    ws = torch.empty(akvs.akvs_decode_workspace_size(m, 0), dtype=torch.uint8, device=DEV)
    out = {}
    us = {}
    for name, x in (("fine", h), ("bad", bad)):
        logits = torch.empty((rows, vocab), device=DEV)
        toks = torch.empty(rows, dtype=torch.int32, device=DEV)
        us[name] = _gpu_us(lambda: akvs.akvs_lm_head(x, rows, w, m, logits, toks, ws))
        out[name] = (logits, toks)
    others = torch.arange(rows, device=DEV) != 5
    for a, b in zip(out["fine"], out["bad"]):
        assert torch.equal(a[others], b[others])
    row = out["bad"][0][5]
    if fill != fill:
        assert torch.isnan(row).all() and int(out["bad"][1][5]) == -1
    else:  # h = inf: +-inf by the sign of the weight, NaN where it is 0
        ref = torch.where(w[:, 7] == 0, float("nan"), torch.sign(w[:, 7].float()) * fill)
        assert torch.equal(torch.isnan(row), torch.isnan(ref))
        assert torch.equal(row[~torch.isnan(ref)], ref[~torch.isnan(ref)])
    assert us["bad"] < 4 * us["fine"], us


@pytest.mark.parametrize("vocab,d,rows", [(1000, 4096, 2), (512, 5120, 3)])
def test_lm_head_few_rows_of_small_vocabularies(vocab, d, rows):
    """A call over a few rows takes no longer than as many calls over one (a block of the
    several-row kernel walks the whole width, which small vocabularies leave with few blocks)."""
    sh = synthetic.ModelShape("head", 1, d, 2, 2, 64, 128, vocab, 1e4)
    m = akvs.model_cfg(sh)
    w = to_dev(synthetic.random_array((vocab, d), 4) * 0.02, torch.bfloat16)
    h = to_dev(synthetic.random_array((rows, d), 5).astype(np.float32))
    ws = torch.empty(akvs.akvs_decode_workspace_size(m, 0), dtype=torch.uint8, device=DEV)
    logits = torch.empty((rows, vocab), device=DEV)
    toks = torch.empty(rows, dtype=torch.int32, device=DEV)

    def whole():
        for _ in range(50):
            akvs.akvs_lm_head(h, rows, w, m, logits, toks, ws)

    def single():
        for _ in range(50):
            for r in range(rows):
                akvs.akvs_lm_head(h[r:r + 1], 1, w, m, logits[r:r + 1], toks[r:r + 1], ws)

    assert _gpu_us(whole) < 1.4 * _gpu_us(single)


def _check_projections(shape, rows, tol):
    """akvs_probe_qkv and akvs_probe_out_mlp against the oracle over sampled rows."""
    d, hq, hkv, hd = shape.d_model, shape.n_q_heads, shape.n_kv_heads, shape.head_dim
    dt = synthetic.torch_dtype(shape)
    w = synthetic.make_weights(shape, seed=rows, std=0.1 if dt == torch.float32 else 0.02,
                               embed=False)
    dims = oracle.dims_from(shape)
    m = akvs.model_cfg(shape)
    lwd = {k: to_dev(t) for k, t in w["layers"][0].items()}
    lws = akvs.layer_array({"layers": [lwd]})[0]
    h = synthetic.random_array((rows, d), 6).astype(np.float32)
    pos = np.arange(rows, dtype=np.int32)
    table = torch.empty((rows, hd // 2, 2), device=DEV)
    akvs.akvs_rope_table(rows, hd, 1e4, table)
    att = storage_round(synthetic.random_array((rows, hq * hd), 7), dt)
    ws = torch.full((akvs.akvs_step_workspace_size(m, rows),), 255, dtype=torch.uint8, device=DEV)
    q = torch.empty((rows, hq, hd), dtype=dt, device=DEV)
    kf, vf = (torch.empty((rows, hkv, hd), dtype=dt, device=DEV) for _ in range(2))
    hdev = to_dev(h)
    akvs.akvs_probe_qkv(hdev, rows, to_dev(pos), m, lws, table, rows, q, kf, vf, ws)
    akvs.akvs_probe_out_mlp(hdev, rows, to_dev(att), m, lws, ws)
    some = np.union1d(np.arange(0, rows, 4), np.arange(max(rows - 35, 0), rows))
    sw = oracle.split_layer(w["layers"][0], dims)
    h64 = h[some].astype(np.float64)
    for got, ref in zip((q, kf, vf), oracle.model.project_qkv(h64, pos[some], sw, dims)):
        assert max_rel(f64(got)[some], ref) < tol
    ref = oracle.model.output_and_mlp(h64, f64(att)[some], sw, dims)
    assert max_rel(f64(hdev)[some], ref) < tol


@pytest.mark.parametrize("d,hq,hkv,hd,ffn,rows", [
    (72, 3, 1, 64, 100, 1), (72, 3, 1, 64, 100, 17), (8, 1, 1, 64, 4, 16),
    (200, 4, 2, 128, 1028, 33), (200, 4, 2, 128, 1028, 2080)])
def test_fp32_projections(d, hq, hkv, hd, ffn, rows):
    """The fp32 tiles (16 and 32 rows, 64 and 128 columns) at remainders of rows, columns and
    K, against the oracle. Tolerance of the fp32 path."""
    shape = synthetic.ModelShape("v", 1, d, hq, hkv, hd, ffn, 64, 1e4, dtype="f32")
    w = synthetic.make_weights(shape, seed=rows, std=0.1, embed=False)
    dims = oracle.dims_from(shape)
    m = akvs.model_cfg(shape)
    lwd = {k: to_dev(t) for k, t in w["layers"][0].items()}
    lws = akvs.layer_array({"layers": [lwd]})[0]
    h = synthetic.random_array((rows, d), 6).astype(np.float32)
    pos = np.arange(rows, dtype=np.int32) * 2
    table = torch.empty((2 * rows, hd // 2, 2), device=DEV)
    akvs.akvs_rope_table(2 * rows, hd, 1e4, table)
    q = torch.empty((rows, hq, hd), device=DEV)
    kf, vf = (torch.empty((rows, hkv, hd), device=DEV) for _ in range(2))
    ws = torch.empty(akvs.akvs_step_workspace_size(m, rows), dtype=torch.uint8, device=DEV)
    hdev = to_dev(h)
    akvs.akvs_probe_qkv(hdev, rows, to_dev(pos), m, lws, table, 2 * rows, q, kf, vf, ws)
    sw = oracle.split_layer(w["layers"][0], dims)
    for got, ref in zip((q, kf, vf), oracle.model.project_qkv(h.astype(np.float64), pos, sw, dims)):
        assert max_rel(f64(got), ref) < 1e-5
    att = synthetic.random_array((rows, hq * hd), 7).astype(np.float32)
    akvs.akvs_probe_out_mlp(hdev, rows, to_dev(att), m, lws, ws)
    ref = oracle.model.output_and_mlp(h.astype(np.float64), att.astype(np.float64), sw, dims)
    assert max_rel(f64(hdev), ref) < 1e-5


@pytest.mark.parametrize("d,hq,hkv,hd,ffn,rows,codes", [
    (1032, 8, 4, 64, 260, 1399, (1, 1, 0, 1)),        # 32 x 64 tiles
    (264, 24, 8, 128, 260, 897, (3, 0, 0, 0)),        # 32 x 128
    (200, 4, 2, 128, 1028, 33, (2, 0, 0, 0)),         # 16 x 128
    (72, 3, 1, 64, 100, 9001, (10, 10, 10, 10)),      # LDS-tiled, K of 72, 192 and 100
    (264, 5, 1, 64, 260, 6001, (10, 1, 10, 10)),
    (136, 2, 1, 128, 516, 3009, (10, 0, 10, 0))])
def test_fp32_projection_kernels(d, hq, hkv, hd, ffn, rows, codes):
    """Every fp32 tile and the LDS-tiled kernel at remainders of rows, columns and K (a quarter
    of the rows, the last ones among them, against the oracle)."""
    shape = synthetic.ModelShape("v", 1, d, hq, hkv, hd, ffn, 64, 1e4, dtype="f32")
    assert akvs.akvs_projection_kernels(akvs.model_cfg(shape), rows) == codes
    _check_projections(shape, rows, 1e-5)


@pytest.mark.parametrize("hq,hkv,hd,rows,n_keys", [
    (2, 1, 64, 1, 1), (2, 2, 128, 15, 17), (4, 1, 64, 17, 129), (3, 3, 128, 40, 300),
    (1, 1, 64, 16, 1000)])
def test_fp32_attention(hq, hkv, hd, rows, n_keys):
    """Rows and keys around the 16-row tile and the 8 x 16 keys of one turn of its waves."""
    rng = np.random.default_rng(n_keys)
    rows = min(rows, n_keys)
    pos = np.sort(rng.choice(n_keys, size=rows, replace=False)).astype(np.int32)
    q, k, v = (synthetic.random_array((n, h, hd), 40 + i).astype(np.float32)
               for i, (n, h) in enumerate([(rows, hq), (n_keys, hkv), (n_keys, hkv)]))
    q[0] *= 30  # one row of large scores
    m = akvs.ModelCfg(1, 64, hq, hkv, hd, 64, 16, 1e4, 1e-6, akvs.AKVS_F32)
    out = torch.empty((rows, hq * hd), device=DEV)
    akvs.akvs_sparse_query_attention(to_dev(q), to_dev(pos), rows, to_dev(k), to_dev(v), n_keys, m,
                                     out)
    ref = oracle.attention(q.astype(np.float64), pos, k.astype(np.float64), v.astype(np.float64),
                           np.arange(n_keys)).reshape(rows, -1)
    assert max_rel(f64(out), ref) < 1e-5


def _attention_visible_only(q, pos, k, v):
    """The oracle's attention, each row over no other keys than those it may see."""
    with np.errstate(invalid="ignore"):
        return np.concatenate([oracle.attention(q[i:i + 1], pos[i:i + 1], k[:p + 1], v[:p + 1],
                                                np.arange(p + 1)) for i, p in enumerate(pos)]
                              ).reshape(len(pos), -1)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("hd,pos,key", [
    (64, np.arange(40), 18),    # inside a 16-row block: rows 16 and 17 may not see it
    (128, np.arange(40), 39),   # the last key of the last block, which masked keys re-read
    (64, np.arange(0, 300, 9), 142), (128, np.array([3, 4, 5, 290]), 6),
    (64, np.array([130, 131, 132]), 131)])
def test_fp32_attention_hidden_values_stay_hidden(hd, pos, key, bad):
    """An infinite or NaN value reaches the rows that see its key and no other: the rows before
    it stay exact, those after it hold what the plain sums give."""
    pos = pos.astype(np.int32)
    rows, n_keys = len(pos), 300
    q, k, v = (synthetic.random_array((n, h, hd), 60 + i).astype(np.float32)
               for i, (n, h) in enumerate([(rows, 2), (n_keys, 1), (n_keys, 1)]))
    v[key, 0, ::3] = bad
    m = akvs.ModelCfg(1, 64, 2, 1, hd, 64, 16, 1e4, 1e-6, akvs.AKVS_F32)
    out = torch.empty((rows, 2 * hd), device=DEV)
    akvs.akvs_sparse_query_attention(to_dev(q), to_dev(pos), rows, to_dev(k), to_dev(v), n_keys, m,
                                     out)
    ref = _attention_visible_only(q.astype(np.float64), pos, k.astype(np.float64),
                                  v.astype(np.float64))
    got = f64(out)
    fin = np.isfinite(ref)
    assert fin[pos < key].all() and not fin[pos >= key].all()
    assert max_rel(got[fin], ref[fin]) < 1e-5
    np.testing.assert_array_equal(got[~fin], ref[~fin])


def test_fp32_attention_seen_nan_costs_nothing():
    """A NaN value that every row sees is no reason to form the rows again: the call takes its
    usual time."""
    hq, hkv, hd, rows, n_keys = 8, 2, 128, 1000, 2000
    m = akvs.ModelCfg(1, 64, hq, hkv, hd, 64, 16, 1e4, 1e-6, akvs.AKVS_F32)
    q, k, v = (torch.randn((n, h, hd), device=DEV) for n, h in ((rows, hq), (n_keys, hkv),
                                                                (n_keys, hkv)))
    pos = torch.arange(n_keys - rows, n_keys, dtype=torch.int32, device=DEV)
    out = torch.empty((rows, hq * hd), device=DEV)
    us = []
    for _ in range(2):
        us.append(_gpu_us(lambda: akvs.akvs_sparse_query_attention(q, pos, rows, k, v, n_keys, m,
                                                                   out)))
        v[3, :, 7] = float("nan")
    assert us[1] < 2 * us[0], us
    nan = torch.isnan(out.view(rows, hq, hd))
    assert nan[:, :, 7].all() and int(nan.sum()) == rows * hq


@pytest.mark.parametrize("hd,pos,key", [
    (64, np.arange(40), 16), (128, np.arange(40), 32),    # alone in its wave's share of a row
    (128, np.arange(0, 300, 3), 144), (64, np.array([127, 128, 129]), 128),
    (64, np.array([0]), 0)])
def test_fp32_attention_nan_scores_are_kept(hd, pos, key):
    """A NaN key makes NaN of every row that sees it, also where it is the only visible key of
    a wave's tiles, and of no other row."""
    pos = pos.astype(np.int32)
    rows, n_keys = len(pos), 300
    q, k, v = (synthetic.random_array((n, h, hd), 70 + i).astype(np.float32)
               for i, (n, h) in enumerate([(rows, 2), (n_keys, 1), (n_keys, 1)]))
    k[key, 0, 5] = np.nan
    m = akvs.ModelCfg(1, 64, 2, 1, hd, 64, 16, 1e4, 1e-6, akvs.AKVS_F32)
    out = torch.empty((rows, 2 * hd), device=DEV)
    akvs.akvs_sparse_query_attention(to_dev(q), to_dev(pos), rows, to_dev(k), to_dev(v), n_keys, m,
                                     out)
    got = f64(out)
    assert np.isnan(got[pos >= key]).all()
    clean = pos < key
    if clean.any():
        ref = _attention_visible_only(q[clean].astype(np.float64), pos[clean],
                                      k.astype(np.float64), v.astype(np.float64))
        assert max_rel(got[clean], ref) < 1e-5


def test_attention_pieces_keep_nan_scores():
    """bf16 rows whose key range is cut into pieces: a row whose piece holds no other visible key
    than a NaN one is NaN, wherever the pieces begin."""
    hq, hkv, hd, n_keys = 4, 1, 128, 4500
    m = akvs.ModelCfg(1, 64, hq, hkv, hd, 64, 16, 1e4, 1e-6, akvs.AKVS_BF16)
    keys = np.arange(64, n_keys, 64)
    q, k, v = (storage_round(synthetic.random_array((n, h, hd), 80 + i), torch.bfloat16)
               for i, (n, h) in enumerate([(len(keys), hq), (n_keys, hkv), (n_keys, hkv)]))
    qd, kd, vd, pd = to_dev(q), to_dev(k), to_dev(v), to_dev(keys.astype(np.int32))
    nbytes = akvs.akvs_attention_workspace_size(m, len(keys), n_keys)
    assert nbytes > 0
    ws = torch.zeros(nbytes, dtype=torch.uint8, device=DEV)
    for i, key in enumerate(keys):
        saved = kd[key].clone()
        kd[key, 0, 5] = float("nan")
        out = torch.empty((len(keys), hq * hd), dtype=torch.bfloat16, device=DEV)
        akvs.akvs_sparse_query_attention(qd, pd, len(keys), kd, vd, n_keys, m, out, ws)
        nan = torch.isnan(out).all(dim=1).cpu().numpy()
        assert nan[i:].all() and not torch.isnan(out[:i]).any()
        kd[key] = saved


@pytest.mark.parametrize("d,hq,hkv,hd,ffn,rows", [
    (2048, 16, 4, 128, 2176, 1), (2048, 16, 4, 128, 2176, 31), (2048, 16, 4, 128, 2176, 33),
    (2048, 16, 4, 128, 2176, 65), (2048, 16, 4, 128, 2176, 97), (2048, 16, 4, 128, 2176, 200),
    (2048, 16, 4, 128, 2176, 385), (3072, 24, 8, 128, 8192, 129), (4096, 32, 4, 128, 8192, 96),
    (320, 5, 1, 64, 448, 1), (320, 5, 1, 64, 448, 95), (320, 5, 1, 64, 448, 130),
    (64, 1, 1, 64, 64, 40)])
def test_few_row_projections(d, hq, hkv, hd, ffn, rows):
    """Few rows at row, column and K remainders (a K of 2176 is an odd multiple of 128), with and
    without the K split, against the oracle; the same bits twice. The width-2048 to -4096 shapes
    run on the few-row tiles (101 of akvs_projection_kernels and up), the last four, too small
    for them, on the 128 x 128 8-wave tile."""
    shape = synthetic.ModelShape("v", 1, d, hq, hkv, hd, ffn, 64, 1e4)
    w = synthetic.make_weights(shape, seed=rows, embed=False)
    dims = oracle.dims_from(shape)
    m = akvs.model_cfg(shape)
    lwd = {k: to_dev(t) for k, t in w["layers"][0].items()}
    lws = akvs.layer_array({"layers": [lwd]})[0]
    h = synthetic.random_array((rows, d), 6).astype(np.float32)
    pos = np.arange(rows, dtype=np.int32) * 2
    table = torch.empty((2 * rows, hd // 2, 2), device=DEV)
    akvs.akvs_rope_table(2 * rows, hd, 1e4, table)
    att = storage_round(synthetic.random_array((rows, hq * hd), 7), torch.bfloat16)
    nbytes = akvs.akvs_step_workspace_size(m, rows)
    runs = []
    for fill in (0, 255):  # what the workspace holds does not matter
        ws = torch.full((nbytes,), fill, dtype=torch.uint8, device=DEV)
        q = torch.empty((rows, hq, hd), dtype=torch.bfloat16, device=DEV)
        kf, vf = (torch.empty((rows, hkv, hd), dtype=torch.bfloat16, device=DEV) for _ in range(2))
        hdev = to_dev(h)
        akvs.akvs_probe_qkv(hdev, rows, to_dev(pos), m, lws, table, 2 * rows, q, kf, vf, ws)
        akvs.akvs_probe_out_mlp(hdev, rows, to_dev(att), m, lws, ws)
        runs.append((q, kf, vf, hdev))
    for a, b in zip(*runs):
        assert torch.equal(a, b)
    sw = oracle.split_layer(w["layers"][0], dims)
    for got, ref in zip(runs[0], oracle.model.project_qkv(h.astype(np.float64), pos, sw, dims)):
        assert max_rel(f64(got), ref) < 1e-2  # a bf16 rounding of inputs and outputs: 2^-8 each
    ref = oracle.model.output_and_mlp(h.astype(np.float64), f64(att), sw, dims)
    assert max_rel(f64(runs[0][3]), ref) < 1e-2


@pytest.mark.parametrize("d,hq,hkv,hd,ffn,rows,codes", [
    (512, 32, 8, 64, 1024, 200, (111, 104, 101, 101)),    # heads of 64 on 64 x 64,
    (512, 32, 8, 64, 1024, 385, (121, 101, 111, 101)),    # 96 x 64
    (1024, 32, 8, 64, 1024, 501, (131, 101, 111, 101)),   # and 96 x 128 tiles
    (512, 8, 2, 64, 1088, 1, (101, 101, 101, 131)),       # 17 k-tiles of 64
    (1088, 8, 2, 64, 2176, 499, (131, 111, 131, 111)),
    (512, 8, 2, 64, 4160, 97, (101, 101, 205, 138)),      # 65 k-tiles in 8 slices, 96 x 128
    (3072, 8, 2, 64, 4160, 97, (306, 101, 303, 148)),     # and 128 x 128; 8-wave K splits
    (512, 24, 8, 128, 1024, 201, (121, 118, 101, 101)),
    (512, 8, 2, 64, 4160, 901, (111, 101, 201, 136)),     # the 8-wave tiles: 192 x 256,
    (512, 8, 2, 64, 4160, 701, (111, 101, 202, 138)),     # 256 x 128,
    (512, 8, 2, 64, 4160, 385, (101, 101, 203, 138)),     # 192 x 128,
    (512, 8, 2, 64, 18944, 97, (101, 101, 204, 108)),     # 128 x 256
    (512, 8, 2, 64, 8192, 897, (111, 101, 200, 312))])    # and 256 x 256
def test_bf16_projection_kernels(d, hq, hkv, hd, ffn, rows, codes):
    """Each few-row and 8-wave tile, named by akvs_projection_kernels, at remainders of rows,
    columns and k-tiles, against the oracle (a bf16 rounding of inputs and outputs)."""
    shape = synthetic.ModelShape("v", 1, d, hq, hkv, hd, ffn, 64, 1e4)
    assert akvs.akvs_projection_kernels(akvs.model_cfg(shape), rows) == codes
    _check_projections(shape, rows, 1e-2)


@pytest.mark.parametrize("hq,hkv,hd,rows,n_keys", [
    (10, 2, 128, 33, 4500), (14, 2, 128, 57, 5261), (40, 8, 128, 159, 1100), (3, 1, 64, 9, 4900),
    (24, 8, 128, 1, 4300), (10, 2, 64, 200, 1700), (10, 2, 64, 192, 4097), (16, 1, 128, 193, 4100),
    (16, 1, 128, 129, 1024), (14, 2, 128, 128, 1000), (8, 2, 128, 16, 4097), (8, 2, 128, 17, 4097),
    (10, 2, 128, 17, 6145), (14, 2, 64, 128, 6144), (14, 2, 64, 64, 6200),
    (4, 2, 128, 203, 203), (4, 2, 64, 384, 768), (4, 2, 128, 385, 769), (4, 4, 128, 20, 384),
    (4, 4, 128, 20, 385)])
def test_attention_packed_heads_and_short_contexts(hq, hkv, hd, rows, n_keys):
    """Row lists of several query heads (G of 3 to 16), up to 16 pieces per tile, and the key
    counts around which short contexts run whole; the same result for any workspace content."""
    rng = np.random.default_rng(rows)
    pos = np.sort(rng.choice(n_keys, size=rows, replace=False)).astype(np.int32)
    q, k, v = (storage_round(synthetic.random_array((n, h, hd), 50 + i), torch.bfloat16)
               for i, (n, h) in enumerate([(rows, hq), (n_keys, hkv), (n_keys, hkv)]))
    m = akvs.ModelCfg(1, 64, hq, hkv, hd, 64, 16, 1e4, 1e-6, akvs.AKVS_BF16)
    ref = oracle.attention(f64(q), pos, f64(k), f64(v), np.arange(n_keys)).reshape(rows, -1)
    nbytes = akvs.akvs_attention_workspace_size(m, rows, n_keys)
    outs = []
    for ws in (None, torch.full((max(nbytes, 1),), 255, dtype=torch.uint8, device=DEV),
               torch.zeros(max(nbytes, 1), dtype=torch.uint8, device=DEV)):
        out = torch.empty((rows, hq * hd), dtype=torch.bfloat16, device=DEV)
        akvs.akvs_sparse_query_attention(to_dev(q), to_dev(pos), rows, to_dev(k), to_dev(v), n_keys,
                                         m, out, ws)
        assert max_rel(f64(out), ref) < 1e-2
        outs.append(out)
    assert torch.equal(outs[1], outs[2])


@pytest.mark.parametrize("dtype,hkv,hd", [("bf16", 8, 128), ("bf16", 4, 128), ("bf16", 3, 64)])
@pytest.mark.parametrize("units", [1, 63, 64, 65, 130])
def test_correction_finds_the_unit_of_many(dtype, hkv, hd, units):
    """A token's unit from the unit table alone, around multiples of the 64 starts that a wave
    compares at once (whole waves per position at 1024 and 512 wide rows, not at 192)."""
    lens = [1 + (5 * i) % 4 for i in range(units)]
    cs = make_offset_case(dtype, lens, hkv, hd, seed=units)
    mu_k, mu_v, k_corr, v_corr = gpu_offset_and_correction(cs, hkv, hd)
    _, _, rk, rv = oracle_offset_and_correction(cs)
    assert max_rel(f64(k_corr), rk) < 4e-3 and max_rel(f64(v_corr), rv) < 4e-3  # one bf16 rounding


@pytest.mark.parametrize("units", [128, 129, 256, 4097, 8193])
def test_correction_finds_the_unit_in_several_looks(units):
    """The same with more units than one look tells apart, around the counts where the number of
    looks and the spacing of their starts change."""
    rng = np.random.default_rng(units)
    lens = [int(x) for x in rng.integers(1, 4, size=units)]
    cs = make_offset_case("bf16", lens, 4, 64, seed=units)
    mu_k, mu_v, k_corr, v_corr = gpu_offset_and_correction(cs, 4, 64)
    _, _, rk, rv = oracle_offset_and_correction(cs)
    assert max_rel(f64(k_corr), rk) < 4e-3 and max_rel(f64(v_corr), rv) < 4e-3  # one bf16 rounding


@pytest.mark.parametrize("longest", [1, 15, 16, 17, 31, 100, 255, 256, 257])
def test_selection_block_sizes(longest):
    """Probe lists and recomputed rows bit exact where the longest unit sets the block's threads
    (one to sixteen waves of 16 tokens each), with shorter units beside it and many ties."""
    rng = np.random.default_rng(longest)
    lens = [longest, 1] + [int(x) for x in rng.integers(1, longest + 1, size=40)]
    tc, q, refresh = sum(lens), 3, (3, 10)
    d_k = rng.integers(0, 5, size=tc).astype(np.float32) * 0.25
    d_v = rng.random(tc).astype(np.float32) * 3
    got, sum_b, _ = run_select(d_k, d_v, lens, q, refresh)
    keep = np.zeros(tc, bool)
    for side, d in (("probe_k", d_k), ("probe_v", d_v)):
        ref = np.concatenate([oracle.select_top(d[s:s + n], oracle.probe_budget(n, *refresh)) + s
                              for s, n in zip(oracle.chunk_starts(lens), lens)])
        np.testing.assert_array_equal(got[side][:sum_b], ref)
        keep[ref] = True
    rows = np.concatenate([np.nonzero(keep)[0], np.arange(tc, tc + q)])
    np.testing.assert_array_equal(got["rows"][:int(got["n_rows"][0])], rows)


@pytest.mark.parametrize("hq,hkv,hd,rows,n_keys,least", [
    (32, 8, 64, 160, 4500, 8357120), (40, 8, 128, 192, 6200, 20276480)])
def test_attention_in_the_smaller_workspace(hq, hkv, hd, rows, n_keys, least):
    """Few rows over many keys in a workspace of 8 pieces a tile (or the unplanned split), smaller
    than the size asked for: accepted, the same values; 256 bytes less are refused."""
    m = akvs.ModelCfg(1, 64, hq, hkv, hd, 64, 16, 1e4, 1e-6, akvs.AKVS_BF16)
    full = akvs.akvs_attention_workspace_size(m, rows, n_keys)
    assert full > least
    pos = np.linspace(100, n_keys - 1, rows).astype(np.int32)
    q, k, v = (storage_round(synthetic.random_array((n, h, hd), 90 + i), torch.bfloat16)
               for i, (n, h) in enumerate([(rows, hq), (n_keys, hkv), (n_keys, hkv)]))
    qd, kd, vd, pd = to_dev(q), to_dev(k), to_dev(v), to_dev(pos)
    some = np.arange(0, rows, 7)
    ref = oracle.attention(f64(q)[some], pos[some], f64(k), f64(v),
                           np.arange(n_keys)).reshape(len(some), -1)
    for nbytes in (full, least):
        out = torch.empty((rows, hq * hd), dtype=torch.bfloat16, device=DEV)
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device=DEV)
        akvs.akvs_sparse_query_attention(qd, pd, rows, kd, vd, n_keys, m, out, ws)
        assert max_rel(f64(out)[some], ref) < 1e-2
    with pytest.raises(akvs.AkvsError):
        akvs.akvs_sparse_query_attention(qd, pd, rows, kd, vd, n_keys, m, out, ws[:least - 256])


def test_reuse_calls_in_the_smaller_workspace():
    """The same of whole reuse calls, one and two requests (up to 184 rows over 4464 keys)."""
    shape = synthetic.ModelShape("v", 3, 64, 32, 8, 64, 64, 500, 1e4)
    eng = Engine(shape, dev_weights(synthetic.make_weights(shape, seed=3)))
    m, lens, q = eng.m, [220] * 20, 64
    cfg = akvs.reuse_cfg(lens, q, (1, 100))
    tc, least, least2 = sum(lens), 84720128, 115074304
    two = (akvs.ReuseCfg * 2)(cfg, cfg)
    assert akvs.akvs_workspace_size(m, cfg) > least
    assert akvs.akvs_batch_workspace_size(m, two, 2) > least2
    rng = np.random.default_rng(1)
    tokens = to_dev(rng.integers(0, 500, size=tc + q).astype(np.int32))
    k, v = (to_dev(rng.standard_normal((3, tc, 8, 64)).astype(np.float32), torch.bfloat16)
            for _ in range(2))
    ref = eng.reuse_prefill(tokens, lens, q, k, v, refresh=(1, 100))
    args = (eng.weights["embed"], eng.layers, eng.weights["final_norm"], m)

    def outputs():
        o = _reuse_outputs(eng, q, tc, len(ref["probe_k"]), tc + q, len(ref["probe_v"]))
        return o, akvs.ReuseOut(*(akvs.ptr(o[x]) for x in (
            "h_query", "k_corr", "v_corr", "probe_k", "probe_v", "d_k", "d_v", "rows", "n_rows")))

    cache = akvs.cache_struct(k, v)
    (o, s), (o1, s1), (o2, s2) = outputs(), outputs(), outputs()
    ws = torch.full((max(least, least2),), 255, dtype=torch.uint8, device=DEV)
    akvs.akvs_reuse_prefill(tokens, *args, cfg, cache, s, ws[:least])
    ca, cc, co = akvs.batch_arrays([cfg, cfg], [cache, cache], [s1, s2])
    akvs.akvs_reuse_prefill_batch([tokens, tokens], *args, ca, cc, co, ws[:least2])
    n = int(ref["n_rows"])
    for got in (o, o1, o2):
        assert int(got["n_rows"]) == n and torch.equal(got["rows"][:n], ref["rows"][:n])
        for x in ("h_query", "k_corr", "v_corr"):
            assert max_rel(f64(got[x]), f64(ref[x])) < 2e-2
    with pytest.raises(akvs.AkvsError):
        akvs.akvs_reuse_prefill(tokens, *args, cfg, cache, s, ws[:least - 256])


def test_attention_pieces_lose_no_precision():
    """Rows cut into 16 pieces, whose outputs are held in 16 bits until the merge: 2.35e-3 from 64
    bits, what the bf16 probabilities and outputs make (2.63e-3 with bf16 partials in 8 pieces,
    2.76e-3 in 16)."""
    hq, hkv, hd, rows, n_keys = 28, 4, 128, 159, 8000
    rng = np.random.default_rng(rows)
    pos = np.sort(rng.choice(n_keys, size=rows, replace=False)).astype(np.int32)
    q, k, v = (storage_round(rng.standard_normal((n, h, hd)), torch.bfloat16)
               for n, h in ((rows, hq), (n_keys, hkv), (n_keys, hkv)))
    m = akvs.ModelCfg(1, 64, hq, hkv, hd, 64, 16, 1e4, 1e-6, akvs.AKVS_BF16)
    ws = torch.empty(akvs.akvs_attention_workspace_size(m, rows, n_keys), dtype=torch.uint8,
                     device=DEV)
    out = torch.empty((rows, hq * hd), dtype=torch.bfloat16, device=DEV)
    akvs.akvs_sparse_query_attention(to_dev(q), to_dev(pos), rows, to_dev(k), to_dev(v), n_keys, m,
                                     out, ws)
    some = np.arange(0, rows, 4)
    ref = oracle.attention(f64(q)[some], pos[some], f64(k), f64(v),
                           np.arange(n_keys)).reshape(len(some), -1)
    assert np.linalg.norm(f64(out)[some] - ref) < 2.5e-3 * np.linalg.norm(ref)


@pytest.mark.parametrize("hd,rows,n_keys", [(128, 40, 4500), (64, 300, 1300)])
def test_attention_pieces_of_any_magnitude(hd, rows, n_keys):
    """Values far outside the range of fp16 in either direction, one KV head each: the partial
    outputs of the pieces keep bf16's range."""
    scales = [1.0, 1e6, 3e4, 1e-5, 1e30, 1e-30]
    hkv, hq = len(scales), 2 * len(scales)
    rng = np.random.default_rng(hd)
    pos = np.sort(rng.choice(n_keys, size=rows, replace=False)).astype(np.int32)
    q, k, v = (storage_round(synthetic.random_array((n, h, hd), 95 + i), torch.bfloat16)
               for i, (n, h) in enumerate([(rows, hq), (n_keys, hkv), (n_keys, hkv)]))
    v = (v.float() * torch.tensor(scales)[None, :, None]).to(torch.bfloat16)
    m = akvs.ModelCfg(1, 64, hq, hkv, hd, 64, 16, 1e4, 1e-6, akvs.AKVS_BF16)
    nbytes = akvs.akvs_attention_workspace_size(m, rows, n_keys)
    assert nbytes > 0
    out = torch.empty((rows, hq, hd), dtype=torch.bfloat16, device=DEV)
    akvs.akvs_sparse_query_attention(to_dev(q), to_dev(pos), rows, to_dev(k), to_dev(v), n_keys, m,
                                     out, torch.empty(nbytes, dtype=torch.uint8, device=DEV))
    some = np.arange(0, rows, 3)
    ref = oracle.attention(f64(q)[some], pos[some], f64(k), f64(v), np.arange(n_keys))
    got = f64(out)[some]
    for h in range(hq):
        assert max_rel(got[:, h], ref.reshape(len(some), hq, hd)[:, h]) < 1e-2
