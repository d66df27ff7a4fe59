"""Kernels at the sizes where a tile, a remainder or a dispatch rule ends, through the engine, against the oracle.

Every check is teacher-forced on the engine's own tokens (tests.gpu_helpers.compare): 1e-4 for fp32 engines, 2e-2 for
bf16 ones against the oracle with a bf16 K/V cache, the bounds of the other GPU tests."""
import numpy as np
import pytest

from moa_inputs import ModelShape, f32_to_bf16_bits, generate_weights, pack_blob
from moa_inputs.configs import EngineConsts
from paper_2606_03014_amd import Engine
from tests.gpu_helpers import compare, run_requests

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need the MI355X"


def _check(shape, dtype, lens, G, seed, models=1, consts=None):
    ws = [generate_weights(shape, dtype, seed, 97, m) for m in range(models)]
    rng = np.random.default_rng([seed, 13])
    reqs = [(rng.integers(0, shape.vocab, n).astype(np.int32), i % models, G) for i, n in enumerate(lens)]
    consts = consts or EngineConsts(num_kv_blocks=256, max_num_seqs=max(8, len(lens)), max_prefill_tokens=96,
                                    max_model_len=512)
    toks, logs = run_requests(shape, dtype, consts, ws, reqs)
    for i, (p, m, _) in enumerate(reqs):
        compare(shape, ws[m], p, toks[i], logs[i], dtype == "bf16", 1e-4 if dtype == "f32" else 2e-2,
                what=f"call {i} ({len(p)} tokens)", report_pure=False)


# fp32 GEMM: K = 64 (one 16-k step per wave), 256 and 320; one to 33 rows in a step (16-row chunks and their
# remainders); a vocabulary past 1,024 64-column items takes the four-tile variant
@pytest.mark.parametrize("ffn,vocab,lens", [(64, 64, [1]), (320, 192, [16, 1, 17]), (64, 65600, [33, 5])])
def test_fp32_gemm_edges(ffn, vocab, lens):
    shape = ModelShape(n_layers=1, d_model=256, n_heads=1, n_kv_heads=1, head_dim=64, ffn_dim=ffn, vocab=vocab)
    _check(shape, "f32", lens, 3, seed=ffn + vocab, models=min(2, len(lens)))


def _mix(x):
    for shift, mul in ((16, 0x7FEB352D), (15, 0x846CA68B)):
        x = ((x ^ (x >> np.uint64(shift))) * np.uint64(mul)) & np.uint64(0xFFFFFFFF)
    return x ^ (x >> np.uint64(16))


def _hash_history(shape, dtype, tag, ctx):
    """The device-filled history as a host array [n_layers, 2, ctx, n_kv, head_dim]."""
    u64, m32 = np.uint64, np.uint64(0xFFFFFFFF)
    plane = np.arange(2 * shape.n_layers, dtype=u64).reshape(-1, 1, 1)
    pos = np.arange(ctx, dtype=u64).reshape(1, -1, 1)
    el = np.arange(shape.n_kv_heads * shape.head_dim, dtype=u64).reshape(1, 1, -1)
    u = _mix((u64(tag * 0x9E3779B9) & m32) ^ _mix((plane << u64(24)) ^ pos) ^ ((el * u64(0x85EBCA6B)) & m32))
    v = ((u >> u64(8)).astype(np.float32) / np.float32(8388608.0) - np.float32(1.0))
    v = v.reshape(shape.n_layers, 2, ctx, shape.n_kv_heads, shape.head_dim)
    return f32_to_bf16_bits(v) if dtype == "bf16" else v


# one launch fills every admitted history (KV blocks that are whole, part and absent; several admissions in one step
# and, with three seats, in later ones), one uploads their tokens and block lists, one gathers the tokens
@pytest.mark.parametrize("dtype,hd", [("f32", 64), ("bf16", 64), ("f32", 128), ("bf16", 128)])
@pytest.mark.parametrize("seats", [3, 16])
def test_device_filled_histories_equal_uploaded_ones(dtype, hd, seats):
    shape = ModelShape(n_layers=2, d_model=256, n_heads=4, n_kv_heads=2, head_dim=hd, ffn_dim=256, vocab=512)
    w = generate_weights(shape, dtype, 4, 97, 0)
    ctxs = [0, 1, 15, 16, 17, 31, 255, 256, 257, 40]
    consts = EngineConsts(num_kv_blocks=256, max_num_seqs=seats, max_prefill_tokens=64, max_model_len=2048)
    prompt = np.random.default_rng(8).integers(0, shape.vocab, 1500).astype(np.int32)    # past one copied run
    got = []
    for upload in (False, True):
        eng = Engine(shape, dtype, consts, 1)
        try:
            mid = eng.load(pack_blob(w, shape))
            caps, rids = [], []
            for i, n in enumerate(ctxs):
                kv = _hash_history(shape, dtype, i, n) if upload and n else None
                rids.append(eng.submit_with_history(mid, 5 * i, n, 3, kv))
                caps.append(np.full(3 * shape.vocab, np.nan, dtype=np.float32))
                eng.capture_logits(rids[-1], caps[-1])
            rids.append(eng.submit(prompt, mid, 4))
            while eng.step().step >= 0:
                pass
            out = {r[0]: r[3] for r in eng.collect()}
            eng.sync()
            got.append(([out[r] for r in rids], caps))
        finally:
            eng.close()
    for i in range(len(ctxs)):
        assert np.all(np.isfinite(got[0][1][i]))
        assert np.array_equal(got[0][1][i], got[1][1][i]), f"history of {ctxs[i]}: logits differ"
    for a, b in zip(got[0][0], got[1][0]):
        assert np.array_equal(a, b)


# small-M GEMM: 1, 8, 9, 16, 17, 32 and 33 rows of a model beside another with fewer or more; splits of one to eleven
# four-k-step stages (ffn 1408 has no split), a qkv width that is no multiple of 256 (384). The one-row batch alone has
# its layers on the row GEMMs and only its head here
@pytest.mark.parametrize("rows", [(1,), (1, 7), (8, 3), (9, 2), (16, 1), (17, 8), (32,), (33, 5), (64, 16), (65,)])
@pytest.mark.parametrize("d,ffn,nh,nkv", [(256, 1408, 4, 1), (1024, 512, 2, 2), (512, 128, 8, 2)])
def test_bf16_gemm_small_rows(rows, d, ffn, nh, nkv):
    shape = ModelShape(n_layers=1, d_model=d, n_heads=nh, n_kv_heads=nkv, head_dim=64, ffn_dim=ffn, vocab=1152)
    ws = [generate_weights(shape, "bf16", d + ffn, 97, m) for m in range(len(rows))]
    rng = np.random.default_rng(list(rows))
    reqs = [(rng.integers(0, shape.vocab, 1 + (i % 3)).astype(np.int32), m, 2) for m, r in enumerate(rows)
            for i in range(r)]
    consts = EngineConsts(num_kv_blocks=256, max_num_seqs=96, max_prefill_tokens=256, max_model_len=64)
    toks, logs = run_requests(shape, "bf16", consts, ws, reqs)
    for i in sorted({0, 1, 7, 8, len(reqs) // 2, len(reqs) - 2, len(reqs) - 1}):
        if 0 <= i < len(reqs):
            compare(shape, ws[reqs[i][1]], reqs[i][0], toks[i], logs[i], True, 2e-2, what=f"{rows} call {i}",
                    report_pure=False)


# large-M GEMM: chunks of 128 rows and a part, K of 4 k-steps (ffn 128, fewer than a split keeps), k-splits of uneven
# length, 256- and 512-column tiles, a second model with a few rows in the same launches
@pytest.mark.parametrize("rows", [(256,), (257, 3), (385,), (300, 290)])
@pytest.mark.parametrize("d,ffn", [(256, 128), (1024, 768)])
def test_bf16_gemm_large_rows(rows, d, ffn):
    shape = ModelShape(n_layers=1, d_model=d, n_heads=4, n_kv_heads=2, head_dim=64, ffn_dim=ffn, vocab=512)
    consts = EngineConsts(num_kv_blocks=256, max_num_seqs=8, max_prefill_tokens=1024, max_model_len=512)
    _check(shape, "bf16", rows, 2, seed=sum(rows) + d, models=len(rows), consts=consts)


# row GEMMs (steps of up to six rows over all models) and the step on either side of that: K of 4 k-steps (one split),
# both head widths, one to eight query heads per KV head, prompts of one to three tokens prefilled in such steps, one
# model and three on two streams. Every norm has gains of its own: another layer's, another model's or another column's
# would show
@pytest.mark.parametrize("rows", [(1,), (2, 3, 1), (6,), (7,), (4, 3)])
@pytest.mark.parametrize("d,ffn,nh,nkv,hd", [(256, 128, 8, 1, 64), (512, 1408, 2, 2, 128), (2048, 256, 16, 8, 128)])
def test_bf16_row_gemms(rows, d, ffn, nh, nkv, hd):
    shape = ModelShape(n_layers=2, d_model=d, n_heads=nh, n_kv_heads=nkv, head_dim=hd, ffn_dim=ffn, vocab=512)
    ws = [generate_weights(shape, "bf16", d + ffn, 97, m) for m in range(len(rows))]
    rng = np.random.default_rng(list(rows))
    for w in ws:
        for n in w:
            if n.endswith("norm"):
                w[n] = f32_to_bf16_bits(rng.uniform(0.25, 1.75, d).astype(np.float32))
    reqs = [(rng.integers(0, shape.vocab, 1 + (i + m) % 3).astype(np.int32), m, 4) for m, r in enumerate(rows)
            for i in range(r)]
    consts = EngineConsts(num_kv_blocks=64, max_num_seqs=8, max_prefill_tokens=6, max_model_len=64)
    toks, logs = run_requests(shape, "bf16", consts, ws, reqs)
    one, logs1 = run_requests(shape, "bf16", consts, ws, reqs, one_stream=True)
    for i, (p, m, _) in enumerate(reqs):
        compare(shape, ws[m], p, toks[i], logs[i], True, 2e-2, what=f"{rows} call {i}", report_pure=False)
        assert np.array_equal(toks[i], one[i]) and np.array_equal(logs[i], logs1[i])


# prefill attention: key tiles of 32 and row tiles of 32 and 128 with their edges, one tile alone, both head widths, chunks
# of 96 rows that begin inside a tile's block; with W_q times 32 the scores spread over tens of log2 units, so that rows'
# reference maxima move in later tiles and probabilities reach 2^8
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("lens", [(1, 31, 32, 33), (63, 64, 65, 97), (127, 128, 129, 161), (300,)])
@pytest.mark.parametrize("sharp", [False, True])
def test_prefill_attention_tiles(hd, lens, sharp):
    shape = ModelShape(n_layers=1, d_model=512, n_heads=4, n_kv_heads=2, head_dim=hd, ffn_dim=256, vocab=512)
    w = generate_weights(shape, "bf16", 11, 97, 0)
    if sharp:
        q = [n for n in w if n.endswith("wq")]
        assert len(q) == 1
        w[q[0]] = np.where(w[q[0]] & 0x7f80, w[q[0]] + np.uint16(5 << 7), w[q[0]]).astype(np.uint16)
    for budget in (96, 512):
        consts = EngineConsts(num_kv_blocks=128, max_num_seqs=8, max_prefill_tokens=budget, max_model_len=512)
        rng = np.random.default_rng(list(lens))
        reqs = [(rng.integers(0, shape.vocab, n).astype(np.int32), 0, 2) for n in lens]
        toks, logs = run_requests(shape, "bf16", consts, [w], reqs)
        for i, (p, _, _) in enumerate(reqs):
            compare(shape, w, p, toks[i], logs[i], True, 2e-2, what=f"{len(p)} tokens, budget {budget}",
                    report_pure=False)
